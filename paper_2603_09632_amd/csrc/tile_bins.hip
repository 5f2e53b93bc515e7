// a2, tile sort by binning: the (tile, Gaussian) instances are counted per
// tile, dropped into their tile's segment and sorted there by (depth,
// Gaussian).  Five launches: count, scan, scatter, sort, and a merge that only
// lists above 2,048 instances need (a second one above 2M).
//
// A radix sort over the 41-46 key bits moves every pair five or six times and
// takes 19 dependent launches, whose latency alone was most of its time.  The
// tile is the upper part of the key and takes few values, so one pass with one
// digit per tile groups the pairs, and what is left is many short independent
// sorts of unique keys: the order within a segment before its sort does not
// matter, so the scatter needs no stable ranking.
//
// What bounds it: the latency of five launches and, in each, of a chain of two
// or three memory accesses; the 8-byte writes of the scatter go to as many
// cache lines as there are pairs.  Measured whole, radix form -> this form:
// 1M Gaussians in 3,225 tiles with 656k instances 125 -> 45 us; 123k Gaussians
// in 315 tiles with 50k instances 78 -> 22 us.
#include <algorithm>

#include "order.h"
#include "sort.h"
#include "tile_bins.h"
#include "wave.h"

namespace xgs {

// A Gaussian's rectangle and count, read together (a rectangle is only
// meaningful where the count is not 0), and its depth.
struct BinItem {
    uint2 r;
    uint32_t cnt, d;
};

__device__ __forceinline__ BinItem bin_item(int64_t i, int64_t end, const uint2* __restrict__ tile_rect,
                                            const uint32_t* __restrict__ touched) {
    BinItem o;
    o.r = make_uint2(0u, 0u);
    o.cnt = o.d = 0u;
    if (i < end) {
        o.r = tile_rect[i];
        o.cnt = touched[i];
    }
    return o;
}

// Calls f(tile, lane that owns it, its depth) for each tile of the lane's
// item, row by row of its rectangle; each f of a group of GROUP first gets
// its tile's slot (take), then uses it (put), so that the slots' latencies
// overlap.  A lane walks a list of up to kOwnTiles itself; the tiles of a
// longer one are spread over the wavefront, so that one splat over the whole
// image does not hold up 63 others.
constexpr uint32_t kOwnTiles = 32;

template <class Take, class Put>
__device__ __forceinline__ void for_tiles(const BinItem& o, uint32_t tiles_x, uint32_t tiles, Take take, Put put) {
    constexpr int GROUP = 4;
    const int lane = threadIdx.x & 63;
    const bool own = o.cnt <= kOwnTiles;
    if (own) {
        const uint32_t x0 = o.r.x & 0xFFFFu, x1 = o.r.y & 0xFFFFu;
        uint32_t row = (o.r.x >> 16) * tiles_x, x = x0;
        for (uint32_t k = 0; k < o.cnt; k += GROUP) {
            uint32_t slot[GROUP];
            bool ok[GROUP];
#pragma unroll
            for (int j = 0; j < GROUP; ++j) {
                const uint32_t tile = row + x;
                ok[j] = k + j < o.cnt && tile < tiles;
                if (ok[j]) slot[j] = take(tile);
                if (++x >= x1) {
                    x = x0;
                    row += tiles_x;
                }
            }
#pragma unroll
            for (int j = 0; j < GROUP; ++j)
                if (ok[j]) put(slot[j], lane, o.d);
        }
    }
    for (uint64_t m = __ballot(!own); m; m &= m - 1) {
        const int src = __builtin_ctzll(m);
        const uint32_t rx = __builtin_amdgcn_readlane(o.r.x, src), ry = __builtin_amdgcn_readlane(o.r.y, src);
        const uint32_t c = __builtin_amdgcn_readlane(o.cnt, src), ds = __builtin_amdgcn_readlane(o.d, src);
        const uint32_t x0 = rx & 0xFFFFu, y0 = rx >> 16, wd = max((ry & 0xFFFFu) - x0, 1u);
        for (uint32_t k = lane; k < c; k += 64) {
            const uint32_t tile = (y0 + k / wd) * tiles_x + x0 + k % wd;
            if (tile < tiles) put(take(tile), src, ds);
        }
    }
}

// Block b: instances per tile of Gaussians [b chunk, (b + 1) chunk), counted
// in LDS and written as row b of hist.
__global__ void __launch_bounds__(kBinThreads) bin_count_kernel(
    int64_t n, int64_t chunk, const uint2* __restrict__ tile_rect, const uint32_t* __restrict__ touched, int tiles_x,
    int T, uint32_t* __restrict__ hist) {
    extern __shared__ uint32_t cnt[];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = min(n, i0 + chunk);
    int64_t base = i0 + 64 * w;  // the next round's items are read ahead of the current round
    BinItem item = bin_item(base + lane, i1, tile_rect, touched);
    for (int k = t; k < T; k += kBinThreads) cnt[k] = 0u;
    __syncthreads();
    for (; base < i1; base += kBinThreads) {
        const BinItem cur = item;
        item = bin_item(base + kBinThreads + lane, i1, tile_rect, touched);
        for_tiles(cur, (uint32_t)tiles_x, (uint32_t)T,
                  [&](uint32_t tile) { atomicAdd(&cnt[tile], 1u); return 0u; }, [](uint32_t, int, uint32_t) {});
    }
    __syncthreads();
    uint32_t* row = hist + (size_t)blockIdx.x * T;
    for (int k = t; k < T; k += kBinThreads) row[k] = cnt[k];
}

// Workgroup g: tiles [64 g, 64 g + 64), one per lane; wavefront s takes the
// s-th sixteenth of the blocks.  Turns each tile's counts into their exclusive
// prefix over the blocks, in place, and writes the tile's total.  Every count
// is loaded before the first is added.
__global__ void __launch_bounds__(kBinThreads) bin_scan_kernel(uint32_t* __restrict__ hist, int blocks, int T,
                                                              uint32_t* __restrict__ totals) {
    constexpr int PER = kBinMaxBlocks / kBinWaves;
    __shared__ uint32_t part[kBinWaves][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int tile = blockIdx.x * 64 + lane;
    const int per = (blocks + kBinWaves - 1) / kBinWaves;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int b = w * per + k;
        v[k] = (k < per && b < blocks && tile < T) ? hist[(size_t)b * T + tile] : 0u;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) sum += v[k];
    part[w][lane] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (int k = 0; k < kBinWaves; ++k) {
        const uint32_t x = part[k][lane];
        run += k < w ? x : 0u;
        total += x;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int b = w * per + k;
        if (k < per && b < blocks && tile < T) hist[(size_t)b * T + tile] = run;
        run += v[k];
    }
    if (w == 0 && tile < T) totals[tile] = total;
}

// Block b < blocks drops its Gaussians' instances into their tiles' segments:
// the next slot of each tile (its first position in the list, from a scan of
// the totals that every block does for itself, plus the block's offset within
// the tile) sits in LDS.  Block 0 also writes ranges, count and status; the
// block after the last writes the runs of the long lists and the tile order.  More instances than cap: the
// lists are empty and status says why.
__global__ void __launch_bounds__(kBinThreads) bin_scatter_kernel(
    int64_t n, int64_t chunk, const uint2* __restrict__ tile_rect, const uint32_t* __restrict__ touched,
    const float4* __restrict__ splat, int tiles_x, int T, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ totals, int blocks, int64_t cap, uint64_t* __restrict__ pairs,
    uint32_t* __restrict__ ranges, int64_t* __restrict__ count, int32_t* __restrict__ status,
    uint32_t* __restrict__ order, uint2* __restrict__ runs, uint32_t* __restrict__ n_runs) {
    extern __shared__ uint32_t pos[];
    __shared__ uint32_t wtot[kBinWaves];
    __shared__ float wabout[kBinWaves];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    // wavefront w scans its run of tiles 64 at a time, then adds the runs
    // before it; every total and offset is loaded before the first is used
    constexpr int STEPS = kBinMaxTiles / kBinThreads;
    const int per = ((T + kBinWaves - 1) / kBinWaves + 63) / 64 * 64;
    const int lo = min(T, w * per), hi = min(T, lo + per);
    const bool last = (int)blockIdx.x == blocks;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = min(n, i0 + chunk);  // empty for the last block
    const float* depth = reinterpret_cast<const float*>(splat);
    int64_t at = i0 + 64 * w;
    BinItem item = bin_item(at + lane, i1, tile_rect, touched);
    const uint32_t* row = hist + (size_t)(last ? 0 : blockIdx.x) * T;
    uint32_t tv[STEPS], off[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int k = lo + 64 * j + lane;
        tv[j] = k < hi ? totals[k] : 0u;
        off[j] = k < hi ? row[k] : 0u;
    }
    // The positions fit 32 bits wherever they are used, but the total that says
    // so may not (64 tiles of 2^26 instances each make 2^32): a sum in floats, right
    // to some millionths, tells whether it does.
    float about = 0.f;
    uint32_t first[STEPS], carry = 0;
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        if (lo + 64 * j >= hi) break;  // uniform across the wavefront
        const uint32_t incl = wave_incl_scan(tv[j], lane);
        first[j] = carry + incl - tv[j];
        carry += __builtin_amdgcn_readlane(incl, 63);
        about += (float)tv[j];
    }
    about = wave_sum(about);
    if (lane == 0) {
        wtot[w] = carry;
        wabout[w] = about;
    }
    __syncthreads();
    uint32_t base = 0, total = 0;
    about = 0.f;
#pragma unroll
    for (int k = 0; k < kBinWaves; ++k) {
        const uint32_t x = wtot[k];
        base += k < w ? x : 0u;
        total += x;
        about += wabout[k];
    }
    // (the capacity is below 2^28)
    const bool over = about > 0x1p31f || total > (uint32_t)cap;
    if (last) {
        // the runs of the lists above kBinBlockKeys
        uint32_t nr[STEPS], mine = 0;
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            nr[j] = !over && tv[j] > (uint32_t)kBinBlockKeys ? (tv[j] + kBinBlockKeys - 1) / kBinBlockKeys : 0u;
            mine += nr[j];
        }
        const uint32_t incl = wave_incl_scan(mine, lane);
        __syncthreads();
        if (lane == 63) wtot[w] = incl;
        __syncthreads();
        uint32_t to = incl - mine, all = 0;
#pragma unroll
        for (int k = 0; k < kBinWaves; ++k) {
            to += k < w ? wtot[k] : 0u;
            all += wtot[k];
        }
#pragma unroll
        for (int j = 0; j < STEPS; ++j)
            for (uint32_t q = 0; q < nr[j]; ++q)
                runs[to++] = make_uint2((uint32_t)(lo + 64 * j + lane), q * kBinBlockKeys);
        if (t == 0) *n_runs = all;
        if (order) order_tiles(T, order, pos, [&](int i) { return over ? 0u : totals[i]; });
        return;
    }
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int k = lo + 64 * j + lane;
        if (lo + 64 * j >= hi) break;
        if (k >= hi) continue;
        const uint32_t at0 = first[j] + base;
        if (blockIdx.x == 0) {
            const uint32_t len = over ? 0u : tv[j];
            ranges[2 * k] = len ? at0 : 0u;
            ranges[2 * k + 1] = len ? at0 + len : 0u;
        }
        pos[k] = at0 + off[j];
    }
    if (blockIdx.x == 0 && t == 0) {
        *count = over ? 0 : (int64_t)total;
        *status = over ? 1 : 0;
    }
    if (over) return;  // uniform over the grid
    __syncthreads();
    for (; at < i1; at += kBinThreads) {
        BinItem cur = item;
        // few Gaussians of a scene are in view: their depths alone are read
        if (cur.cnt) cur.d = __float_as_uint(depth[8 * (at + lane) + 6]);
        item = bin_item(at + kBinThreads + lane, i1, tile_rect, touched);
        for_tiles(cur, (uint32_t)tiles_x, (uint32_t)T, [&](uint32_t tile) { return atomicAdd(&pos[tile], 1u); },
                  [&](uint32_t to, int src, uint32_t d) { pairs[to] = ((uint64_t)d << 32) | (uint32_t)(at + src); });
    }
}

// Value of the lane whose index differs in the bits of D.
template <int D>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v, int lane) {
    if constexpr (D == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);        // quad_perm 1 0 3 2
    else if constexpr (D == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad_perm 2 3 0 1
    else if constexpr (D == 3) return __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, true);   // quad_perm 3 2 1 0
    else if constexpr (D == 7) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);  // row_half_mirror
    else if constexpr (D == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);  // row_ror:8
    else if constexpr (D == 15) return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true); // row_mirror
    else if constexpr (D == 4) return xor_lane<3>(xor_lane<7>(v, lane), lane);
    else if constexpr (D == 16 || D == 32) return (uint32_t)xlane_partner<D>((int)v, lane);
    else if constexpr (D == 31) return xor_lane<16>(xor_lane<15>(v, lane), lane);
    else return xor_lane<32>(xor_lane<31>(v, lane), lane);
}

// Exchange with the partner lane: the lane without D's top bit keeps the
// smaller key.  FLIP: element e meets element E - 1 - e of the partner.
template <int E, int D, bool FLIP>
__device__ __forceinline__ void lane_step(uint64_t (&k)[E], int lane) {
    constexpr int TOP = D & 32 ? 32 : D & 16 ? 16 : D & 8 ? 8 : D & 4 ? 4 : D & 2 ? 2 : 1;
    const bool upper = (lane & TOP) != 0;
    uint64_t o[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const uint64_t v = k[FLIP ? E - 1 - e : e];
        o[e] = ((uint64_t)xor_lane<D>((uint32_t)(v >> 32), lane) << 32) | xor_lane<D>((uint32_t)v, lane);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] = (o[e] < k[e]) != upper ? o[e] : k[e];
}

template <int E>
__device__ __forceinline__ void reg_step(uint64_t (&k)[E], int a, int b) {
    const uint64_t lo = k[a] < k[b] ? k[a] : k[b], hi = k[a] < k[b] ? k[b] : k[a];
    k[a] = lo;
    k[b] = hi;
}

// Half-cleaners at distances J, J / 2, ..., 1 (element index = lane E + e).
template <int E, int J>
__device__ __forceinline__ void clean(uint64_t (&k)[E], int lane) {
    if constexpr (J >= E) {
        lane_step<E, J / E, false>(k, lane);
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((e & J) == 0) reg_step<E>(k, e, e | J);
    }
    if constexpr (J > 1) clean<E, J / 2>(k, lane);
}

// Merges sorted runs of R / 2 elements into runs of R, up to 64 E: the first
// step compares mirrored positions, so every run stays ascending.
template <int E, int R>
__device__ __forceinline__ void merge_runs(uint64_t (&k)[E], int lane) {
    if constexpr (R <= E) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((e & (R / 2)) == 0) reg_step<E>(k, e, e ^ (R - 1));
    } else {
        lane_step<E, R / E - 1, true>(k, lane);
    }
    if constexpr (R > 2) clean<E, R / 4 ? R / 4 : 1>(k, lane);
    if constexpr (R < 64 * E) merge_runs<E, 2 * R>(k, lane);
}

// Sorts the m <= 64 E pairs at src; sink(position, pair) receives them.
template <int E, class Sink>
__device__ __forceinline__ void sort_wave(const uint64_t* __restrict__ src, int m, int lane, Sink sink) {
    uint64_t k[E];
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] = 64 * e + lane < m ? src[64 * e + lane] : ~0ull;
    merge_runs<E, 2>(k, lane);
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (lane * E + e < m) sink(lane * E + e, k[e]);
}

template <class Sink>
__device__ __forceinline__ void sort_wave_upto(const uint64_t* src, int m, int lane, Sink sink) {
    static_assert(kBinWaveKeys == 256, "the largest form below");
    if (m <= 64) sort_wave<1>(src, m, lane, sink);
    else if (m <= 128) sort_wave<2>(src, m, lane, sink);
    else sort_wave<4>(src, m, lane, sink);
}

// Exchange across wavefronts through LDS: element g meets element g ^ M, and
// the half without M's top bit keeps the smaller one.
template <int E>
__device__ __forceinline__ void block_step(uint64_t (&k)[E], uint64_t* lds, uint32_t M, bool upper) {
    const uint32_t g = threadIdx.x * E;
#pragma unroll
    for (int e = 0; e < E; ++e) lds[g + e] = k[e];
    __syncthreads();
    uint64_t o[E];
#pragma unroll
    for (int e = 0; e < E; ++e) o[e] = lds[(g + e) ^ M];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] = (o[e] < k[e]) != upper ? o[e] : k[e];
}

// Sorts the m <= 256 E pairs at src with one workgroup: the same network, its
// last two merges crossing the four wavefronts.  (Buckets of equal depth
// ranges in LDS were as fast on evenly spread depths and 8 to 20 times slower
// where a tile sees two surfaces.)
template <int E, class Sink>
__device__ __forceinline__ void sort_block(uint64_t* lds, const uint64_t* __restrict__ src, int m, Sink sink) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint64_t k[E];
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] = 256 * e + t < m ? src[256 * e + t] : ~0ull;
    merge_runs<E, 2>(k, lane);
    block_step<E>(k, lds, 128 * E - 1, w & 1);
    clean<E, 32 * E>(k, lane);
    block_step<E>(k, lds, 256 * E - 1, w & 2);
    block_step<E>(k, lds, 64 * E, w & 1);
    clean<E, 32 * E>(k, lane);
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (t * E + e < m) sink(t * E + e, k[e]);
}

template <class Sink>
__device__ __forceinline__ void sort_block_upto(uint64_t* lds, const uint64_t* src, int m, Sink sink) {
    static_assert(kBinBlockKeys == 2048, "the largest form below");
    if (m <= 512) sort_block<2>(lds, src, m, sink);
    else if (m <= 1024) sort_block<4>(lds, src, m, sink);
    else sort_block<8>(lds, src, m, sink);
}

__device__ __forceinline__ void finish_pair(uint64_t* __restrict__ keys, uint32_t* __restrict__ vals, uint32_t at,
                                            uint32_t tile, uint64_t k) {
    keys[at] = ((uint64_t)tile << 32) | (k >> 32);
    vals[at] = (uint32_t)k;
}

// Workgroups [0, longs): the runs of the lists above kBinBlockKeys, sorted in
// place, then the lists above kBinWaveKeys, in tile order or by a stride over
// all tiles.  The others: four tiles each, one per wavefront, sorted in
// registers.
__global__ void __launch_bounds__(256) bin_sort_kernel(uint64_t* __restrict__ pairs, const uint32_t* __restrict__ ranges,
                                                      const uint32_t* __restrict__ order, int T, int longs,
                                                      const uint2* __restrict__ runs, const uint32_t* __restrict__ n_runs,
                                                      uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    __shared__ uint64_t lds[kBinBlockKeys];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if ((int)blockIdx.x >= longs) {
        const int slot = ((int)blockIdx.x - longs) * 4 + w;
        if (slot >= T) return;
        const uint32_t tile = __builtin_amdgcn_readfirstlane(order ? order[slot] : (uint32_t)slot);
        const uint32_t a = __builtin_amdgcn_readfirstlane(ranges[2 * tile]);
        const uint32_t m = __builtin_amdgcn_readfirstlane(ranges[2 * tile + 1]) - a;
        if (m == 0 || m > (uint32_t)kBinWaveKeys) return;
        sort_wave_upto(pairs + a, (int)m, lane, [&](int i, uint64_t k) { finish_pair(keys, vals, a + i, tile, k); });
        return;
    }
    const uint32_t nr = *n_runs;
    for (uint32_t r = blockIdx.x; r < nr; r += longs) {
        const uint32_t tile = runs[r].x, a = ranges[2 * tile] + runs[r].y, end = ranges[2 * tile + 1];
        uint64_t* at = pairs + a;
        sort_block_upto(lds, at, (int)min(end - a, (uint32_t)kBinBlockKeys), [&](int i, uint64_t k) { at[i] = k; });
    }
    for (int slot = blockIdx.x; slot < T; slot += longs) {
        const uint32_t tile = order ? order[slot] : (uint32_t)slot;
        const uint32_t a = ranges[2 * tile], m = ranges[2 * tile + 1] - a;
        // the order is by sixteenths of the length: below this no longer list follows
        if (order && m < (uint32_t)kBinWaveKeys) return;
        if (m <= (uint32_t)kBinWaveKeys || m > (uint32_t)kBinBlockKeys) continue;
        sort_block_upto(lds, pairs + a, (int)m, [&](int i, uint64_t k) { finish_pair(keys, vals, a + i, tile, k); });
    }
}

// Adds to b[] the number of the len ascending elements at(0), at(1), ... below
// each of k[]: three probes a step and key, which do not wait for each other
// (past the end they read the last element, which is not counted).
template <int N, class At>
__device__ __forceinline__ void count_below(uint32_t len, const uint64_t (&k)[N], uint32_t (&b)[N], At at) {
    if (len == 0) return;
    uint32_t p[N] = {};
    for (uint32_t s = 1u << ((31 - __builtin_clz(len)) & ~1); s >= 1; s >>= 2) {
        uint64_t v[N][3];
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (uint32_t q = 0; q < 3; ++q) v[j][q] = at(min(p[j] + (q + 1) * s, len) - 1);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            uint32_t less = 0;
#pragma unroll
            for (uint32_t q = 0; q < 3; ++q) less += p[j] + (q + 1) * s <= len && v[j][q] < k[j] ? s : 0u;
            p[j] += less;
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] += p[j];
}

// Sorts get(0 .. m - 1), m <= 1024 E, with a workgroup of 16 wavefronts; sink(position,
// pair) receives them.
template <int E, class Get, class Sink>
__device__ __forceinline__ void sort_wide(uint64_t* lds, uint32_t m, Get get, Sink sink) {
    const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint64_t k[E];
#pragma unroll
    for (int e = 0; e < E; ++e) k[e] = 1024 * e + t < m ? get(1024 * e + t) : ~0ull;
    merge_runs<E, 2>(k, lane);
#pragma unroll 1
    for (uint32_t r = 2; r <= 16; r *= 2) {  // wavefronts whose pairs are merged
        block_step<E>(k, lds, 64 * E * r - 1, (w & (r / 2)) != 0);
#pragma unroll 1
        for (uint32_t d = r / 4; d >= 1; d /= 2) block_step<E>(k, lds, 64 * E * d, (w & d) != 0);
        clean<E, 32 * E>(k, lane);
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (t * E + e < m) sink(t * E + e, k[e]);
}

// The places of the run at `own` of a list of m pairs: a pair's is its index in its run
// plus the number of smaller ones in each other run, four of which are in LDS at a
// time (8 bytes more every 16 pairs, or the search's strides would meet in one
// bank).
template <class Sink>
__device__ __forceinline__ void rank_run(uint64_t* lds, const uint64_t* __restrict__ list, uint32_t m, uint32_t own,
                                         Sink sink) {
    const uint32_t t = threadIdx.x, mine = min(m - own, (uint32_t)kBinBlockKeys);
    auto at = [&](uint32_t i) -> uint64_t& { return lds[i + (i >> 4)]; };
    uint64_t k[2];
    uint32_t rank[2];
#pragma unroll
    for (uint32_t e = 0; e < 2; ++e) {
        rank[e] = 2 * t + e;
        k[e] = rank[e] < mine ? list[own + rank[e]] : ~0ull;
    }
    for (uint32_t o = 0; o < m; o += kBinMergeKeys) {
        const uint32_t here = min(m - o, (uint32_t)kBinMergeKeys);
#pragma unroll
        for (uint32_t e = 0; e < kBinMergeKeys / 1024; ++e)
            if (1024 * e + t < here) at(1024 * e + t) = list[o + 1024 * e + t];
        __syncthreads();
#pragma unroll
        for (uint32_t v = 0; v < kBinMergeKeys; v += kBinBlockKeys)
            if (v < here && o + v != own)
                count_below(min(here - v, (uint32_t)kBinBlockKeys), k, rank, [&](uint32_t i) { return at(v + i); });
        __syncthreads();
    }
#pragma unroll
    for (uint32_t e = 0; e < 2; ++e)
        if (2 * t + e < mine) sink(rank[e], k[e]);
}

// The lists above kBinBlockKeys.  The first pass makes one of up to kBinFan sorted
// runs: lists of up to kBinFanKeys are done with it, in keys and vals; of longer
// ones it leaves runs of kBinFanKeys in merged, of which the last pass makes one.
//
// A workgroup takes a range of values of about kBinBlockKeys pairs, twice that where
// there are more runs than workgroups (one to a CU): its ends are order statistics of samples, one every 256 pairs of each run (more from 4,096
// samples on; at another offset in each run, so that runs of one profile do not have theirs in
// the same places), its pairs are what each run holds between them, gathered and
// sorted.  A range with more pairs than fit is halved until what is taken does,
// and the rest of it follows: any runs come out sorted, if not as fast.  So a
// pair costs a pass about one sort of 2,048, whatever the length of its list.  Lists of
// up to kBinRankKeys, few runs, are cheaper by ranks.
//
// What bounds it: the steps of the two sorts (16 wavefronts, a barrier for each
// exchange between them) and the scattered loads of the search for the ends.
// Whole sorts in a grid of 3,225 tiles, radix form / ranks in every other run of a
// list, whose cost is the square of its runs / this (us): one list of 30,000 83 / 86
// / 61, of 100,000 85 / 199 / 70, of 1M 157 / 1,752 / 158, of 2M 229 / - / 355, of 5M
// 505 / - / 1,080; four lists of 250,000 157 / 474 / 162.
template <bool LAST>
__global__ void __launch_bounds__(1024) bin_merge_kernel(const uint64_t* __restrict__ src,
                                                        const uint32_t* __restrict__ ranges,
                                                        const uint2* __restrict__ runs,
                                                        const uint32_t* __restrict__ n_runs,
                                                        uint64_t* __restrict__ merged, uint64_t* __restrict__ keys,
                                                        uint32_t* __restrict__ vals) {
    constexpr uint32_t LEN = LAST ? kBinFanKeys : kBinBlockKeys, LOG_LEN = __builtin_ctz(LEN);
    static_assert((LEN & (LEN - 1)) == 0 && LEN >> 8 >= 1, "whole samples a run");
    __shared__ uint64_t lds[kBinMergeKeys + kBinMergeKeys / 16];
    __shared__ uint64_t cut[2];
    __shared__ uint32_t pre[kBinFan], first[kBinFan], wsum[16];
    const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6;
    // exclusive prefix of v over the workgroup, and the total
    auto scan = [&](uint32_t v, uint32_t& total) {
        const uint32_t incl = wave_incl_scan(v, (int)lane);
        __syncthreads();
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t before = incl - v;
        total = 0;
#pragma unroll
        for (uint32_t q = 0; q < 16; ++q) {
            before += q < w ? wsum[q] : 0u;
            total += wsum[q];
        }
        return before;
    };
    const uint32_t units = *n_runs, wide = units > (uint32_t)kBinMaxBlocks ? 1u : 0u;
    // a workgroup's runs: one a round, or two neighbours
    for (uint32_t u = blockIdx.x << wide; u < units; u += wide && !(u & 1) ? 1 : (gridDim.x << wide) - wide) {
        const uint32_t tile = runs[u].x, own = runs[u].y;
        const uint32_t a = ranges[2 * tile], m = ranges[2 * tile + 1] - a;
        // uniform, as all of the control flow below
        if (LAST && m <= (uint32_t)kBinFanKeys) continue;
        if (!LAST && m <= (uint32_t)kBinRankKeys) {
            rank_run(lds, src + a, m, own, [&](uint32_t i, uint64_t k) { finish_pair(keys, vals, a + i, tile, k); });
            continue;
        }
        if (own / kBinBlockKeys & wide) continue;
        const uint32_t group = LAST ? 0u : own / kBinFanKeys * kBinFanKeys;
        const uint32_t size = LAST ? m : min(m - group, (uint32_t)kBinFanKeys);
        const uint32_t n = (size + LEN - 1) / LEN;
        const uint64_t* list = src + a + group;
        // this range's number and theirs, the samples, and those at its ends
        const uint32_t range = kBinBlockKeys << wide, j = (own - group) / range, nb = (size + range - 1) / range;
        uint32_t log_s = 8;
        while (size > 4096u << log_s) ++log_s;
        auto offset = [&](uint32_t r) { return (r * 0x9E3779B1u) >> (32 - log_s); };
        const uint32_t log_per = LOG_LEN - log_s, tail = size - (n - 1) * LEN, o = offset(n - 1);
        const uint32_t samples = ((n - 1) << log_per) + (tail > o ? ((tail - o - 1) >> log_s) + 1 : 0u);
        const uint32_t c0 = (uint32_t)((uint64_t)j * samples / nb), c1 = (uint32_t)((uint64_t)(j + 1) * samples / nb);
        auto sample = [&](uint32_t i) {
            const uint32_t r = i >> log_per;
            return list[r * LEN + ((i - (r << log_per)) << log_s) + offset(r)];
        };
        auto at_cut = [&](uint32_t i, uint64_t k) {
            if (i == c0) cut[0] = k;
            if (i == c1) cut[1] = k;
        };
        __syncthreads();  // the cuts of the range before are read
        if (samples <= 1024) sort_wide<1>(lds, samples, sample, at_cut);
        else if (samples <= 2048) sort_wide<2>(lds, samples, sample, at_cut);
        else sort_wide<4>(lds, samples, sample, at_cut);
        __syncthreads();
        const uint64_t end = j + 1 < nb ? cut[1] : ~0ull;
        uint64_t ends[2] = {j > 0 ? cut[0] : 0ull, end};
        // thread r: the pairs of run r below the two ends
        const uint32_t len = t < n ? min(size - t * LEN, LEN) : 0u;
        const uint64_t* run = list + (t < n ? t : 0u) * LEN;
        uint32_t below[2] = {0u, 0u};
        count_below(len, ends, below, [&](uint32_t i) { return run[i]; });
        uint32_t start;
        scan(below[0], start);
        for (;;) {
            uint32_t count, before = scan(below[1] - below[0], count);
            // pairs are distinct, so that 8,192 neighbouring values fit at the latest (if a
            // caller's rectangles repeat a pair, the bounds below still end the loops)
            while (count > (uint32_t)kBinMergeKeys && ends[1] - ends[0] > 1) {
                ends[1] = ends[0] + (ends[1] - ends[0]) / 2;
                const uint64_t half[1] = {ends[1]};
                uint32_t b[1] = {0u};
                count_below(len, half, b, [&](uint32_t i) { return run[i]; });
                below[1] = b[0];
                before = scan(below[1] - below[0], count);
            }
            if (t < n) {
                pre[t] = before;
                first[t] = t * LEN + below[0];
            }
            __syncthreads();
            auto get = [&](uint32_t i) {
                uint32_t r = 0;  // the last run that starts at or before i
                for (uint32_t q = 1u << (31 - __builtin_clz(n)); q >= 1; q >>= 1)
                    if (r + q < n && pre[r + q] <= i) r += q;
                return list[first[r] + (i - pre[r])];
            };
            const bool final = LAST || m <= (uint32_t)kBinFanKeys;
            const uint32_t to0 = a + group + start;
            auto put = [&](uint32_t i, uint64_t k) {
                const uint32_t to = to0 + i;
                if (!final) merged[to] = k;
                else finish_pair(keys, vals, to, tile, k);
            };
            if (count <= 1024) sort_wide<1>(lds, count, get, put);
            else if (count <= 2048) sort_wide<2>(lds, count, get, put);
            else if (count <= 4096) sort_wide<4>(lds, count, get, put);
            else sort_wide<8>(lds, min(count, (uint32_t)kBinMergeKeys), get, put);
            if (ends[1] == end) break;
            start += count;
            ends[0] = ends[1];
            ends[1] = end;
            below[0] = below[1];
            const uint64_t all[1] = {end};
            uint32_t b[1] = {0u};
            count_below(len, all, b, [&](uint32_t i) { return run[i]; });
            below[1] = b[0];
        }
    }
}

BinWs carve_bins(void* base, int64_t n, int64_t cap, int64_t tiles, size_t* bytes) {
    Carve c(base);
    BinWs w;
    w.pairs = c.take<uint64_t>(cap > 0 ? cap : 1);
    w.hist = c.take<uint32_t>((size_t)bin_plan(n).blocks * (tiles > 0 ? tiles : 1));
    w.totals = c.take<uint32_t>(tiles > 0 ? tiles : 1);
    w.runs = c.take<uint2>(bin_max_runs(cap));
    w.n_runs = c.take<uint32_t>(1);
    w.merged = c.take<uint64_t>(cap > kBinFanKeys ? cap : 0);
    *bytes = c.total();
    return w;
}

bool bins_apply(int64_t n, int64_t cap, int64_t tiles) {
    return n > 0 && n < ((int64_t)1 << 31) && cap > 0 && tiles > 0 && tiles <= kBinMaxTiles &&
           cap / tiles <= kBinMaxMeanList;
}

xgs_status bin_tile_sort(const xgs_projected* p, int64_t n, int tiles_x, int64_t tiles, const BinWs& w,
                         xgs_binning* b, hipStream_t st) {
    const BinPlan pl = bin_plan(n);
    const int T = (int)tiles;
    const uint2* rect = reinterpret_cast<const uint2*>(p->tile_rect);
    const size_t lds = (size_t)T * sizeof(uint32_t);
    hipLaunchKernelGGL(bin_count_kernel, dim3((unsigned)pl.blocks), dim3(kBinThreads), lds, st, n, pl.chunk, rect,
                       p->tiles_touched, tiles_x, T, w.hist);
    hipLaunchKernelGGL(bin_scan_kernel, dim3((unsigned)((T + 63) / 64)), dim3(kBinThreads), 0, st, w.hist, pl.blocks,
                       T, w.totals);
    hipLaunchKernelGGL(bin_scatter_kernel, dim3((unsigned)(pl.blocks + 1)), dim3(kBinThreads),
                       std::max(lds, kOrderLdsBytes), st, n, pl.chunk, rect, p->tiles_touched,
                       reinterpret_cast<const float4*>(p->splat), tiles_x, T, w.hist, w.totals, pl.blocks,
                       b->max_instances, w.pairs, b->ranges, b->num_instances, b->status, b->tile_order, w.runs,
                       w.n_runs);
    const int longs = std::min(T, kBinLongBlocks);
    hipLaunchKernelGGL(bin_sort_kernel, dim3((unsigned)(longs + (T + 3) / 4)), dim3(256), 0, st, w.pairs, b->ranges,
                       b->tile_order, T, longs, w.runs, w.n_runs, b->keys, b->vals);
    auto merge = [&](auto kernel, const uint64_t* src) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min<int64_t>(bin_max_runs(b->max_instances), kBinMergeBlocks)),
                           dim3(1024), 0, st, src, b->ranges, w.runs, w.n_runs, w.merged, b->keys, b->vals);
    };
    if (b->max_instances > kBinBlockKeys) merge(bin_merge_kernel<false>, w.pairs);
    if (b->max_instances > kBinFanKeys) merge(bin_merge_kernel<true>, w.merged);
    return check_launch("xgs_tile_sort bins");
}

}  // namespace xgs
