// Tile processing order for the compositing kernels: tiles by descending
// list length (in buckets of 16 instances, capped at 255 buckets), ties by
// tile index, so the longest lists are dispatched first and the short ones
// fill the machine behind them.  One workgroup runs a stable counting sort on
// the key 255 - bucket: each of the 16 wavefronts owns a contiguous range of
// tile ids and walks it 64 tiles at a time; lanes with equal keys find each
// other with eight ballots (one per key bit), so a lane's rank among equal
// keys is a popcount and no atomics are needed.  The result is fully
// determined.  Up to kOrderMax tiles; beyond that the order is the identity.
#pragma once
#include "sort.h"

namespace xgs {

constexpr int kOrderMax = 16384;
constexpr int kOrderWaves = 16;
constexpr int kOrderThreads = 64 * kOrderWaves;
// per wavefront and key a counter, then four wavefront sums
constexpr size_t kOrderLdsBytes = (kOrderWaves * 256 + 4) * sizeof(uint32_t);

// For a lane in `valid`: the lanes of `valid` whose key equals its own.
__device__ __forceinline__ uint64_t same_key_lanes(uint32_t key, uint64_t valid) {
    // one key across the valid lanes (runs of empty tiles): no bit ballots
    const uint32_t k0 = __builtin_amdgcn_readlane(key, valid ? __builtin_ctzll(valid) : 0);
    if (__ballot(((valid >> __lane_id()) & 1ull) && key != k0) == 0ull) return valid;
    uint64_t m = valid;
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
        const bool on = (key >> bit) & 1u;
        const uint64_t bl = __ballot(on);
        m &= on ? bl : ~bl;
    }
    return m;
}

// Run by one workgroup of kOrderThreads threads; len(i) is the length of tile
// i's list and lds holds kOrderLdsBytes that nobody else uses.
template <class Len>
__device__ __forceinline__ void order_tiles(int T, uint32_t* __restrict__ order, uint32_t* lds, Len len) {
    constexpr int kIters = kOrderMax / kOrderThreads;  // 64-tile steps per wavefront
    uint32_t(*cnt)[256] = reinterpret_cast<uint32_t(*)[256]>(lds);  // count, then next output slot
    uint32_t* ws = lds + kOrderWaves * 256;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int i = t; i < kOrderWaves * 256; i += kOrderThreads) lds[i] = 0;
    const int per = (T + kOrderWaves - 1) / kOrderWaves;
    const int lo = min(T, w * per), hi = min(T, lo + per);
    const uint64_t lt = (1ull << lane) - 1ull;
    // every key of the wavefront's range is loaded up front (in-bounds
    // clamped reads past the range, ignored): a load per 64-tile step would
    // put a full memory latency in front of each step, twice
    uint32_t key[kIters];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
        const int i = lo + it * 64 + lane;
        const uint32_t l = len(min(i, T - 1));
        key[it] = i < hi ? 255u - min(l >> 4, 255u) : 0u;
    }
    __syncthreads();
    // rank among the step's equal keys (bits 0-7) and their number (bits 8-15)
    uint32_t rc[kIters];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
        if (lo + it * 64 >= hi) break;  // uniform across the wavefront
        const bool ok = lo + it * 64 + lane < hi;
        const uint64_t m = same_key_lanes(key[it], __ballot(ok));
        const uint32_t rank = (uint32_t)__popcll(m & lt), same = (uint32_t)__popcll(m);
        rc[it] = rank | (same << 8);
        if (ok && rank == 0) cnt[w][key[it]] += same;
    }
    __syncthreads();
    // exclusive prefix over keys of the totals (four wavefront scans), then
    // over waves within a key
    uint32_t s = 0, incl = 0;
    if (t < 256) {
#pragma unroll
        for (int v = 0; v < kOrderWaves; ++v) s += cnt[v][t];
        incl = wave_incl_scan(s, lane);
        if (lane == 63) ws[w] = incl;
    }
    __syncthreads();
    if (t < 256) {
        uint32_t pre = incl - s;  // tiles with a smaller key
#pragma unroll
        for (int k = 0; k < 4; ++k) pre += k < w ? ws[k] : 0u;
#pragma unroll
        for (int v = 0; v < kOrderWaves; ++v) {
            const uint32_t c = cnt[v][t];
            cnt[v][t] = pre;
            pre += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
        if (lo + it * 64 >= hi) break;
        const int i = lo + it * 64 + lane;
        const bool ok = i < hi;
        const uint32_t base = ok ? cnt[w][key[it]] : 0u;
        const uint32_t pos = base + (rc[it] & 0xFFu);
        if (ok && pos < (uint32_t)T) order[pos] = (uint32_t)i;
        // every lane has read its base before the group leader advances it
        if (ok && (rc[it] & 0xFFu) == 0) cnt[w][key[it]] = base + (rc[it] >> 8);
    }
}

}  // namespace xgs
