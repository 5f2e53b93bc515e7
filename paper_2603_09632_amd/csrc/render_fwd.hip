// a3: front-to-back alpha compositing of RGB, depth and semantic channels,
// Eq. (rendering) with the feature and depth substitutions (Sec. 3.1, App. B),
// evaluated only at the sampled grid pixels (App. D): the rasterizer never
// forms the dense map when stride > 1.
#include <algorithm>

#include "render_common.h"

namespace xgs {

// CS: compile-time semantic channel count.  EXACT: csem == CS, so feature
// rows have a compile-time stride and merge into wide scalar loads; otherwise
// CS only bounds csem and channels >= csem are neither read nor written.
//
// A wavefront takes an 8x8 quadrant of a tile.  It reads the tile list 64
// entries at a time (one per lane: list entry and splat record, the record of
// the next 64 and the entries of the 64 after those in flight), keeps the
// splats that can reach alpha >= 1/255 somewhere in its quadrant (quad_hit; the
// others would be skipped by all 64 pixels) and appends them to a ring in LDS;
// the walk then takes the ring 16 at a time.  Eight alphas are formed first (0
// where a pair is skipped), then the chain of T, six instructions a splat: a
// pixel that stops keeps -T, which stops every later step by itself, so the
// chain needs no masks.  The weights w_k(p) = alpha_k T_k go through LDS and the
// channel sums out[p][c] += sum_k w_k(p) chan_k[c] run as a 64 x 16 x COLS product
// on v_mfma_f32_16x16x4_f32 (features first, then colour and depth); a pixel's
// row in LDS holds weight 4 kk + g at 4 g + kk, so that a lane's weights of the
// four steps are one 16-byte read.  Every sum runs in list order, splat by
// splat (the 16x16x4 and 4x4x1 forms both add one rounded product at a time).
// The channel rows are loaded before the
// walk and used after it.  The accumulators hold the wave's output block until
// the end.
//
// What bounds it: the vector and matrix instructions of the walk (on the 1M frame
// below their cycles are 62% and 31% of a SIMD's, and they hardly overlap, at 4
// wavefronts, 3 above 32 channels) and, where few lists are long, the longest
// list's walk.  Measured with masks in scalar
// registers, colour and depth in a tile of 16 columns, one store a pixel and
// channel, and as it is (four pixels of a row are one store): 1M Gaussians, 1200
// x 680, 32 features 155-191 -> 103-143 us by the pose; 300k, 640 x 480, 16
// features 63 -> 45; 123k on a 321 x 240 grid 58 -> 40; 2,000 at 128 x 96 37 -> 22.
//
// BATCH: the tiles of several requests in one launch (serving).  g then
// describes the virtual grid (tx = its width in tiles, tiles = all of it,
// order over it); each workgroup finds its request's slot, takes that slot's
// grid, colours, features and outputs, and reads the tile list of the global
// tile.  Splat records are indexed by global Gaussian index, colours and
// features by index within the slot's scene.
template <int CS, bool EXACT, typename OFF, bool BATCH = false>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(CS > 32 ? 3 : 4))) render_fwd_mfma_kernel(
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ vals,
    const float4* __restrict__ splat, const float* __restrict__ colors,
    const float* __restrict__ features, int csem, TileGrid g, float* __restrict__ out,
    float* __restrict__ final_T, int32_t* __restrict__ n_last, const xgs_batch_slot* __restrict__ slots = nullptr,
    int n_slots = 0) {
    constexpr int CH = 4 + CS;
    // Where the features fill whole tiles, colour and depth are a product of
    // their own (4x4x1, a lane's own weights against the four channels: a quarter
    // of a 16-column tile's cycles); else they share the last tile.
    constexpr bool OWN4 = CS % 16 == 0;
    constexpr int COLS = OWN4 ? CS : CH;
    constexpr int NT = (COLS + 15) / 16;
    constexpr int G = 8;     // alphas formed together
    constexpr int ROW = 20;  // LDS row of a pixel: 16 weights, float4-aligned, banks spread
    __shared__ __align__(16) float wl[64 * ROW];
    __shared__ Ring ring;
    __shared__ __align__(16) float ch4[OWN4 ? 4 * ROW : 4];  // channel c of the batch's 16 splats
    QuadPix P;
    int rtile;  // tile whose list is read (the global tile when batched)
    if constexpr (BATCH) {
        const int slot = quad_slot();
        if (slot >= g.tiles) return;
        rtile = g.order ? (int)uniform(g.order[slot]) : slot;
        BatchTile bt;
        if (!batch_tile(slots, n_slots, g.tx, rtile, bt)) return;
        const xgs_batch_slot& sl = slots[bt.slot];
        // colours and features are indexed by global Gaussian index: shift
        // their bases by the slot's first global index
        const int64_t base = (int64_t)sl.gauss_base;
        colors = reinterpret_cast<const float*>(reinterpret_cast<uintptr_t>(sl.g.colors) -
                                                (uintptr_t)(base * 3 * (int64_t)sizeof(float)));
        features = reinterpret_cast<const float*>(reinterpret_cast<uintptr_t>(sl.g.features) -
                                                  (uintptr_t)(base * (EXACT ? CS : csem) * (int64_t)sizeof(float)));
        out = sl.out;
        final_T = sl.final_T;
        n_last = sl.n_last;
        g = bt.grid;
        P = quad_pixel_at(g, bt.tile, quad_index());
    } else {
        P = quad_pixel(g);
        rtile = P.tile;
    }
    if (P.tile >= g.tiles) return;
    const QuadRect qr = quad_rect(g, P);
    const int lane = threadIdx.x;
    // Column j of the product is feature j, or channel j - CS (colour, depth)
    // past the features.  The columns of the tile where they meet come from one
    // lane-constant source and stride, so that its loads do not branch.
    const int fstr = EXACT ? CS : csem;
    constexpr int MIX = OWN4 ? NT : CS / 16;  // that tile
    static_assert(CS % 16 <= 12, "colour and depth fit the features' last tile: it is the last");
    const int jm = 16 * MIX + (lane & 15);
    const bool mfeat = jm < CS, muse = jm < COLS && (EXACT || jm < csem || jm >= CS);
    const float* const msrc = !muse ? reinterpret_cast<const float*>(splat)
                              : mfeat ? features + jm
                              : jm < CS + 3 ? colors + (jm - CS) : reinterpret_cast<const float*>(splat) + 6;
    const int mstr = !muse ? 8 : mfeat ? fstr : jm < CS + 3 ? 3 : 8;
    f32x4_t acc4 = {0.f, 0.f, 0.f, 0.f};
    f32x4_t acc[4][NT > 0 ? NT : 1];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float T = P.inside ? 1.f : -1.f;  // transmittance; its negative once the pixel has stopped
    int last = 0;
    const uint32_t start = uniform(ranges[2 * rtile]);
    const int len = (int)(uniform(ranges[2 * rtile + 1]) - start);
    if (len > 0) {
        // Candidate registers: splat record c0, c1 and index cg of list position
        // cpos + lane, and the index cn of the position 64 after it (so that a
        // record's load never waits for its list entry).  Positions past the end
        // read the last entry and are not pushed.
        auto entry = [&](int pos) { return (int)vals[start + (uint32_t)min(pos + lane, len - 1)]; };
        int cpos = 0, head = 0, tail = 0;
        bool padded = false;
        int cg = entry(0), cn = entry(64);
        float4 c0 = splat[2 * (uint32_t)cg], c1 = splat[2 * (uint32_t)cg + 1];
        // fills the ring to one batch (or the end of the list)
        auto fill = [&]() {
            while (tail - head < 16 && cpos < len) {
                tail = ring_push(ring, tail, cpos + lane < len && quad_hit(c0, c1, qr), c0, c1, cg, cpos + lane);
                cpos += 64;
                cg = cn;
                c0 = splat[2 * (uint32_t)cg];
                c1 = splat[2 * (uint32_t)cg + 1];
                cn = entry(cpos + 64);
            }
            if (cpos >= len && !padded) {
                padded = true;
                ring_pad(ring, tail, lane, cg);
            }
        };
        for (;;) {
            if (__ballot(T > 0.f) == 0ull) break;
            fill();
            const int nb = min(16, tail - head);
            if (nb == 0) break;
            __syncthreads();
            // channel rows of this batch in B-operand layout: step kk of lane
            // group lane / 16 takes splat 4 kk + lane / 16
            float b[4][NT > 0 ? NT : 1], col = 0.f;
            if constexpr (OWN4)
                col = *at_row<OFF>(colors, (uint32_t)ring.gid[(head + (lane >> 2)) & (kRing - 1)], 3, min(lane & 3, 2));
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const uint32_t gs = (uint32_t)ring.gid[(head + 4 * kk + (lane >> 4)) & (kRing - 1)];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int j = 16 * nt + (lane & 15);
                    if (nt == MIX) b[kk][nt] = msrc[(size_t)gs * mstr];
                    else b[kk][nt] = *at_row<OFF>(features, gs, fstr, EXACT ? j : min(j, csem - 1));
                }
            }
            float w[16];
            int lastk = -1;  // batch index of this pixel's last contributing splat
#pragma unroll
            for (int q = 0; q < 16; q += G) {
                float al[G];
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const int at = (head + q + u) & (kRing - 1);
                    const float4 s0 = ring.rec[at][0];
                    const float2 s1 = *reinterpret_cast<const float2*>(&ring.rec[at][1]);
                    const PairEval e = eval_pair(P.px, P.py, s0.x, s0.y, s0.z, s0.w, s1.x, s1.y);
                    al[u] = e.alpha >= kAlphaMin ? e.alpha : 0.f;
                }
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const float Tn = T * (1.f - al[u]);
                    const bool stop = Tn < kTStop;
                    w[q + u] = stop ? 0.f : al[u] * T;
                    T = stop ? -fabsf(T) : Tn;
                    lastk = w[q + u] > 0.f ? q + u : lastk;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<f32x4_t*>(&wl[lane * ROW + 4 * j]) = f32x4_t{w[j], w[4 + j], w[8 + j], w[12 + j]};
            if (lastk >= 0) last = __float_as_int(ring.rec[(head + lastk) & (kRing - 1)][1].w) + 1;
            if constexpr (OWN4) {
                const float v = (lane & 3) < 3 ? col : ring.rec[(head + (lane >> 2)) & (kRing - 1)][1].z;
                col = (lane >> 2) < nb ? v : 0.f;
                ch4[(lane & 3) * ROW + (lane >> 2)] = col;
            }
            head += nb;
            __syncthreads();
            // masked columns and slots past the batch count as zeros
            float odd = 0.f * col;  // 0, or NaN once a channel is not finite
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int j = 16 * nt + (lane & 15);
                    if (!EXACT || 16 * nt + 16 > COLS)
                        b[kk][nt] = j < COLS && (EXACT || j >= CS || j < csem) ? b[kk][nt] : 0.f;
                    if (nb < 16) b[kk][nt] = 4 * kk + (lane >> 4) < nb ? b[kk][nt] : 0.f;
                    odd += 0.f * b[kk][nt];
                }
            if (__ballot(odd != 0.f) != 0ull) {
                // infinite (or NaN) channels: added by hand to the pixels with a
                // weight for their splat, and taken out of the product, where a
                // weight of zero would not keep them from the others
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        for (int grp = 0; grp < 4; ++grp) {
                            const float v = __shfl(b[kk][nt], 16 * grp + (lane & 15), 64);
                            if (__ballot(!(fabsf(v) < INFINITY)) == 0ull) continue;
#pragma unroll
                            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const float wt = wl[(16 * mt + 4 * (lane >> 4) + r) * ROW + 4 * grp + kk];
                                    if (wt != 0.f && !(fabsf(v) < INFINITY)) acc[mt][nt][r] += wt * v;
                                }
                        }
                        b[kk][nt] = fabsf(b[kk][nt]) < INFINITY ? b[kk][nt] : 0.f;
                    }
                if constexpr (OWN4) {
                    for (int k = 0; k < 16; ++k) {
                        const float v = ch4[(lane & 3) * ROW + k];
                        if (fabsf(v) < INFINITY) continue;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float wt = wl[(4 * (lane >> 2) + r) * ROW + 4 * (k & 3) + (k >> 2)];
                            if (wt != 0.f) acc4[r] += wt * v;
                        }
                    }
                    __syncthreads();
                    if (!(fabsf(col) < INFINITY)) ch4[(lane & 3) * ROW + (lane >> 2)] = 0.f;
                    __syncthreads();
                }
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                f32x4_t ch;
                if constexpr (OWN4) ch = *reinterpret_cast<const f32x4_t*>(&ch4[(lane & 3) * ROW + 4 * mt]);
                const f32x4_t a =
                    *reinterpret_cast<const f32x4_t*>(&wl[(16 * mt + (lane & 15)) * ROW + 4 * (lane >> 4)]);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma16x16x4(a[kk], b[kk][nt], acc[mt][nt]);
                    if constexpr (OWN4) acc4 = mfma4x4x1(w[4 * mt + kk], ch[kk], acc4);
                }
            }
            __syncthreads();
        }
    }
    T = fabsf(T);
    const size_t hw = (size_t)g.hs * g.ws;
    if (P.inside) {
        const size_t pix = (size_t)P.m * g.ws + P.n;
        final_T[pix] = T;
        n_last[pix] = (int32_t)last;
    }
    // Accumulator (mt, nt) holds pixels 16 mt + 4 (lane / 16) + r, four in a row
    // of the image, of column 16 nt + lane % 16; acc4 pixels 4 (lane / 4) + r of
    // channel lane % 4.
    const int qx = P.n - (lane & 7), qy = P.m - (lane >> 3);  // quadrant origin
    auto put = [&](int c, int p, f32x4_t v) {
        const int m = qy + (p >> 3), n = qx + (p & 7);
        if (m >= g.hs || n >= g.ws) return;
        float* const to = out + c * hw + (size_t)m * g.ws + n;
        if (n + 3 < g.ws) *reinterpret_cast<f4u*>(to) = v;
        else
            for (int r = 0; r < 4 && n + r < g.ws; ++r) to[r] = v[r];
    };
    if constexpr (OWN4) put(lane & 3, lane & ~3, acc4);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int j = 16 * nt + (lane & 15);
        if (j < COLS && (EXACT || j >= CS || j < csem))
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) put(j < CS ? 4 + j : j - CS, 16 * mt + 4 * (lane >> 4), acc[mt][nt]);
    }
}

template <int CS, bool EXACT = true>
static void launch_fwd(const xgs_gaussians* g, const xgs_projected* p, const xgs_binning* b,
                       const TileGrid& tg, float* out, float* final_T, int32_t* n_last,
                       hipStream_t st) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(quad_blocks(tg)), dim3(64), 0, st, b->ranges, b->vals,
                           reinterpret_cast<const float4*>(p->splat), g->colors, g->features, g->c_sem, tg, out,
                           final_T, n_last, (const xgs_batch_slot*)nullptr, 0);
    };
    // the longest row of the arrays addressed is that of the features or colours
    if (g->n * 4 * (int64_t)std::max<int>(g->c_sem, 3) <= (int64_t)UINT32_MAX)
        launch(render_fwd_mfma_kernel<CS, EXACT, uint32_t>);
    else launch(render_fwd_mfma_kernel<CS, EXACT, uint64_t>);
}

template <int CS>
static void launch_fwd_batch(const xgs_batch_slot* slots, int n_slots, const xgs_projected* p,
                             const xgs_binning* b, const TileGrid& tg, hipStream_t st) {
    hipLaunchKernelGGL((render_fwd_mfma_kernel<CS, true, uint64_t, true>), dim3(quad_blocks(tg)), dim3(64), 0, st, b->ranges,
                       b->vals, reinterpret_cast<const float4*>(p->splat), nullptr, nullptr, CS, tg, nullptr,
                       nullptr, nullptr, slots, n_slots);
}

}  // namespace xgs

using namespace xgs;

extern "C" xgs_status xgs_batch_render_fwd(const xgs_batch_slot* d_slots, int32_t n_slots, int32_t c_sem,
                                           int32_t tiles_x, int32_t tile_rows, const xgs_projected* p,
                                           const xgs_binning* b, xgs_stream_t stream) {
    clear_error();
    if (!p || !b) return fail(XGS_ERR_INVALID_ARG, "xgs_batch_render_fwd: null argument");
    if (n_slots < 0 || n_slots > XGS_BATCH_MAX_SLOTS)
        return fail(XGS_ERR_INVALID_ARG, "xgs_batch_render_fwd: n_slots must be in [0, 16]");
    if (n_slots > 0 && !d_slots) return fail(XGS_ERR_INVALID_ARG, "xgs_batch_render_fwd: null slot table");
    if (tiles_x < 1 || tile_rows < 1 || tiles_x > 65535 || tile_rows > 65535 ||
        (int64_t)tiles_x * tile_rows >= (int64_t(1) << 31))
        return fail(XGS_ERR_INVALID_ARG, "xgs_batch_render_fwd: bad tile grid");
    if (!p->splat || !b->ranges || !b->vals) return fail(XGS_ERR_INVALID_ARG, "xgs_batch_render_fwd: null array");
    if (!aligned(p->splat, 16)) return fail(XGS_ERR_INVALID_ARG, "xgs_batch_render_fwd: splat must be 16-byte aligned");
    if (n_slots == 0) return XGS_OK;
    TileGrid tg;
    tg.tx = tiles_x; tg.ty = tile_rows; tg.tiles = tiles_x * tile_rows;
    tg.hs = 16 * tile_rows; tg.ws = 16 * tiles_x; tg.s = 1; tg.oy = 0; tg.ox = 0;
    tg.order = b->tile_order;
    hipStream_t st = (hipStream_t)stream;
    switch (c_sem) {
#define XGS_BFWD_CASE(n) case n: launch_fwd_batch<n>(d_slots, n_slots, p, b, tg, st); break;
        XGS_BFWD_CASE(0) XGS_BFWD_CASE(1) XGS_BFWD_CASE(2) XGS_BFWD_CASE(3) XGS_BFWD_CASE(4)
        XGS_BFWD_CASE(8) XGS_BFWD_CASE(16) XGS_BFWD_CASE(32)
#undef XGS_BFWD_CASE
        default:
            return fail(XGS_ERR_UNSUPPORTED, "xgs_batch_render_fwd: c_sem must be one of 0-4, 8, 16, 32");
    }
    return check_launch("xgs_batch_render_fwd");
}

extern "C" xgs_status xgs_render_fwd(const xgs_gaussians* g, const xgs_projected* p,
                                     const xgs_binning* b, const xgs_camera* cam, float* out,
                                     float* final_T, int32_t* n_last, xgs_stream_t stream) {
    clear_error();
    if (!g || !p || !b || !cam) return fail(XGS_ERR_INVALID_ARG, "xgs_render_fwd: null argument");
    if (xgs_status s = validate_camera(cam)) return s;
    if (!out || !final_T || !n_last) return fail(XGS_ERR_INVALID_ARG, "xgs_render_fwd: null output");
    if (g->c_sem < 0 || g->c_sem > XGS_MAX_C_SEM)
        return fail(XGS_ERR_UNSUPPORTED, "xgs_render_fwd: c_sem must be in [0, 64]");
    if (g->n > 0 && (!g->colors || (g->c_sem > 0 && !g->features) || !p->splat))
        return fail(XGS_ERR_INVALID_ARG, "xgs_render_fwd: null Gaussian array");
    if (!b->ranges || !b->vals) return fail(XGS_ERR_INVALID_ARG, "xgs_render_fwd: null binning array");
    if (!aligned(p->splat, 16)) return fail(XGS_ERR_INVALID_ARG, "xgs_render_fwd: splat must be 16-byte aligned");
    TileGrid tg = tile_grid(*cam, b->tile_order);
    hipStream_t st = (hipStream_t)stream;
    switch (g->c_sem) {
#define XGS_FWD_CASE(n) case n: launch_fwd<n>(g, p, b, tg, out, final_T, n_last, st); break;
        XGS_FWD_CASE(0) XGS_FWD_CASE(1) XGS_FWD_CASE(2) XGS_FWD_CASE(3) XGS_FWD_CASE(4)
        XGS_FWD_CASE(8) XGS_FWD_CASE(12) XGS_FWD_CASE(16) XGS_FWD_CASE(20) XGS_FWD_CASE(24) XGS_FWD_CASE(28)
        XGS_FWD_CASE(32)
        XGS_FWD_CASE(48) XGS_FWD_CASE(64)
#undef XGS_FWD_CASE
        default:
            if (g->c_sem <= 12) launch_fwd<12, false>(g, p, b, tg, out, final_T, n_last, st);
            else if (g->c_sem <= 16) launch_fwd<16, false>(g, p, b, tg, out, final_T, n_last, st);
            else if (g->c_sem <= 28) launch_fwd<28, false>(g, p, b, tg, out, final_T, n_last, st);
            else if (g->c_sem <= 32) launch_fwd<32, false>(g, p, b, tg, out, final_T, n_last, st);
            else launch_fwd<64, false>(g, p, b, tg, out, final_T, n_last, st);
    }
    return check_launch("xgs_render_fwd");
}
