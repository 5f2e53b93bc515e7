// a4: backward of the compositing step and of the EWA projection.
//
// Pixel pass: each wavefront takes an 8x8 quadrant of a tile and walks the
// tile list back to front from the largest n_last of its pixels.  A pixel
// recovers the transmittance in front of Gaussian k as T_k = T_{k+1}/(1-a_k),
// starting from final_T, so nothing per (pixel, Gaussian) is stored by the
// forward pass.  With S_k = sum_{j>k} a_j T_j (g . c_j), the derivative of
// Eq. (rendering) is dL/da_k = T_k (g . c_k) - S_k / (1 - a_k).  The per-pixel
// contributions of a Gaussian are summed over the wavefront by reduce-scatters
// (each exchange halves the number of live values per lane) before one atomic
// add per value.
//
// Gaussian pass: gradients of (mean2d, conic, depth) are carried back through
// conic = Sigma'^-1, Sigma' = J Sigma_cam J^T + 0.3 I, Sigma_cam = Rv Sigma Rv^T,
// Sigma = (R S)(R S)^T, p = Rv mu + t (App. A).
#include <algorithm>

#include "render_common.h"
#include "sort.h"
#include "wave.h"

namespace xgs {

// Workspace row per Gaussian (64 bytes, 10 floats used): with h = a_k dL/da_k
// (0 where alpha is clamped) and (dx, dy) from the splat's mean to the pixel,
// dL/dmean2d, the sums of h dx^2, h dx dy, h dy^2 and h over the pixels (dL/dconic
// and dL/dopacity but for constants and the opacity), then dL/ddepth and
// dL/dcolour.  One row of one half cache line, because the atomics cost by the
// requests that they make, not by their values: with the sums in rows of 32
// bytes, colours and depth added on their own and features 16 at a time (80
// requests for a batch of 16 splats and 32 features) the call took 431 us on 1M
// Gaussians at 1200 x 680; with this row and 32 features at a time, 373; with no
// atomics at all, 350.
enum { GW_MX = 0, GW_MY = 1, GW_XX = 2, GW_XY = 3, GW_YY = 4, GW_1 = 5, GW_DEPTH = 6, GW_COLOR = 7, GW_USED = 10,
       GW_STRIDE = 16 };

// What bounds it: the instructions of one wavefront's walk (about 1,000 vector
// and 84 matrix instructions a batch of 16 splats, 2 wavefronts a SIMD at 32
// features) and, where few lists are long, the longest list's walk.  The whole
// call with 6 sums a pixel reduced two splats at a time and per-value atomics,
// and as it is: 1M Gaussians, 1200 x 680, 32 features 622 -> 375 us; 300k, 640 x
// 480, 16 features 173 -> 94; 123k on a 321 x 240 grid, 20 features 131 -> 78.
// Measured and not taken: the two products interleaved with the walk of the
// batch between them (486 against 440 us at that stage); three wavefronts a SIMD
// instead of two at 16 features, and a higher issue priority for long lists (no
// change).
//
// The walk runs back to front.  The tile list is read 64 entries at a time
// (one per lane: list entry and splat record, the next 64 in flight), the
// splats that can reach alpha >= 1/255 somewhere in the wavefront's quadrant
// are appended to a ring in LDS (quad_hit; the others are skipped by all 64
// pixels) and the walk takes the ring 16 at a time, with the channel rows of
// the next batch in flight.
//
// A pixel takes the splats eight at a time: first the eight alphas, which do
// not depend on each other (0 for a pair that does not contribute, which then
// leaves T and S as they are without further selects; its s and h are selected,
// because an infinite channel or gradient makes S infinite), then the chain of T
// and S.  With b = a / (1 - a): w = b T, h = b (T g.c - S), S += w g.c, T /= 1 - a.
// The sums over the quadrant are formed in two steps.  Over the rows (lane
// bits 3-5): h, h dy and h dy^2 of the eight splats, by a reduce-scatter that
// halves the splats at each exchange, so that lanes 8 s .. 8 s + 7 end with
// the column sums of splat s.  Over the columns: from those and the column's dx
// the six values of the row (h, dL/dmean2d = sum of h (A dx + B dy, B dx + C dy),
// h dx^2, h dx dy, h dy^2), whose reduce-scatter leaves one on each of six lanes.
// The channel gradients dL/dc_k = sum_p w_k(p) g(p) of the batch are one
// product W^T G on v_mfma_f32_16x16x4_f32 (features first, then
// colour and depth), and
// the batch's g.c another; g.c and then w go through one LDS array.
//
// POSE (CS = 0): only the sums that the pose gradient reads.  The semantic
// channels' upstream gradient is taken as zero (they are not read), no channel
// gradient but the depth's is formed, and that one as a fourth sum per splat
// (w g_depth) instead of a product; a splat's seven sums are added from eight
// lanes.  The kernel on 1M Gaussians, 1200 x 680, 32 features:
// 347 us with every gradient, 135 so; with the zeroing and the projection pass
// that a pose needs no more, a tracking step 657 -> 351 us.
template <int CS, bool GEO, bool EXACT, typename OFF, bool POSE = false>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(CS <= 16 ? 3 : 1))) render_bwd_mfma_kernel(
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ vals,
    const float4* __restrict__ splat, const float* __restrict__ colors,
    const float* __restrict__ features, int csem, TileGrid g, const float* __restrict__ d_out,
    const float* __restrict__ final_T, const int32_t* __restrict__ n_last,
    float* __restrict__ d_features, float* __restrict__ geo) {
    constexpr int CH = 4 + CS;
    constexpr int CHP = (CH + 3) / 4 * 4;           // LDS row stride (float4 rows)
    constexpr int COLS = POSE ? 0 : GEO ? CH : CS;  // columns of W^T G: features, then colour and depth
    constexpr int NT = (COLS + 15) / 16;
    static_assert(!GEO || CS % 16 <= 12, "colour and depth are in one tile");
    constexpr int ROW = 20;                         // LDS row of a pixel: 16 splats, float4-aligned, banks spread
    __shared__ __align__(16) float wl[64 * ROW];    // g.c of (pixel, splat), then its weight
    __shared__ Ring ring;
    __shared__ __align__(16) float chl[GEO ? 16 * CHP : 4];
    const QuadPix P = quad_pixel(g);
    if (P.tile >= g.tiles) return;
    const QuadRect qr = quad_rect(g, P);
    const int lane = threadIdx.x;
    // the sum that ends on this lane after the column reduce-scatter (ids: 0 h,
    // 1 mean y, 2 h dy^2, 3 mean x, 4 h dx dy, 5 h dx^2), as its place in the row
    // (POSE: also 6 depth)
    const int id = POSE ? ((lane & 7) == 3 ? 6 : 3 * ((lane >> 2) & 1) + (lane & 3))
                        : 3 * ((lane >> 2) & 1) + ((lane & 1) ? 2 : (lane >> 1) & 1);
    const bool my_own = POSE ? (lane & 7) != 7 : (lane & 3) != 3;
    const int my_word = id == 6 ? GW_DEPTH : id == 0 ? GW_1 : id == 1 ? GW_MY : id == 2 ? GW_YY : id == 3 ? GW_MX : id == 4 ? GW_XY : GW_XX;
    const size_t hw = (size_t)g.hs * g.ws;
    const int fstride = EXACT ? CS : csem;
    const int qx = P.n - (lane & 7), qy = P.m - (lane >> 3);  // quadrant origin
    // upstream gradients in B-operand layout: pixel 4 kk + lane / 16, channel 16 nt + lane % 16
    float bg[NT > 0 ? NT : 1][16];
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
        const int p = 4 * kk + (lane >> 4);
        const int m = qy + (p >> 3), n = qx + (p & 7);
        const bool in = m < g.hs && n < g.ws;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int j = 16 * nt + (lane & 15);
            const int c = j < CS ? 4 + j : j - CS;
            const bool use = in && j < COLS && (EXACT || j >= CS || j < csem);
            bg[nt][kk] = use ? d_out[c * hw + (size_t)m * g.ws + n] : 0.f;
        }
    }
    // Upstream gradients as the B operand of S = C G^T (channel 4 kc + lane / 16,
    // pixel 16 nt + lane % 16): S[k][p] = g(p) . c_k for the batch's 16 splats.
    constexpr int KC = CHP / 4;
    float gt[GEO ? KC : 1][4];
    if constexpr (GEO) {
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int p = 16 * nt + (lane & 15), c = 4 * kc + (lane >> 4);
                const int m = qy + (p >> 3), n = qx + (p & 7);
                const bool use = m < g.hs && n < g.ws && c < CH && (EXACT || c < 4 + csem);
                gt[kc][nt] = use ? d_out[c * hw + (size_t)m * g.ws + n] : 0.f;
            }
    }
    float T = 1.f, gdepth = 0.f;
    int nl = 0;
    if (P.inside) {
        const size_t pix = (size_t)P.m * g.ws + P.n;
        T = final_T[pix];
        nl = n_last[pix];
        if (POSE) gdepth = d_out[3 * hw + pix];
    }
    int jmax = nl;
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) jmax = max(jmax, __shfl_xor(jmax, k, 64));
    const uint32_t start = uniform(ranges[2 * P.tile]);
    const int top = (int)uniform((uint32_t)jmax);

    if (top == 0) return;  // no pixel of the quadrant blended anything

    // Candidate registers: the splat record c0, c1 and index cg of list
    // position cpos - 1 - lane, and the index cn of the position 64 before it
    // (so that a record's load never waits for its list entry).  Positions
    // before the list's start read its first entry and are not pushed.
    auto entry = [&](int pos) { return (int)vals[start + (uint32_t)max(pos - 1 - lane, 0)]; };
    int cpos = top, head = 0, tail = 0;
    bool padded = false;
    int cg = entry(cpos), cn = entry(cpos - 64);
    float4 c0 = splat[2 * (uint32_t)cg], c1 = splat[2 * (uint32_t)cg + 1];
    // keeps at least two batches after `used` in the ring (or everything that is
    // left); the slots written lie past the two batches being read
    auto fill = [&](int used) {
        while (tail - used < 32 && cpos > 0) {
            const int pos = cpos - 1 - lane;
            tail = ring_push(ring, tail, pos >= 0 && quad_hit(c0, c1, qr), c0, c1, cg, pos);
            cpos -= 64;
            cg = cn;
            c0 = splat[2 * (uint32_t)cg];
            c1 = splat[2 * (uint32_t)cg + 1];
            cn = entry(cpos - 64);
        }
        if (cpos <= 0 && !padded) {
            padded = true;
            ring_pad(ring, tail, lane, cg);
        }
    };
    // Channel rows of a batch (only the S = C G^T product reads them): lane
    // 4 k + c takes splat k: colour c or the depth, and where the rows are whole
    // groups of four features, groups c, c + 4, ... of its row.  (Vector loads of
    // 4-byte alignment: a row may start anywhere.)  Other rows are read as 64
    // consecutive (splat, feature) pairs per load.  Slots past the batch hold
    // the index of some splat; nothing of them is used.
    constexpr bool QUADS = EXACT && CS % 4 == 0;
    constexpr int GRP = QUADS ? (CS + 15) / 16 : 0;
    constexpr int PERF = QUADS ? 0 : (16 * CS + 63) / 64;
    constexpr int CSD = CS > 0 ? CS : 1;  // divisor (no feature loads when CS = 0)
    float cv[1 + PERF], cdepth = 0.f;
    f4u cq[GRP > 0 ? GRP : 1];
    auto fetch_channels = [&](int base, int n) {
        if (!GEO || n == 0) return;
        const int k = lane >> 2, c = lane & 3;
        const int at = (base + k) & (kRing - 1);
        const uint32_t i = (uint32_t)ring.gid[at];
        cdepth = ring.rec[at][1].z;
        cv[0] = *at_row<OFF>(colors, i, 3, min(c, 2));
#pragma unroll
        for (int t = 0; t < GRP; ++t)
            if (16 * t + 16 <= CS || 16 * t + 4 * c < CS)
                cq[t] = *reinterpret_cast<const f4u*>(at_row<OFF>(features, i, CS, 16 * t + 4 * c));
#pragma unroll
        for (int t = 1; t <= PERF; ++t) {
            const int e = lane + 64 * (t - 1);
            const int ke = e / CSD, f = e - ke * CSD;
            // past the sixteen splats the ring may hold no index yet
            const uint32_t ie = (uint32_t)ring.gid[(base + min(ke, 15)) & (kRing - 1)];
            cv[t] = *at_row<OFF>(features, ie, fstride, EXACT ? f : min(f, csem - 1));
        }
    };
    auto store_channels = [&]() {
        if constexpr (GEO) {
            float* const row = chl + (lane >> 2) * CHP;
            row[lane & 3] = (lane & 3) < 3 ? cv[0] : cdepth;
#pragma unroll
            for (int t = 0; t < GRP; ++t)
                if (16 * t + 16 <= CS || 16 * t + 4 * (lane & 3) < CS)
                    *reinterpret_cast<f32x4_t*>(row + 4 + 16 * t + 4 * (lane & 3)) = cq[t];
#pragma unroll
            for (int t = 1; t <= PERF; ++t) {
                const int e = lane + 64 * (t - 1);
                const int k = e / CSD, f = e - k * CSD;
                if (64 * t <= 16 * CS || k < 16) chl[k * CHP + 4 + f] = EXACT || f < csem ? cv[t] : 0.f;
            }
        }
    };
    if constexpr (GEO && CHP > CH) {  // padding columns, read as zeros by the product
        for (int i = lane; i < 16 * (CHP - CH); i += 64) chl[(i / (CHP - CH)) * CHP + CH + i % (CHP - CH)] = 0.f;
    }
    // A batch's memory operations are ordered so that nothing waits for an
    // atomic's return: vector memory operations complete in order and the
    // compiler cannot count conditional ones, so a wait for any load after an
    // atomic would drain the atomics too.  Each round issues the loads of the
    // next batch's channels first, waits for them after the walk, refills the
    // ring (whose candidates were loaded a round before), and issues its atomics
    // last: they have the next round's walk to complete.
    fill(head);
    __syncthreads();
    int nb = min(16, tail - head);
    fetch_channels(head, nb);
    store_channels();
    float S = 0.f;
    while (nb > 0) {
        __syncthreads();
        const int nb2 = min(16, tail - head - nb);
        fetch_channels(head + nb, nb2);
        if constexpr (GEO) {
            // S = C G^T on the matrix cores (A: splat lane % 16, channel 4 kc + lane / 16),
            // stored as wl[pixel][splat] for the walk
            f32x4_t sacc[4];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) sacc[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const float a = chl[(lane & 15) * CHP + 4 * kc + (lane >> 4)];
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) sacc[nt] = mfma16x16x4(a, gt[kc][nt], sacc[nt]);
            }
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                *reinterpret_cast<f32x4_t*>(&wl[(16 * nt + (lane & 15)) * ROW + 4 * (lane >> 4)]) = sacc[nt];
        }
        if constexpr (GEO) __syncthreads();
        float gsum[2] = {0.f, 0.f};  // this lane's sum of each eight splats
#pragma unroll
        for (int q = 0; q < 16; q += 8) {
            f32x4_t* const row = reinterpret_cast<f32x4_t*>(&wl[lane * ROW + q]);
            float al[8], dy[8], w[8];
            bool ok[8], any = false;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int at = (head + q + u) & (kRing - 1);
                const float4 s0 = ring.rec[at][0], s1 = ring.rec[at][1];
                const PairEval e = eval_pair(P.px, P.py, s0.x, s0.y, s0.z, s0.w, s1.x, s1.y);
                ok[u] = __float_as_int(s1.w) < nl && e.alpha >= kAlphaMin;
                al[u] = ok[u] ? e.alpha : 0.f;
                dy[u] = e.dy;
                any = any || ok[u];
            }
            if (__ballot(any) == 0ull) {
                row[0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                row[1] = row[0];
                continue;
            }
            constexpr int V = POSE ? 4 : 3;  // sums of a splat over the rows
            float a[8 * V];
            f32x4_t sd[2];
            if constexpr (GEO) {
                sd[0] = row[0];
                sd[1] = row[1];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float rom = __builtin_amdgcn_rcpf(1.f - al[u]);  // 1 - alpha >= 0.01
                const float b = al[u] * rom;
                w[u] = b * T;
                if constexpr (GEO) {
                    const float s = ok[u] ? sd[u >> 2][u & 3] : 0.f;  // a colour may be infinite
                    // 0 < alpha < the clamp, in one comparison of bits: a pair without a part in
                    // the pixel has h = 0 also where S is not finite
                    const bool live = __float_as_uint(al[u]) - 1u < __float_as_uint(kAlphaMax) - 1u;
                    const float h = live ? b * (T * s - S) : 0.f;
                    S += w[u] * s;
                    a[V * u] = h;
                    a[V * u + 1] = h * dy[u];
                    a[V * u + 2] = h * dy[u] * dy[u];
                    if constexpr (POSE) a[V * u + 3] = w[u] * (ok[u] ? gdepth : 0.f);
                }
                T *= rom;
            }
            if constexpr (!POSE) {
                row[0] = f32x4_t{w[0], w[1], w[2], w[3]};
                row[1] = f32x4_t{w[4], w[5], w[6], w[7]};
            }
            if constexpr (GEO) {
                rs_step<8 * V, 32>(a, (lane & 32) == 0);
                rs_step<4 * V, 16>(a, (lane & 16) == 0);
                rs_step<2 * V, 8>(a, (lane & 8) == 0);
                const int k = q + (lane >> 3), at = (head + k) & (kRing - 1);
                const float4 s0 = ring.rec[at][0];
                const float C = ring.rec[at][1].x, dx = P.px - s0.x, hx = a[0] * dx;
                float v[3 + V] = {a[0], s0.w * hx + C * a[1], a[2], s0.z * hx + s0.w * a[1], a[1] * dx, hx * dx};
                if constexpr (POSE) v[6] = a[3];
                rs_step<3 + V, 4>(v, (lane & 4) == 0);
                rs_step<V, 2>(v, (lane & 2) == 0);
                rs_step<2, 1>(v, (lane & 1) == 0);
                gsum[q >> 3] = v[0];
            }
        }
        __syncthreads();
        f32x4_t acc[NT > 0 ? NT : 1];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            if constexpr (NT == 0) break;
            const float a = wl[(4 * kk + (lane >> 4)) * ROW + (lane & 15)];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma16x16x4(a, bg[nt][kk], acc[nt]);
        }
        // every load of this round is complete past this point
        store_channels();
        fill(head + nb);
        if constexpr (POSE) {
#pragma unroll
            for (int q = 0; q < 16; q += 8) {
                const int k = q + (lane >> 3);
                const uint32_t gs = (uint32_t)ring.gid[(head + k) & (kRing - 1)];
                if (my_own && k < nb) unsafeAtomicAdd(at_row<OFF>(geo, gs, GW_STRIDE, my_word), gsum[q >> 3]);
            }
        } else if constexpr (GEO) {
            // the rows of the batch, gathered in LDS (the weights' rows are free):
            // 16 lanes then add a splat's whole row
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 16; q += 8)
                if (my_own) wl[(q + (lane >> 3)) * ROW + my_word] = gsum[q >> 3];
            const int c = (lane & 15) - CS % 16;  // colour or depth column of this lane
            if (c >= 0 && c < 4)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    wl[(4 * (lane >> 4) + r) * ROW + (c < 3 ? GW_COLOR + c : (int)GW_DEPTH)] = acc[CS / 16][r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int slot = 4 * r + (lane >> 4);
                const uint32_t gs = (uint32_t)ring.gid[(head + slot) & (kRing - 1)];
                const float v = wl[slot * ROW + (lane & 15)];
                if (slot < nb && (lane & 15) < GW_USED) unsafeAtomicAdd(at_row<OFF>(geo, gs, GW_STRIDE, lane & 15), v);
            }
        }
        // acc[nt][r]: Gaussian slot 4 (lane / 16) + r, column 16 nt + lane % 16.
        // Two whole tiles of features: rows of 16 lanes are swapped so that 32
        // lanes hold 32 consecutive features of one slot.
        constexpr int PAIRS = EXACT ? CS / 32 : 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int pr = 0; pr < PAIRS; ++pr) {
                const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[2 * pr][r]),
                                                               __float_as_uint(acc[2 * pr + 1][r]), false, false);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int slot = 4 * (2 * (lane >> 5) + h) + r;
                    const uint32_t gs = (uint32_t)ring.gid[(head + slot) & (kRing - 1)];
                    if (slot < nb)
                        unsafeAtomicAdd(at_row<OFF>(d_features, gs, fstride, 32 * pr + (lane & 31)),
                                        __uint_as_float(x[h]));
                }
            }
            const int slot = 4 * (lane >> 4) + r;
            const uint32_t gs = (uint32_t)ring.gid[(head + slot) & (kRing - 1)];
#pragma unroll
            for (int nt = 2 * PAIRS; nt < (CS + 15) / 16; ++nt) {
                const int j = 16 * nt + (lane & 15);
                if (slot < nb && (16 * nt + 16 <= CS || j < CS) && (EXACT || j < csem))
                    unsafeAtomicAdd(at_row<OFF>(d_features, gs, fstride, j), acc[nt][r]);
            }
        }
        __syncthreads();
        head += nb;
        nb = nb2;
    }
}

struct CamDevB {
    float fx, fy, limx, limy, near_;
    float R[9], t[3];
};

// Adjoint of one Gaussian's projection down to the camera frame (App. A):
// recomputes p = Rv mu + t, R(q), the scales, M = R S, Sigma_cam = (Rv M)
// (Rv M)^T and J at the guarded p, then carries dL/dmean2d, dL/dconic and
// dL/ddepth (the workspace row) to dL/dp and dL/dSigma_cam.
struct CamAdj {
    float p[3];
    float R[3][3], s[3], M[3][3], Sc[3][3];
    float dSc[3][3], dp[3];
    float q[4], inv;
};

__device__ __forceinline__ void cam_adjoint(int64_t i, const float* __restrict__ means,
                                            const float* __restrict__ log_scales,
                                            const float4* __restrict__ quats, const float4* __restrict__ splat,
                                            const float* __restrict__ gw, const CamDevB& c, CamAdj& a) {
    const float4 s0 = splat[2 * i], s1 = splat[2 * i + 1];
    const float K00 = s0.z, K01 = s0.w, K11 = s1.x;
    // dL/dconic: q = A dx^2 + 2 B dx dy + C dy^2 and dL/dq = -h / 2
    const float gmx = gw[GW_MX], gmy = gw[GW_MY];
    const float gA = -0.5f * gw[GW_XX], gB = -gw[GW_XY], gC = -0.5f * gw[GW_YY], gd = gw[GW_DEPTH];
    const float mx = means[3 * i], my = means[3 * i + 1], mz = means[3 * i + 2];
    const float px = c.R[0] * mx + c.R[1] * my + c.R[2] * mz + c.t[0];
    const float py = c.R[3] * mx + c.R[4] * my + c.R[5] * mz + c.t[1];
    const float pz = c.R[6] * mx + c.R[7] * my + c.R[8] * mz + c.t[2];
    a.p[0] = px; a.p[1] = py; a.p[2] = pz;
    float4 q = quats[i];
    const float qn = sqrtf(q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w);
    a.inv = 1.f / qn;
    const float w = q.x * a.inv, x = q.y * a.inv, y = q.z * a.inv, z = q.w * a.inv;
    a.q[0] = w; a.q[1] = x; a.q[2] = y; a.q[3] = z;
    const float R[3][3] = {{1.f - 2.f * (y * y + z * z), 2.f * (x * y - w * z), 2.f * (x * z + w * y)},
                           {2.f * (x * y + w * z), 1.f - 2.f * (x * x + z * z), 2.f * (y * z - w * x)},
                           {2.f * (x * z - w * y), 2.f * (y * z + w * x), 1.f - 2.f * (x * x + y * y)}};
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) a.R[r][k] = R[r][k];
    a.s[0] = __expf(log_scales[3 * i]); a.s[1] = __expf(log_scales[3 * i + 1]); a.s[2] = __expf(log_scales[3 * i + 2]);
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) a.M[r][k] = R[r][k] * a.s[k];
    // Sigma_cam = (Rv M)(Rv M)^T
    float TM[3][3];
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k)
            TM[r][k] = c.R[3 * r] * a.M[0][k] + c.R[3 * r + 1] * a.M[1][k] + c.R[3 * r + 2] * a.M[2][k];
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) a.Sc[r][k] = TM[r][0] * TM[k][0] + TM[r][1] * TM[k][1] + TM[r][2] * TM[k][2];
    const float iz = 1.f / pz;
    const float u = px * iz, v = py * iz;
    const bool clx = u < -c.limx || u > c.limx, cly = v < -c.limy || v > c.limy;
    const float tx = fminf(fmaxf(u, -c.limx), c.limx) * pz;
    const float ty = fminf(fmaxf(v, -c.limy), c.limy) * pz;
    const float J[2][3] = {{c.fx * iz, 0.f, -c.fx * tx * iz * iz}, {0.f, c.fy * iz, -c.fy * ty * iz * iz}};
    // conic K = (A, B, C) from the splat record; dSigma' = -K Ghat K
    const float G00 = gA, G01 = 0.5f * gB, G11 = gC;
    const float KG00 = K00 * G00 + K01 * G01, KG01 = K00 * G01 + K01 * G11;
    const float KG10 = K01 * G00 + K11 * G01, KG11 = K01 * G01 + K11 * G11;
    const float dS00 = -(KG00 * K00 + KG01 * K01);
    const float dS01 = -(KG00 * K01 + KG01 * K11);
    const float dS11 = -(KG10 * K01 + KG11 * K11);
    const float dS[2][2] = {{dS00, dS01}, {dS01, dS11}};
    // dSc = J^T dS J ; dJ = 2 dS J Sc
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) {
            float acc = 0.f;
            for (int aa = 0; aa < 2; ++aa)
                for (int bb = 0; bb < 2; ++bb) acc += J[aa][r] * dS[aa][bb] * J[bb][k];
            a.dSc[r][k] = acc;
        }
    float JSc[2][3];
    for (int r = 0; r < 2; ++r)
        for (int k = 0; k < 3; ++k) JSc[r][k] = J[r][0] * a.Sc[0][k] + J[r][1] * a.Sc[1][k] + J[r][2] * a.Sc[2][k];
    float dJ[2][3];
    for (int r = 0; r < 2; ++r)
        for (int k = 0; k < 3; ++k) dJ[r][k] = 2.f * (dS[r][0] * JSc[0][k] + dS[r][1] * JSc[1][k]);
    // J(p), mean2d(p), depth(p) -> p
    const float iz2 = iz * iz, iz3 = iz2 * iz;
    const float dtx_dpx = clx ? 0.f : 1.f, dtx_dpz = clx ? tx * iz : 0.f;
    const float dty_dpy = cly ? 0.f : 1.f, dty_dpz = cly ? ty * iz : 0.f;
    a.dp[0] = dJ[0][2] * (-c.fx * iz2) * dtx_dpx + gmx * c.fx * iz;
    a.dp[1] = dJ[1][2] * (-c.fy * iz2) * dty_dpy + gmy * c.fy * iz;
    a.dp[2] = dJ[0][0] * (-c.fx * iz2) + dJ[1][1] * (-c.fy * iz2) +
              dJ[0][2] * (-c.fx * iz2 * dtx_dpz + 2.f * c.fx * tx * iz3) +
              dJ[1][2] * (-c.fy * iz2 * dty_dpz + 2.f * c.fy * ty * iz3) - gmx * c.fx * px * iz2 -
              gmy * c.fy * py * iz2 + gd;
}

// Per-Gaussian chain rule from (mean2d, conic, depth) to (mean, log-scale,
// quaternion), and the opacity's gradient; the forward quantities are
// recomputed from the parameters.
__global__ void __launch_bounds__(256) project_bwd_kernel(
    int64_t n, const float* __restrict__ means, const float* __restrict__ log_scales,
    const float4* __restrict__ quats, const int32_t* __restrict__ radius,
    const float4* __restrict__ splat, const float* __restrict__ geo, CamDevB c,
    float* __restrict__ d_means, float* __restrict__ d_ls, float4* __restrict__ d_quats,
    float* __restrict__ d_opacity, float* __restrict__ d_colors) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float gm[3] = {0.f, 0.f, 0.f}, gl[3] = {0.f, 0.f, 0.f}, gc[3] = {0.f, 0.f, 0.f}, go = 0.f;
    float4 gq = make_float4(0.f, 0.f, 0.f, 0.f);
    if (radius[i] > 0) {
        CamAdj a;
        cam_adjoint(i, means, log_scales, quats, splat, geo + (size_t)i * GW_STRIDE, c, a);
        go = geo[(size_t)i * GW_STRIDE + GW_1] / splat[2 * i + 1].y;  // da/do = a / o where not clamped
        for (int k = 0; k < 3; ++k) gc[k] = geo[(size_t)i * GW_STRIDE + GW_COLOR + k];
        // dSigma = Rv^T dSc Rv
        float tmp[3][3], dSig[3][3];
        for (int r = 0; r < 3; ++r)
            for (int k = 0; k < 3; ++k)
                tmp[r][k] = c.R[r] * a.dSc[0][k] + c.R[3 + r] * a.dSc[1][k] + c.R[6 + r] * a.dSc[2][k];
        for (int r = 0; r < 3; ++r)
            for (int k = 0; k < 3; ++k)
                dSig[r][k] = tmp[r][0] * c.R[k] + tmp[r][1] * c.R[3 + k] + tmp[r][2] * c.R[6 + k];
        // dM = 2 dSig M ; dR = dM diag(s) ; ds = diag(R^T dM)
        float dR[3][3];
        for (int k = 0; k < 3; ++k) {
            float ds = 0.f;
            for (int r = 0; r < 3; ++r) {
                const float dM = 2.f * (dSig[r][0] * a.M[0][k] + dSig[r][1] * a.M[1][k] + dSig[r][2] * a.M[2][k]);
                ds += dM * a.R[r][k];
                dR[r][k] = dM * a.s[k];
            }
            gl[k] = ds * a.s[k];
        }
        const float w = a.q[0], x = a.q[1], y = a.q[2], z = a.q[3];
        float g0 = 2.f * (-z * dR[0][1] + y * dR[0][2] + z * dR[1][0] - x * dR[1][2] - y * dR[2][0] + x * dR[2][1]);
        float g1 = 2.f * (y * dR[0][1] + z * dR[0][2] + y * dR[1][0] - 2.f * x * dR[1][1] - w * dR[1][2] +
                          z * dR[2][0] + w * dR[2][1] - 2.f * x * dR[2][2]);
        float g2 = 2.f * (-2.f * y * dR[0][0] + x * dR[0][1] + w * dR[0][2] + x * dR[1][0] + z * dR[1][2] -
                          w * dR[2][0] + z * dR[2][1] - 2.f * y * dR[2][2]);
        float g3 = 2.f * (-2.f * z * dR[0][0] - w * dR[0][1] + x * dR[0][2] + w * dR[1][0] - 2.f * z * dR[1][1] +
                          y * dR[1][2] + x * dR[2][0] + y * dR[2][1]);
        const float dot = w * g0 + x * g1 + y * g2 + z * g3;
        gq = make_float4((g0 - w * dot) * a.inv, (g1 - x * dot) * a.inv, (g2 - y * dot) * a.inv,
                         (g3 - z * dot) * a.inv);
        // p -> mu
        for (int k = 0; k < 3; ++k) gm[k] = c.R[k] * a.dp[0] + c.R[3 + k] * a.dp[1] + c.R[6 + k] * a.dp[2];
    }
    d_means[3 * i] = gm[0]; d_means[3 * i + 1] = gm[1]; d_means[3 * i + 2] = gm[2];
    d_ls[3 * i] = gl[0]; d_ls[3 * i + 1] = gl[1]; d_ls[3 * i + 2] = gl[2];
    d_quats[i] = gq;
    d_opacity[i] = go;
    d_colors[3 * i] = gc[0]; d_colors[3 * i + 1] = gc[1]; d_colors[3 * i + 2] = gc[2];
}

// Camera-pose gradient (Eq. (tracking): extrinsics optimised with the map
// frozen) for the left perturbation T(xi) = exp(xi^) T, xi = (rho, phi):
// p -> p + rho + phi x p and Sigma_cam -> Sigma_cam + phi^ Sigma_cam -
// Sigma_cam phi^, so per Gaussian dL/drho = dL/dp and
// dL/dphi = p x dL/dp + axial(Sc G - G Sc), G = dL/dSigma_cam,
// axial(A) = (A_23 - A_32, A_31 - A_13, A_12 - A_21).  Each workgroup sums
// 256 Gaussians in a fixed tree order into partial[block][6].
__global__ void __launch_bounds__(256) pose_grad_kernel(
    int64_t n, const float* __restrict__ means, const float* __restrict__ log_scales,
    const float4* __restrict__ quats, const int32_t* __restrict__ radius, const float4* __restrict__ splat,
    const float* __restrict__ geo, CamDevB c, float* __restrict__ partial) {
    __shared__ float red[4][6];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (i < n && radius[i] > 0) {
        CamAdj a;
        cam_adjoint(i, means, log_scales, quats, splat, geo + (size_t)i * GW_STRIDE, c, a);
        float A[3][3];
        for (int r = 0; r < 3; ++r)
            for (int k = 0; k < 3; ++k) {
                float acc = 0.f;
                for (int m = 0; m < 3; ++m) acc += a.Sc[r][m] * a.dSc[m][k] - a.dSc[r][m] * a.Sc[m][k];
                A[r][k] = acc;
            }
        const float* p = a.p;
        const float* dp = a.dp;
        v[0] = dp[0]; v[1] = dp[1]; v[2] = dp[2];
        v[3] = p[1] * dp[2] - p[2] * dp[1] + (A[1][2] - A[2][1]);
        v[4] = p[2] * dp[0] - p[0] * dp[2] + (A[2][0] - A[0][2]);
        v[5] = p[0] * dp[1] - p[1] * dp[0] + (A[0][1] - A[1][0]);
    }
#pragma unroll
    for (int k = 0; k < 6; ++k)
        for (int o = 32; o >= 1; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k) red[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 6)
        partial[(size_t)blockIdx.x * 6 + threadIdx.x] =
            (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// Thread j sums the partials of blocks j, j + 256, ... in order, then a
// fixed tree combines the 256 sums: deterministic.
__global__ void __launch_bounds__(256) pose_total_kernel(const float* __restrict__ partial, int64_t nb,
                                                        float* __restrict__ d_pose) {
    __shared__ float red[6][256];
    const int t = threadIdx.x;
    float s[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int64_t b = t; b < nb; b += 256)
#pragma unroll
        for (int k = 0; k < 6; ++k) s[k] += partial[(size_t)b * 6 + k];
#pragma unroll
    for (int k = 0; k < 6; ++k) red[k][t] = s[k];
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (t < o)
#pragma unroll
            for (int k = 0; k < 6; ++k) red[k][t] += red[k][t + o];
        __syncthreads();
    }
    if (t < 6) d_pose[t] = red[t][0];
}

template <int CS, bool GEO, bool EXACT = true, bool POSE = false>
static void launch_bwd(const xgs_gaussians* g, const xgs_projected* p, const xgs_binning* b,
                       const TileGrid& tg, const float* d_out, const float* final_T,
                       const int32_t* n_last, xgs_gaussians_grad* gr, float* geo, hipStream_t st) {
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(quad_blocks(tg)), dim3(64), 0, st, b->ranges, b->vals,
                           reinterpret_cast<const float4*>(p->splat), g->colors, g->features, g->c_sem, tg, d_out,
                           final_T, n_last, gr->features, geo);
    };
    // the longest row of the arrays addressed is that of the features or of
    // the workspace
    const int64_t row = 4 * (int64_t)std::max<int>(g->c_sem, GW_STRIDE);
    if (g->n * row <= (int64_t)UINT32_MAX) launch(render_bwd_mfma_kernel<CS, GEO, EXACT, uint32_t, POSE>);
    else launch(render_bwd_mfma_kernel<CS, GEO, EXACT, uint64_t, POSE>);
}

template <bool GEO>
static void dispatch_bwd(const xgs_gaussians* g, const xgs_projected* p, const xgs_binning* b,
                         const TileGrid& tg, const float* d_out, const float* final_T,
                         const int32_t* n_last, xgs_gaussians_grad* gr, float* geo, hipStream_t st) {
    const int cs = g->c_sem;
    if (!GEO && cs == 0) return;
    switch (cs) {
#define XGS_BWD_CASE(n) case n: launch_bwd<n, GEO>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st); return;
        XGS_BWD_CASE(1) XGS_BWD_CASE(2) XGS_BWD_CASE(3) XGS_BWD_CASE(4) XGS_BWD_CASE(8)
        XGS_BWD_CASE(12) XGS_BWD_CASE(16) XGS_BWD_CASE(20) XGS_BWD_CASE(24) XGS_BWD_CASE(28) XGS_BWD_CASE(32)
        XGS_BWD_CASE(48)
#undef XGS_BWD_CASE
        default: break;
    }
    if constexpr (GEO) {
        if (cs == 0) launch_bwd<0, true>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 12) launch_bwd<12, true, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 16) launch_bwd<16, true, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 24) launch_bwd<24, true, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 28) launch_bwd<28, true, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 32) launch_bwd<32, true, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else launch_bwd<54, true, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
    } else {
        if (cs == 64) launch_bwd<64, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 16) launch_bwd<16, false, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else if (cs <= 32) launch_bwd<32, false, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        else launch_bwd<64, false, false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
    }
}

static CamDevB cam_dev_b(const xgs_camera& cam) {
    CamDevB c;
    c.fx = cam.fx; c.fy = cam.fy; c.near_ = cam.near_plane;
    c.limx = kGuard * (0.5f * cam.width) / cam.fx;
    c.limy = kGuard * (0.5f * cam.height) / cam.fy;
    for (int r = 0; r < 3; ++r) {
        for (int k = 0; k < 3; ++k) c.R[3 * r + k] = cam.viewmat[4 * r + k];
        c.t[r] = cam.viewmat[4 * r + 3];
    }
    return c;
}

}  // namespace xgs

using namespace xgs;

static size_t pose_blocks(int64_t n) { return (size_t)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

extern "C" size_t xgs_render_bwd_workspace(int64_t n) {
    Carve c(nullptr);
    c.take<float>((size_t)(n > 0 ? n : 1) * GW_STRIDE);
    c.take<float>(pose_blocks(n) * 6);
    return c.total();
}

// The accumulated gradients (features; with the geometry the workspace rows,
// from which the projection pass writes the others) start at zero: one launch.
// radius (may be NULL): only the workspace rows of the Gaussians in view, the
// only ones that are read again (of 1M Gaussians of a room about one in eight:
// 9 MB instead of 64).
static xgs_status zero_accumulated(const xgs_gaussians* g, bool features, bool geo_on, xgs_gaussians_grad* gr,
                                   float* geo, const int32_t* radius, hipStream_t st) {
    ZeroRanges zr{};
    if (features && g->c_sem > 0) { zr.p[zr.k] = reinterpret_cast<uint32_t*>(gr->features); zr.n[zr.k++] = g->n * g->c_sem; }
    if (geo_on) {
        static_assert(GW_STRIDE == ZeroRanges::kRow, "workspace rows");
        zr.seen = radius;
        zr.seen_k = zr.k;
        zr.p[zr.k] = reinterpret_cast<uint32_t*>(geo); zr.n[zr.k++] = GW_STRIDE * g->n;
    }
    return zero_ranges(zr, st);
}

extern "C" xgs_status xgs_render_bwd_zero(const xgs_gaussians* g, int32_t flags, xgs_gaussians_grad* gr, void* ws,
                                          size_t ws_bytes, xgs_stream_t stream) {
    clear_error();
    if (!g || !gr) return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd_zero: null argument");
    if ((flags & ~XGS_BWD_PREZEROED) != XGS_BWD_ALL && (flags & ~XGS_BWD_PREZEROED) != XGS_BWD_FEATURES_ONLY)
        return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd_zero: unknown flags");
    const bool geo_on = (flags & ~XGS_BWD_PREZEROED) == XGS_BWD_ALL;
    if (g->n < 0 || g->c_sem < 0 || g->c_sem > XGS_MAX_C_SEM || gr->n != g->n || gr->c_sem != g->c_sem)
        return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd_zero: gradient shapes differ from the Gaussians");
    if (!aligned(ws, 256)) return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd_zero: workspace must be 256-byte aligned");
    if (!ws || ws_bytes < xgs_render_bwd_workspace(g->n))
        return fail(XGS_ERR_CAPACITY, "xgs_render_bwd_zero: workspace too small");
    if (g->n == 0) return XGS_OK;
    if ((g->c_sem > 0 && !gr->features) || (geo_on && (!gr->colors || !gr->opacity)))
        return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd_zero: null gradient array");
    xgs_status s = zero_accumulated(g, true, geo_on, gr, static_cast<float*>(ws), nullptr, (hipStream_t)stream);
    if (s) return s;
    return check_launch("xgs_render_bwd_zero");
}

extern "C" xgs_status xgs_render_bwd(const xgs_gaussians* g, const xgs_projected* p,
                                     const xgs_binning* b, const xgs_camera* cam, const float* d_out,
                                     const float* final_T, const int32_t* n_last, int32_t flags,
                                     xgs_gaussians_grad* gr, void* ws, size_t ws_bytes,
                                     xgs_stream_t stream) {
    clear_error();
    if (!g || !p || !b || !cam || !gr) return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: null argument");
    if (xgs_status s = validate_camera(cam)) return s;
    const bool prezeroed = (flags & XGS_BWD_PREZEROED) != 0;
    flags &= ~XGS_BWD_PREZEROED;
    if (flags != XGS_BWD_ALL && flags != XGS_BWD_FEATURES_ONLY && (flags != XGS_BWD_POSE || prezeroed))
        return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: unknown flags");
    const bool pose = flags == XGS_BWD_POSE, geo_on = flags != XGS_BWD_FEATURES_ONLY;
    if (g->c_sem < 0 || g->c_sem > XGS_MAX_C_SEM)
        return fail(XGS_ERR_UNSUPPORTED, "xgs_render_bwd: c_sem must be in [0, 64]");
    if (geo_on && g->c_sem > 54)
        return fail(XGS_ERR_UNSUPPORTED, "xgs_render_bwd: c_sem <= 54 (4 + c_sem + 6 sums per lane)");
    if (gr->n != g->n || gr->c_sem != g->c_sem)
        return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: gradient shapes differ from the Gaussians");
    if (!d_out || !final_T || !n_last) return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: null image buffer");
    if (g->n > 0) {
        if (!g->colors || (g->c_sem > 0 && !g->features) || !p->splat || !p->radius)
            return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: null Gaussian array");
        if (!pose && g->c_sem > 0 && !gr->features)
            return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: null feature gradient");
        if (geo_on && !pose && (!gr->means || !gr->log_scales || !gr->quats || !gr->opacity || !gr->colors ||
                       !g->means || !g->log_scales || !g->quats))
            return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: null gradient array");
        if (geo_on && !pose && !aligned(gr->quats, 16))
            return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: quats gradient must be 16-byte aligned");
    }
    if (!aligned(ws, 256)) return fail(XGS_ERR_INVALID_ARG, "xgs_render_bwd: workspace must be 256-byte aligned");
    if (!ws || ws_bytes < xgs_render_bwd_workspace(g->n))
        return fail(XGS_ERR_CAPACITY, "xgs_render_bwd: workspace too small");
    if (g->n == 0) return XGS_OK;
    hipStream_t st = (hipStream_t)stream;
    float* geo = static_cast<float*>(ws);
    xgs_status s;
    // the accumulated gradients and the workspace rows start at zero, unless the
    // caller had xgs_render_bwd_zero do it beforehand
    if (!prezeroed && (s = zero_accumulated(g, !pose, geo_on, gr, geo, p->radius, st))) return s;
    TileGrid tg = tile_grid(*cam, b->tile_order);
    if (pose) {
        launch_bwd<0, true, true, true>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        return check_launch("xgs_render_bwd pose");
    }
    if (geo_on) {
        dispatch_bwd<true>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
        if ((s = check_launch("xgs_render_bwd pixels"))) return s;
        const CamDevB c = cam_dev_b(*cam);
        hipLaunchKernelGGL(project_bwd_kernel, dim3((unsigned)((g->n + 255) / 256)), dim3(256), 0, st, g->n,
                           g->means, g->log_scales, reinterpret_cast<const float4*>(g->quats), p->radius,
                           reinterpret_cast<const float4*>(p->splat), geo, c, gr->means, gr->log_scales,
                           reinterpret_cast<float4*>(gr->quats), gr->opacity, gr->colors);
        return check_launch("xgs_render_bwd projection");
    }
    dispatch_bwd<false>(g, p, b, tg, d_out, final_T, n_last, gr, geo, st);
    return check_launch("xgs_render_bwd features");
}

extern "C" xgs_status xgs_pose_grad(const xgs_gaussians* g, const xgs_projected* p, const xgs_camera* cam,
                                    const void* ws, size_t ws_bytes, float* d_pose, xgs_stream_t stream) {
    clear_error();
    if (!g || !p || !cam || !d_pose) return fail(XGS_ERR_INVALID_ARG, "xgs_pose_grad: null argument");
    if (xgs_status s = validate_camera(cam)) return s;
    if (!aligned(ws, 256)) return fail(XGS_ERR_INVALID_ARG, "xgs_pose_grad: workspace must be 256-byte aligned");
    if (!ws || ws_bytes < xgs_render_bwd_workspace(g->n))
        return fail(XGS_ERR_CAPACITY, "xgs_pose_grad: workspace too small");
    if (g->n > 0 && (!g->means || !g->log_scales || !g->quats || !p->splat || !p->radius))
        return fail(XGS_ERR_INVALID_ARG, "xgs_pose_grad: null Gaussian array");
    Carve cv(const_cast<void*>(ws));
    const float* geo = cv.take<float>((size_t)(g->n > 0 ? g->n : 1) * GW_STRIDE);
    float* partial = cv.take<float>(pose_blocks(g->n) * 6);
    hipStream_t st = (hipStream_t)stream;
    if (g->n == 0) return fill_f32(d_pose, 6, 0.f, st);
    const size_t nb = pose_blocks(g->n);
    hipLaunchKernelGGL(pose_grad_kernel, dim3((unsigned)nb), dim3(256), 0, st, g->n, g->means, g->log_scales,
                       reinterpret_cast<const float4*>(g->quats), p->radius,
                       reinterpret_cast<const float4*>(p->splat), geo, cam_dev_b(*cam), partial);
    hipLaunchKernelGGL(pose_total_kernel, dim3(1), dim3(256), 0, st, partial, (int64_t)nb, d_pose);
    return check_launch("xgs_pose_grad");
}
