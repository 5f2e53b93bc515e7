// Semantic phase: mixture weights, per-pixel decode and the masked grid loss.
//
// Sec. 3.2.2 (online VQ module): every Gaussian carries logits z_i over the L
// codewords of the shared codebook E [L][D]; its mixture weights are
// w_i = softmax(z_i) and its decoded feature is E^T w_i.  The weights are
// rendered as the semantic channels (a3), and App. E decodes per pixel,
// G^(x) = E^T w(x).  App. D (masked loss evaluation) compares G^ with the grid
// targets G* under the validity mask V:
//   L = lambda [ (1/n) sum_{x valid} (1 - cos(G^(x), G*(x)))
//              + (1/(n D)) sum_{x valid} |G^(x) - G*(x)|_1 ],
// n = number of valid pixels, cos(a, b) = <a, b> / max(|a||b|, 1e-8).
// The geometry is frozen in this phase (Sec. 3.2.2, parallelized pipeline),
// so the backward is the feature-only pass of a4 followed by the softmax.
#include <algorithm>
#include <cstdint>

#include "common.h"
#include "wave.h"

namespace xgs {

constexpr float kCosEps = 1e-8f;
constexpr int SEM_NPT = 2;              // 16-pixel tiles per wavefront (decode + loss)
constexpr int SEM_PIX = 64 * SEM_NPT;   // grid pixels per workgroup (decode + loss)

// ------------------------------------------------------------------ softmax
template <int L>
__global__ void __launch_bounds__(256) sem_softmax_kernel(const float* __restrict__ z, int64_t N,
                                                         float* __restrict__ w) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    float v[L];
    const float4* zr = reinterpret_cast<const float4*>(z + i * L);
#pragma unroll
    for (int k = 0; k < L / 4; ++k) {
        const float4 q = zr[k];
        v[4 * k] = q.x; v[4 * k + 1] = q.y; v[4 * k + 2] = q.z; v[4 * k + 3] = q.w;
    }
    float m = v[0];
#pragma unroll
    for (int k = 1; k < L; ++k) m = fmaxf(m, v[k]);
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < L; ++k) {
        v[k] = expf(v[k] - m);
        s += v[k];
    }
    const float inv = 1.f / s;
    float4* wr = reinterpret_cast<float4*>(w + i * L);
#pragma unroll
    for (int k = 0; k < L / 4; ++k)
        wr[k] = make_float4(v[4 * k] * inv, v[4 * k + 1] * inv, v[4 * k + 2] * inv, v[4 * k + 3] * inv);
}

// dL/dz = w (dL/dw - <dL/dw, w>)
template <int L>
__global__ void __launch_bounds__(256) sem_softmax_bwd_kernel(const float* __restrict__ w,
                                                             const float* __restrict__ dw, int64_t N,
                                                             float* __restrict__ dz) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    float wv[L], gv[L];
    const float4* wr = reinterpret_cast<const float4*>(w + i * L);
    const float4* gr = reinterpret_cast<const float4*>(dw + i * L);
#pragma unroll
    for (int k = 0; k < L / 4; ++k) {
        const float4 a = wr[k], b = gr[k];
        wv[4 * k] = a.x; wv[4 * k + 1] = a.y; wv[4 * k + 2] = a.z; wv[4 * k + 3] = a.w;
        gv[4 * k] = b.x; gv[4 * k + 1] = b.y; gv[4 * k + 2] = b.z; gv[4 * k + 3] = b.w;
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < L; ++k) s += gv[k] * wv[k];
    float4* out = reinterpret_cast<float4*>(dz + i * L);
#pragma unroll
    for (int k = 0; k < L / 4; ++k)
        out[k] = make_float4(wv[4 * k] * (gv[4 * k] - s), wv[4 * k + 1] * (gv[4 * k + 1] - s),
                             wv[4 * k + 2] * (gv[4 * k + 2] - s), wv[4 * k + 3] * (gv[4 * k + 3] - s));
}

// ------------------------------------------------------------- valid count
// Valid pixels, one sum per block (kCountBlocks of them; the loss kernels add
// them up, one per lane).  One atomic per wavefront on one counter took 43 us at
// 640 x 480, this 4.7.
constexpr int kCountBlocks = 64;

__global__ void __launch_bounds__(1024) sem_count_kernel(const uint8_t* __restrict__ V, int64_t P,
                                                        int* __restrict__ counts) {
    __shared__ int red[16];
    const int64_t t = (int64_t)blockIdx.x * 1024 + threadIdx.x, stride = (int64_t)gridDim.x * 1024;
    // bytes before 16-byte alignment, 16-byte words, the bytes after them
    const int64_t head = min(P, (int64_t)((16 - ((uintptr_t)V & 15)) & 15)), body = (P - head) / 16;
    int c = 0;
    auto nonzero = [](uint32_t w) {
        return (int)((w & 0xFFu) != 0) + (int)((w & 0xFF00u) != 0) + (int)((w & 0xFF0000u) != 0) + (int)(w > 0xFFFFFFu);
    };
    for (int64_t q = t; q < body; q += stride) {
        const uint4 v = reinterpret_cast<const uint4*>(V + head)[q];
        c += nonzero(v.x) + nonzero(v.y) + nonzero(v.z) + nonzero(v.w);
    }
    if (t < head) c += V[t] != 0;
    const int64_t tail0 = head + 16 * body;
    if (t < P - tail0) c += V[tail0 + t] != 0;
    for (int k = 32; k >= 1; k >>= 1) c += __shfl_xor(c, k, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int s = 0;
        for (int k = 0; k < 16; ++k) s += red[k];
        counts[blockIdx.x] = s;
    }
}

// The number of valid pixels, in every lane: the sum of the blocks' counts, or
// all P (at most INT_MAX) without a mask.
__device__ __forceinline__ int valid_total(const uint8_t* V, const int* __restrict__ counts, int64_t P) {
    if (!V) return (int)min(P, (int64_t)0x7FFFFFFF);
    int n = counts[threadIdx.x & 63];
    static_assert(kCountBlocks == 64, "one count per lane");
    const int lane = threadIdx.x & 63;
    n += xlane_partner<32>(n, lane);
    n += xlane_partner<16>(n, lane);
    n += xlane_partner<8>(n, lane);
    n += xlane_partner<4>(n, lane);
    n += xlane_partner<2>(n, lane);
    n += xlane_partner<1>(n, lane);
    return n;
}

// ----------------------------------------------------------- decode + loss
// One workgroup: 64 SEM_NPT consecutive grid pixels, wavefront q taking
// SEM_NPT tiles of 16 pixels and every codeword column (two tiles per wave:
// each G* plane is then read in 128-byte runs; measured 0.39 -> 0.35 ms at
// 640 x 480, D = 512, against one tile, and four tiles was slower).  The decode F = W E (W the
// pixels' mixture weights, E the L x D codebook) and the gradient product
// dL/dW = g E^T both run on v_mfma_f32_16x16x4_f32 (FP32 products, FP32
// sums), in transposed form so that no operand changes lanes:
//   F^T tile (16 columns d x 16 pixels p) = sum over codes of E^T W^T, with
//     A[d][code] = E[code][d] (from L2) and B[code][p] = W[p][code] (held in
//     registers for the whole kernel); the accumulator puts column
//     d = 16 mt + 4 (lane / 16) + r and pixel p = lane % 16 in lane `lane`,
//     element r;
//   dL/dW^T (16 codes x 16 pixels) += sum over d of E g^T, contracting over
//     d = 16 mt + 4 k + r in step (mt, r), k = lane / 16: then the B operand
//     g[p][d] is exactly the lane's own accumulator element r, and A is the
//     float4 E[code][16 mt + 4 (lane / 16) .. + 3].
// Pass 1 sums, per pixel, <a, b>, |a|^2, |b|^2 and |a - b|_1 (a = G^, b = G*)
// over the lane's columns, then over the four lanes holding the pixel (lane
// swaps at distance 32 and 16: every lane ends with the same bits).  Pass 2
// recomputes the tiles, forms
//   g_d = lambda [ -(b_d / den - [den > eps] cos a_d / |a|^2) / n + sign(a_d - b_d) / (n D) ]
// and accumulates dL/dw.  The loss of the workgroup's valid pixels goes to
// partial[block], summed in a fixed order.
template <int L>
__global__ void __launch_bounds__(256) sem_loss_kernel(const float* __restrict__ wmap, int64_t P, int D,
                                                      const float* __restrict__ E,
                                                      const float* __restrict__ Gs,
                                                      const uint8_t* __restrict__ V, float lambda,
                                                      const int* __restrict__ counts,
                                                      float* __restrict__ d_out, float* __restrict__ partial) {
    constexpr int KS = L / 4;             // code steps of the decode
    constexpr int CT = (L + 15) / 16;     // code tiles of the gradient
    constexpr int NP = SEM_NPT;           // 16-pixel tiles per wavefront
    __shared__ float wsum[4];
    const int t = threadIdx.x, lane = t & 63, hi = lane >> 4, lo = lane & 15;
    const int q = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t p0 = (int64_t)blockIdx.x * SEM_PIX + 16 * NP * q;
    int64_t pix[NP], pc[NP];
    bool in[NP], valid[NP];
    float wb[NP][KS];  // B operand of the decode: W[p][code = 4 ks + hi]
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        pix[j] = p0 + 16 * j + lo;  // this lane's pixel in tile j (B and accumulator column)
        in[j] = pix[j] < P;
        pc[j] = in[j] ? pix[j] : P - 1;
        valid[j] = in[j] && (V == nullptr || V[pc[j]] != 0);
#pragma unroll
        for (int k = 0; k < KS; ++k) wb[j][k] = wmap[(size_t)(4 + 4 * k + hi) * P + pc[j]];
    }
    const int MT = (D + 15) / 16;

    // Operands of column tile mt, loaded one tile ahead of their use: the
    // decode's A values (E^T) and the targets b (G*).
    struct Tile {
        float ea[KS];
        float b[NP][4];
    };
    auto load_tile = [&](int mt, Tile& o) {
        const int d = 16 * mt + lo;
#pragma unroll
        for (int k = 0; k < KS; ++k) o.ea[k] = d < D ? E[(size_t)(4 * k + hi) * D + d] : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int dr = 16 * mt + 4 * hi + r;
#pragma unroll
            for (int j = 0; j < NP; ++j) o.b[j][r] = dr < D ? Gs[(size_t)dr * P + pc[j]] : 0.f;
        }
    };
    auto decode = [&](const Tile& o, int j) {
        f32x4_t f = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) f = __builtin_amdgcn_mfma_f32_16x16x4f32(o.ea[k], wb[j][k], f, 0, 0, 0);
        return f;
    };

    float s4[NP][4];
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) s4[j][k] = 0.f;
    {
        Tile cur, nxt;
        load_tile(0, cur);
        for (int mt = 0; mt < MT; ++mt) {
            if (mt + 1 < MT) load_tile(mt + 1, nxt);
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const f32x4_t f = decode(cur, j);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float bv = cur.b[j][r];
                    s4[j][0] += f[r] * bv;
                    s4[j][1] += f[r] * f[r];
                    s4[j][2] += bv * bv;
                    s4[j][3] += fabsf(f[r] - bv);
                }
            }
            if (mt + 1 < MT) cur = nxt;
        }
    }
    const int n = valid_total(V, counts, P);
    const float fn = (float)(n > 0 ? n : 1);
    float k1[NP], k2[NP], k3[NP], lj[NP];
    bool live[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float x, y;
            xlane_swap<32>(s4[j][k], s4[j][k], x, y);
            s4[j][k] = x + y;
            xlane_swap<16>(s4[j][k], s4[j][k], x, y);
            s4[j][k] = x + y;
        }
        const float nrm_a = sqrtf(s4[j][1]), nrm_b = sqrtf(s4[j][2]);
        const float prod = nrm_a * nrm_b;
        const float den = fmaxf(prod, kCosEps);
        const float cosv = s4[j][0] / den;
        // g_d = k1 b_d + k2 a_d + k3 sign(a_d - b_d)
        live[j] = valid[j] && n > 0;
        k1[j] = live[j] ? -lambda / (fn * den) : 0.f;
        k2[j] = (live[j] && prod > kCosEps && s4[j][1] > 0.f) ? lambda * cosv / (fn * s4[j][1]) : 0.f;
        k3[j] = live[j] ? lambda / (fn * (float)D) : 0.f;
        lj[j] = live[j] ? lambda * ((1.f - cosv) / fn + s4[j][3] / (fn * (float)D)) : 0.f;
    }
    {
        // this workgroup's share of the loss: pixels in order within a tile
        // (lanes 0..15), tiles in order, then the waves in order
        float wtot = 0.f;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            float v = hi == 0 ? lj[j] : 0.f;
            v += xlane_dpp<8>(v);
            v += xlane_dpp<4>(v);
            v += xlane_dpp<2>(v);
            v += xlane_dpp<1>(v);
            wtot += v;
        }
        if (lane == 0) wsum[q] = wtot;
    }

    f32x4_t acc[NP][CT];
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[j][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    bool any = false;
#pragma unroll
    for (int j = 0; j < NP; ++j) any = any || live[j];
    if (__ballot(any) != 0ull) {
        Tile cur, nxt;
        float4 ec[CT], en[CT];  // gradient A operands: E[16 c + lo][16 mt + 4 hi .. + 3]
        auto load_e4 = [&](int mt, float4 (&o)[CT]) {
            const int d4 = 16 * mt + 4 * hi;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int code = 16 * c + lo;
                o[c] = (code < L && d4 < D) ? *reinterpret_cast<const float4*>(E + (size_t)code * D + d4)
                                            : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        };
        load_tile(0, cur);
        load_e4(0, ec);
        for (int mt = 0; mt < MT; ++mt) {
            if (mt + 1 < MT) {
                load_tile(mt + 1, nxt);
                load_e4(mt + 1, en);
            }
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const f32x4_t f = decode(cur, j);
                float gd[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float df = f[r] - cur.b[j][r];
                    const float sg = df > 0.f ? 1.f : (df < 0.f ? -1.f : 0.f);
                    gd[r] = k1[j] * cur.b[j][r] + k2[j] * f[r] + k3[j] * sg;
                }
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    acc[j][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ec[c].x, gd[0], acc[j][c], 0, 0, 0);
                    acc[j][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ec[c].y, gd[1], acc[j][c], 0, 0, 0);
                    acc[j][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ec[c].z, gd[2], acc[j][c], 0, 0, 0);
                    acc[j][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ec[c].w, gd[3], acc[j][c], 0, 0, 0);
                }
            }
            if (mt + 1 < MT) {
                cur = nxt;
#pragma unroll
                for (int c = 0; c < CT; ++c) ec[c] = en[c];
            }
        }
    }
    // acc[j][c][r]: code 16 c + 4 hi + r, pixel tile j column lo
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        if (!in[j]) continue;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int code = 16 * c + 4 * hi + r;
                if (code < L) d_out[(size_t)(4 + code) * P + pix[j]] = acc[j][c][r];
            }
        if (hi == 0)
#pragma unroll
            for (int c = 0; c < 4; ++c) d_out[(size_t)c * P + pix[j]] = 0.f;
    }
    __syncthreads();
    if (t == 0) partial[blockIdx.x] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
}

// The same with every target read once, for up to 64 tiles of 16 columns (D <=
// 1024): a workgroup takes 32 pixels and holds their targets and decoded values
// in registers between the sums and the gradient, its NW wavefronts splitting
// the column tiles (at most four each: q, q + NW, ...).  The per-pixel sums and
// the gradient's partial products meet in LDS, in wavefront order, and one
// wavefront forms the pixels' coefficients.  Pixel 2 lo + j is column lo of pixel
// tile j, so a lane's two tiles come in one 8-byte load.  A block without a valid
// pixel reads no targets.
//
// What bounds it: latency and issue together.  640 x 480 x 512 under a mask of
// two thirds reads 420 MB, 83 us for a kernel that only loads so; the matrix
// products are 48 us and the arithmetic 65.  The registers are the stage and leave
// two workgroups a CU, so E's operands (L <= 16, where they fit) are asked for
// before the targets and before the barriers: asked for at their use, eight waits
// for L2 a block made 200 us of the 182.  Two reads and two decodes of every
// target (the kernel above) took 302.  More codes are bound by the products: the
// whole call (us) with two reads and so, 32 codes 496 and 267, 64 codes 825 and 528
// (from 513 columns on, 64 codes spill 32 registers a lane: 1,024 1,583 and 966).
constexpr int SEM_REG_PIX = 32;
constexpr int SEM_REG_TILES = 4;   // column tiles of a wavefront

template <class T>
__device__ __forceinline__ const T* lane_at(const float* base, uint32_t bytes) {
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + bytes);
}

template <int L, int NW>
__global__ void __launch_bounds__(64 * NW) sem_loss_regs_kernel(const float* __restrict__ wmap, int64_t P, int D,
                                                               const float* __restrict__ E,
                                                               const float* __restrict__ Gs,
                                                               const uint8_t* __restrict__ V, float lambda,
                                                               const int* __restrict__ counts,
                                                               float* __restrict__ d_out,
                                                               float* __restrict__ partial) {
    typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int KS = L / 4;             // code steps of the decode
    constexpr int CT = (L + 15) / 16;     // code tiles of the gradient
    constexpr int NT = SEM_REG_TILES, PIX = SEM_REG_PIX;
    constexpr bool HELD = L <= 16;        // E's operands are asked for ahead of their use
    __shared__ f32x4_t sums[NW][PIX], coef[PIX];
    __shared__ __align__(16) float red[NW][16][PIX];  // one code tile's partial gradients
    const int t = threadIdx.x, lane = t & 63, hi = lane >> 4, lo = lane & 15;
    const int q = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t p0 = (int64_t)blockIdx.x * PIX;
    const bool full = p0 + PIX <= P;
    const int64_t pa = min(p0 + 2 * lo, P - 1), pb = min(p0 + 2 * lo + 1, P - 1);
    // every wavefront sees the same 32 pixels: the branch is the workgroup's
    const uint64_t even = __ballot(p0 + 2 * lo < P && (V == nullptr || V[pa] != 0));
    const uint64_t odd = __ballot(p0 + 2 * lo + 1 < P && (V == nullptr || V[pb] != 0));
    auto zero_out = [&](int c0, int c1) {
        for (int o = t; o < (c1 - c0) * PIX; o += 64 * NW) {
            const int64_t p = p0 + o % PIX;
            if (p < P) d_out[(size_t)(c0 + o / PIX) * P + p] = 0.f;
        }
    };
    if ((even | odd) == 0) {
        zero_out(0, 4 + L);
        if (t == 0) partial[blockIdx.x] = 0.f;
        return;
    }
    const int MT = (D + 15) / 16;
    // WHOLE: no pixel or column out of range, 32-bit lane offsets in the target rows
    auto body = [&](auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        // the lane's two pixels of row 4 hi + r of a plane group (the group's first row is uniform)
        const uint32_t off = ((uint32_t)(WHOLE ? 4 * hi * P : 0) + 2 * lo) * 4u;
        auto pair = [&](const float* plane) { return f2u{plane[pa], plane[pb]}; };
        // the decode's A values of a tile (E^T), and the gradient's: E[16 c + lo][16 mt + 4 hi .. + 3]
        auto load_ea = [&](int mt, float (&ea)[KS]) {
            const int d = 16 * mt + lo;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                if constexpr (WHOLE) ea[k] = *lane_at<float>(E + (size_t)(4 * k) * D + 16 * mt, (hi * D + lo) * 4u);
                else ea[k] = d < D ? E[(size_t)(4 * k + hi) * D + d] : 0.f;
            }
        };
        auto load_ec = [&](int mt, f4u (&ec)[CT]) {
            const int d4 = 16 * mt + 4 * hi;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                if constexpr (WHOLE && L % 16 == 0)
                    ec[c] = *lane_at<f4u>(E + (size_t)(16 * c) * D + 16 * mt, (lo * D + 4 * hi) * 4u);
                else
                    ec[c] = (16 * c + lo < L && d4 < D) ? *reinterpret_cast<const f4u*>(E + (size_t)(16 * c + lo) * D + d4)
                                                        : f4u{0.f, 0.f, 0.f, 0.f};
            }
        };
        // a wavefront without its last tile loads the last one there is, and leaves it unused;
        // where loads are not whole anyway, it loads none
        auto tile = [&](int i) { return WHOLE ? min(q + NW * i, MT - 1) : q + NW * i; };
        auto load = [&](int i) { return WHOLE || i == 0 || q + NW * i < MT; };
        float wb[2][KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const float* row = wmap + (size_t)(4 + 4 * k + hi) * P;
            const f2u w = WHOLE ? *reinterpret_cast<const f2u*>(row + p0 + 2 * lo) : pair(row);
            wb[0][k] = w[0];
            wb[1][k] = w[1];
        }
        float ea[HELD ? NT : 1][KS];
        if constexpr (HELD)
#pragma unroll
            for (int i = 0; i < NT; ++i)
                if (load(i)) load_ea(tile(i), ea[i]);
        f2u b[NT][4];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if (!load(i)) break;
            const int d0 = 16 * tile(i);  // D % 4 == 0: a lane's four rows are all in or all out
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (WHOLE) b[i][r] = *lane_at<f2u>(Gs + (size_t)(d0 + r) * P + p0, off);
                else b[i][r] = d0 + 4 * hi < D ? pair(Gs + (size_t)(d0 + 4 * hi + r) * P) : f2u{0.f, 0.f};
            }
        }
        zero_out(0, 4);
        f32x4_t f[NT][2];
        float s4[2][4] = {};
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if (q + NW * i >= MT) break;  // uniform
            if constexpr (!HELD) load_ea(q + NW * i, ea[0]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KS; ++k)
                    f[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ea[HELD ? i : 0][k], wb[j][k], f[i][j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float fv = f[i][j][r], bv = b[i][r][j];
                    s4[j][0] += fv * bv;
                    s4[j][1] += fv * fv;
                    s4[j][2] += bv * bv;
                    s4[j][3] += fabsf(fv - bv);
                }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float x, y;
                xlane_swap<32>(s4[j][k], s4[j][k], x, y);
                s4[j][k] = x + y;
                xlane_swap<16>(s4[j][k], s4[j][k], x, y);
                s4[j][k] = x + y;
            }
            if (hi == 0) sums[q][2 * lo + j] = f32x4_t{s4[j][0], s4[j][1], s4[j][2], s4[j][3]};
        }
        f4u ec[HELD ? NT : 1][CT];
        if constexpr (HELD)
#pragma unroll
            for (int i = 0; i < NT; ++i)
                if (load(i)) load_ec(tile(i), ec[i]);
        __syncthreads();
        if (q == (int)(blockIdx.x % NW)) {
            // one wavefront forms the pixels' coefficients, a pixel per lane (twice)
            const int px = lane & 31, n = valid_total(V, counts, P);
            const float fn = (float)(n > 0 ? n : 1);
            f32x4_t s = sums[0][px];
#pragma unroll
            for (int w = 1; w < NW; ++w) s += sums[w][px];
            const float prod = sqrtf(s[1]) * sqrtf(s[2]);
            const float den = fmaxf(prod, kCosEps);
            const float cosv = s[0] / den;
            // g_d = k1 b_d + k2 a_d + k3 sign(a_d - b_d)
            const bool live = ((px & 1 ? odd : even) >> (px >> 1) & 1) != 0 && n > 0;
            f32x4_t k;
            k[0] = live ? -lambda / (fn * den) : 0.f;
            k[1] = (live && prod > kCosEps && s[1] > 0.f) ? lambda * cosv / (fn * s[1]) : 0.f;
            k[2] = live ? lambda / (fn * (float)D) : 0.f;
            k[3] = 0.f;
            if (lane < PIX) coef[px] = k;
            // the block's share of the loss, a fixed tree
            float v = live && lane < PIX ? lambda * ((1.f - cosv) / fn + s[3] / (fn * (float)D)) : 0.f;
            v = wave_sum(v);
            if (lane == 0) partial[blockIdx.x] = v;
        }
        __syncthreads();
        float k1[2], k2[2], k3[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const f32x4_t k = coef[2 * lo + j];
            k1[j] = k[0];
            k2[j] = k[1];
            k3[j] = k[2] * 0x1p22f;  // exact, as is the product with +-2^-22 below
        }
        f32x4_t acc[2][CT];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[j][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if (q + NW * i >= MT) break;
            if constexpr (!HELD) load_ec(q + NW * i, ec[0]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    // sign of the difference times 2^-22, which is 2^127 times the smallest float
                    const float df = f[i][j][r] - b[i][r][j];
                    const float sg = __builtin_amdgcn_fmed3f(df * 0x1p127f, -0x1p-22f, 0x1p-22f);
                    const float gd = k1[j] * b[i][r][j] + k2[j] * f[i][j][r] + k3[j] * sg;
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        acc[j][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(ec[HELD ? i : 0][c][r], gd, acc[j][c], 0, 0, 0);
                }
        }
        // acc[j][c][r]: code 16 c + 4 hi + r, pixel 2 lo + j; one code tile at a time
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            if (c > 0) __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<f2u*>(&red[q][4 * hi + r][2 * lo]) = f2u{acc[0][c][r], acc[1][c][r]};
            __syncthreads();
            for (int o = t; o < 16 * PIX; o += 64 * NW) {
                const int code = o / PIX, px = o % PIX;
                float v = red[0][code][px];
#pragma unroll
                for (int w = 1; w < NW; ++w) v += red[w][code][px];
                if (16 * c + code < L && (WHOLE || p0 + px < P)) d_out[(size_t)(4 + 16 * c + code) * P + p0 + px] = v;
            }
        }
    };
    if (full && D % 16 == 0 && P < (int64_t)1 << 26) body(std::true_type{});
    else body(std::false_type{});
}

// Sums the per-workgroup losses in a fixed order.
__global__ void __launch_bounds__(1024) sem_loss_total_kernel(const float* __restrict__ partial, int nb,
                                                             float* __restrict__ loss) {
    __shared__ float r[1024];
    float s = 0.f;
#pragma unroll 4
    for (int i = threadIdx.x; i < nb; i += 1024) s += partial[i];
    r[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o >= 1; o >>= 1) {
        if (threadIdx.x < o) r[threadIdx.x] += r[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = r[0];
}

static bool sem_l_ok(int L) { return L == 4 || L == 8 || L == 16 || L == 32 || L == 64; }

}  // namespace xgs

using namespace xgs;

#define XGS_SEM_DISPATCH(L, call) \
    switch (L) {                  \
        case 4: call(4); break;   \
        case 8: call(8); break;   \
        case 16: call(16); break; \
        case 32: call(32); break; \
        default: call(64); break; \
    }

extern "C" xgs_status xgs_semantic_softmax(const float* z, int64_t N, int32_t L, float* w, xgs_stream_t stream) {
    clear_error();
    if (N < 0 || !sem_l_ok(L)) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_softmax: L must be 4, 8, 16, 32 or 64");
    if (N == 0) return XGS_OK;
    if (!z || !w) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_softmax: null pointer");
    if (!aligned(z, 16) || !aligned(w, 16)) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_softmax: 16-byte alignment");
    const dim3 grid((unsigned)((N + 255) / 256));
#define XGS_SM(LL) hipLaunchKernelGGL(sem_softmax_kernel<LL>, grid, dim3(256), 0, (hipStream_t)stream, z, N, w)
    XGS_SEM_DISPATCH(L, XGS_SM)
#undef XGS_SM
    return check_launch("xgs_semantic_softmax");
}

extern "C" xgs_status xgs_semantic_softmax_bwd(const float* w, const float* dw, int64_t N, int32_t L, float* dz,
                                               xgs_stream_t stream) {
    clear_error();
    if (N < 0 || !sem_l_ok(L)) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_softmax_bwd: L must be 4, 8, 16, 32 or 64");
    if (N == 0) return XGS_OK;
    if (!w || !dw || !dz) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_softmax_bwd: null pointer");
    if (!aligned(w, 16) || !aligned(dw, 16) || !aligned(dz, 16))
        return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_softmax_bwd: 16-byte alignment");
    const dim3 grid((unsigned)((N + 255) / 256));
#define XGS_SMB(LL) hipLaunchKernelGGL(sem_softmax_bwd_kernel<LL>, grid, dim3(256), 0, (hipStream_t)stream, w, dw, N, dz)
    XGS_SEM_DISPATCH(L, XGS_SMB)
#undef XGS_SMB
    return check_launch("xgs_semantic_softmax_bwd");
}

// Workgroups of the two forms: the one that holds its targets in registers takes
// up to 64 column tiles (four a wavefront, 16 wavefronts), the other what is beyond,
// calls whose workspace holds only the other's partial losses, and those below.
static size_t sem_blocks(int64_t P, int pix) { return (size_t)((P + pix - 1) / pix); }
constexpr int kSemRegsMaxD = 16 * 16 * SEM_REG_TILES;

// Whether two reads of every target are the faster form: without a mask (which spares
// the register form whole blocks), over so many pixels that both fill the card, where
// the register form has wavefronts for many more tiles than there are; more so where
// its loads are not whole (D % 16 != 0).  640 x 480, registers / two reads (us): 16
// codes, D = 320 158 / 190, 516 364 / 303, 528 359 / 304, 592 384 / 343, 656 393 /
// 382; 4 codes, 772 404 / 367, 900 447 / 426; 32 codes, 516 545 / 487, 644 618 / 606;
// 64 codes, 260 521 / 449, 388 654 / 641.  16 codes, D = 516: at 256 x 256 67 / 75, at
// 256 x 384 99 / 93.
static bool sem_reads_twice(int64_t P, int L, int D, bool mask) {
    if (mask || P < 98304) return false;
    const int tiles = (D + 15) / 16;
    const bool ragged = D % 16 != 0;
    if (L <= 16) return tiles > 32 && tiles <= (ragged ? 56 : 40);
    return ragged && ((tiles > 32 && tiles <= 36) || (L == 64 && tiles > 16 && tiles <= 18));
}

template <int L>
static void launch_sem_regs(int64_t P, int D, const float* wmap, const float* E, const float* Gs, const uint8_t* V,
                            float lambda, const int* counts, float* d_out, float* partial, hipStream_t st) {
    const dim3 nb((unsigned)sem_blocks(P, SEM_REG_PIX));
    auto launch = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, nb, dim3(64 * waves), 0, st, wmap, P, D, E, Gs, V, lambda, counts, d_out, partial);
    };
    const int waves = ((D + 15) / 16 + SEM_REG_TILES - 1) / SEM_REG_TILES;
    if (waves <= 1) launch(sem_loss_regs_kernel<L, 1>, 1);
    else if (waves <= 2) launch(sem_loss_regs_kernel<L, 2>, 2);
    else if (waves <= 4) launch(sem_loss_regs_kernel<L, 4>, 4);
    else if (waves <= 8) launch(sem_loss_regs_kernel<L, 8>, 8);
    else launch(sem_loss_regs_kernel<L, 16>, 16);
}

extern "C" size_t xgs_semantic_loss_workspace(int32_t Hs, int32_t Ws) {
    if (Hs < 1 || Ws < 1) return 0;
    Carve c(nullptr);
    c.take<int>(kCountBlocks);
    c.take<float>(sem_blocks((int64_t)Hs * Ws, SEM_REG_PIX));
    return c.total();
}

extern "C" xgs_status xgs_semantic_loss(const float* wmap, int32_t L, int32_t Hs, int32_t Ws, const float* E,
                                        int32_t D, const float* Gstar, const uint8_t* V, float lambda,
                                        float* d_out, float* loss, void* ws, size_t ws_bytes,
                                        xgs_stream_t stream) {
    clear_error();
    if (!sem_l_ok(L)) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_loss: L must be 4, 8, 16, 32 or 64");
    if (Hs < 1 || Ws < 1 || D < 4 || D % 4 != 0)
        return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_loss: need Hs, Ws >= 1 and D a positive multiple of 4");
    if (!wmap || !E || !Gstar || !d_out || !loss) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_loss: null pointer");
    if (!aligned(E, 16)) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_loss: E must be 16-byte aligned");
    if (!aligned(ws, 256)) return fail(XGS_ERR_INVALID_ARG, "xgs_semantic_loss: workspace must be 256-byte aligned");
    const int64_t P = (int64_t)Hs * Ws;
    Carve c(ws);
    int* counts = c.take<int>(kCountBlocks);
    const size_t regs_bytes = [&] { Carve k = c; k.take<float>(sem_blocks(P, SEM_REG_PIX)); return k.total(); }();
    float* partial = c.take<float>(sem_blocks(P, SEM_PIX));
    if (!ws || ws_bytes < c.total()) return fail(XGS_ERR_CAPACITY, "xgs_semantic_loss: workspace too small");
    hipStream_t st = (hipStream_t)stream;
    if (V) hipLaunchKernelGGL(sem_count_kernel, dim3(kCountBlocks), dim3(1024), 0, st, V, P, counts);
    const bool regs = D <= kSemRegsMaxD && ws_bytes >= regs_bytes && !sem_reads_twice(P, L, D, V != nullptr);
    const unsigned nb = (unsigned)sem_blocks(P, regs ? SEM_REG_PIX : SEM_PIX);
    if (regs) {
#define XGS_SL(LL) launch_sem_regs<LL>(P, D, wmap, E, Gstar, V, lambda, counts, d_out, partial, st)
        XGS_SEM_DISPATCH(L, XGS_SL)
#undef XGS_SL
    } else {
#define XGS_SL(LL)                                                                                              \
    hipLaunchKernelGGL(sem_loss_kernel<LL>, dim3(nb), dim3(256), 0, st, wmap, P, D, E, Gstar, V, lambda, counts, \
                       d_out, partial)
        XGS_SEM_DISPATCH(L, XGS_SL)
#undef XGS_SL
    }
    hipLaunchKernelGGL(sem_loss_total_kernel, dim3(1), dim3(1024), 0, st, partial, (int)nb, loss);
    return check_launch("xgs_semantic_loss");
}
