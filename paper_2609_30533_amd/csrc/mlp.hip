// mlp.hip -- the learned proposal network: forward, loss gradient, backward
// and Adam, on BF16 MFMA with FP32 accumulation (gfx950
// v_mfma_f32_16x16x32_bf16).
//
// Network (one row per problem): a shared per-obstacle encoder
// phi = gelu(obs We + be) max-pooled over the problem's obstacles, the trunk
// x0 = [core(16), pooled(64), 0(16)] -> 4 x (Linear 256 + GELU), and the head
// z = h4 W5 + b5 with 168 outputs: 8 mixture logits, 8 x 8 means, 8 x 8 log
// standard deviations (normalised q/pi and t/60), 32 arrival-histogram logits.
// Weights live in FP32 (master copy for Adam); every GEMM rounds its operands
// to bfloat16 when it packs them for the matrix cores and accumulates in FP32.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "st_internal.hpp"

namespace st {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kEncIn = 65, kEncOut = 64, kCore = 16, kDin = 96, kWidth = 256, kOut = 168;
constexpr int kComp = 8, kDim = 8, kBins = 32;
static_assert(kBins % kComp == 0 && 64 % kComp == 0, "loss lane groups");

// flat parameter layout: We, be, W1, b1, W2, b2, W3, b3, W4, b4, W5, b5
struct MlpLayout {
    int64_t off[12];
    int64_t total;
    MlpLayout() {
        const int shapes[6][2] = {{kEncIn, kEncOut}, {kDin, kWidth}, {kWidth, kWidth},
                                  {kWidth, kWidth},  {kWidth, kWidth}, {kWidth, kOut}};
        int64_t o = 0;
        for (int l = 0; l < 6; ++l) {
            off[2 * l] = o;
            o += (int64_t)shapes[l][0] * shapes[l][1];
            off[2 * l + 1] = o;
            o += shapes[l][1];
        }
        total = o;
    }
};

__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * __expf(-0.5f * x * x) * 0.39894228040143268f;
}

// ---------------------------------------------------------------------------
// One step is nine launches: encoder + pool, trunk, loss, backward chain,
// weight gradients of all layers, bias sums of all layers, encoder gradient,
// the splits' sums, Adam.  With a product per layer and launch (11 to 16 us
// each, of which the arithmetic is a fraction) a forward pass of 276 rows was
// bound by six dependent launches, a step of 4096 rows by forty.
// Every matrix operand is rounded to bfloat16 (nearest even) when it is packed,
// products accumulate in FP32 over k in steps of 32 in ascending order, so an
// output does not depend on how rows and columns are tiled.
// v_mfma_f32_16x16x32_bf16: lane l supplies row l % 16 of A and column l % 16 of
// B at k = 8 (l / 16) .. + 7 and receives rows 4 (l / 16) .. + 3 of column l % 16.
// ---------------------------------------------------------------------------

// ---- encoder and pool ------------------------------------------------------
// phi = gelu(obs We + be), masked max over an example's obstacles (first maximum
// wins), x0 = [core, pooled, 0].  A block takes 64 rows at a time, whole
// examples of O <= 64 rows, which are one contiguous piece of obs; it keeps the
// piece for the backward pass (FP32, as read), and of the pre-activations only
// the ones the maxima were taken at.  Bound by reading and keeping obs (4096
// examples of 32: 68 MB, 13 us at this card's copy rate).
struct EncArgs {
    const float *obs, *mask, *core, *We, *be;
    float *xo, *x0, *pre_sel;
    int32_t *arg;
    int M, O, ex;  // examples per tile
};

constexpr int kEncK = 96, kEncLd = kEncK + 8;  // LDS rows of 65 (+ zeros) bf16, 16 bytes of padding

__global__ __launch_bounds__(256) void k_encode(EncArgs a) {
    __shared__ __attribute__((aligned(16))) __bf16 sA[64][kEncLd], sB[64][kEncLd];
    __shared__ float sP[64][kEncOut + 1];
    __shared__ float sBest[4][kEncOut], sPre[4][kEncOut];
    __shared__ int sArg[4][kEncOut];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles = (a.M + a.ex - 1) / a.ex;
    for (int i = tid; i < 64 * kEncLd; i += 256) (&sA[0][0])[i] = (__bf16)0.f, (&sB[0][0])[i] = (__bf16)0.f;
    __syncthreads();
    for (int i = tid; i < kEncIn * kEncOut; i += 256) sB[i % kEncOut][i / kEncOut] = (__bf16)a.We[i];
    const int r16 = lane & 15, kq = (lane >> 4) * 8, wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int parts = a.ex >= 4 ? 1 : 4 / a.ex;  // threads of a channel that share an example's rows
    // a tile's piece of obs, 17 values per thread, all in flight together and the
    // next tile's while this one is worked on (an index past the end repeats the
    // last value)
    constexpr int kPer = (64 * kEncIn + 255) / 256;
    float nx[kPer];
    const int64_t last = (int64_t)a.M * a.O * kEncIn - 1;
    auto fetch = [&](int tile) {
        const int64_t e0 = (int64_t)tile * a.ex * a.O * kEncIn + tid;
#pragma unroll
        for (int k = 0; k < kPer; ++k) nx[k] = a.obs[min(e0 + 256 * k, last)];
    };
    if ((int)blockIdx.x < tiles) fetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int m0 = tile * a.ex, nm = min(a.ex, a.M - m0);
        const int64_t e0 = (int64_t)m0 * a.O * kEncIn;
        const int cnt = nm * a.O * kEncIn;
        __syncthreads();  // the previous tile's pool has read sP, its product sA
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = tid + 256 * k;
            if (i < cnt) {
                const int r = i / kEncIn;
                sA[r][i - r * kEncIn] = (__bf16)nx[k];
                a.xo[e0 + i] = nx[k];
            }
        }
        if (tile + (int)gridDim.x < tiles) fetch(tile + gridDim.x);
        __syncthreads();
        f32x4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k0 = 0; k0 < kEncK; k0 += 32) {
            bf16x8 u[2], w[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) u[i] = *(const bf16x8 *)&sA[wm + 16 * i + r16][k0 + kq];
#pragma unroll
            for (int j = 0; j < 2; ++j) w[j] = *(const bf16x8 *)&sB[wn + 16 * j + r16][k0 + kq];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[i], w[j], acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = wn + 16 * j + r16;
                const float bn = a.be[n];
#pragma unroll
                for (int r = 0; r < 4; ++r) sP[wm + 16 * i + (lane >> 4) * 4 + r][n] = acc[i][j][r] + bn;
            }
        __syncthreads();
        // thread (channel, p): rows p, p + 1 / parts of an example; the parts'
        // maxima combine in row order (an equal one later loses)
        const int ch = tid & 63, slot = wave;
        for (int ex0 = 0; ex0 < nm; ex0 += 4 / parts) {
            const int ex = ex0 + slot / parts, p = slot % parts;
            const int lo = a.O * p / parts, hi = a.O * (p + 1) / parts;
            float best = -INFINITY, pre = 0.f;
            int bo = -1;
            if (ex < nm) {
                const float *mk = a.mask + (int64_t)(m0 + ex) * a.O;
                for (int o = lo; o < hi; ++o) {
                    if (!(mk[o] > 0.f)) continue;
                    const float x = sP[ex * a.O + o][ch];
                    const float ph = gelu_f(x);
                    if (ph > best) {
                        best = ph;
                        pre = x;
                        bo = o;
                    }
                }
            }
            if (parts > 1) {
                __syncthreads();
                sBest[slot][ch] = best;
                sPre[slot][ch] = pre;
                sArg[slot][ch] = bo;
                __syncthreads();
                for (int k = 1; k < parts && p == 0; ++k)
                    if (sBest[slot + k][ch] > best) {
                        best = sBest[slot + k][ch];
                        pre = sPre[slot + k][ch];
                        bo = sArg[slot + k][ch];
                    }
            }
            if (ex < nm && p == 0) {
                const int64_t m = m0 + ex;
                a.x0[m * kDin + kCore + ch] = bo >= 0 ? best : 0.f;
                a.pre_sel[m * kEncOut + ch] = pre;
                a.arg[m * kEncOut + ch] = bo;
                if (ch < kCore) a.x0[m * kDin + ch] = a.core[m * kCore + ch];
                else if (ch < kDin - kEncOut) a.x0[m * kDin + kEncOut + ch] = 0.f;
            }
        }
    }
}
static_assert(kOut % 4 == 0 && kEncOut % 4 == 0, "k_sums takes four outputs at a time");
static_assert(kDin - kCore - kEncOut == kCore, "x0 ends in as many zeros as core has entries");

// The encoder's gradient: an example's pooled gradient of a channel goes to the
// one obstacle the maximum was taken at, so dWe[k][c] = sum over examples of
// bf16(obs[arg][k]) bf16(d[c]) with d[c] = dx0[c] gelu'(pre_sel[c]): 65 products
// per example and channel instead of 65 O.  One wave per example, lane = channel,
// the example's rows in LDS (65 floats apart: lanes at different obstacles read
// different banks), the column of We's gradient in 65 registers.  part[z]: block
// z's sums, [65][64] and then the bias's [64].
struct EncBackArgs {
    const float *xo, *dx0, *pre_sel;
    const int32_t *arg;
    float *part;
    int M, O;
};

__global__ __launch_bounds__(256) void k_encode_back(EncBackArgs a) {
    extern __shared__ float s_rows[];  // [waves][O][65]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    float *rows = s_rows + wave * a.O * kEncIn;
    float acc[kEncIn], bias = 0.f;
#pragma unroll
    for (int k = 0; k < kEncIn; ++k) acc[k] = 0.f;
    const int n = a.O * kEncIn;
    for (int64_t m = (int64_t)blockIdx.x * nw + wave; m < a.M; m += (int64_t)gridDim.x * nw) {
        const int o = a.arg[m * kEncOut + lane];
        const float d = o >= 0 ? a.dx0[m * kDin + kCore + lane] * gelu_grad_f(a.pre_sel[m * kEncOut + lane]) : 0.f;
        const float *src = a.xo + m * n;
        // a wave's own rows: its LDS accesses stay in order
        for (int i0 = lane; i0 < n; i0 += 64 * 8) {  // eight loads in flight
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = src[min(i0 + 64 * k, n - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i0 + 64 * k < n) rows[i0 + 64 * k] = (float)(__bf16)v[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const float db = (float)(__bf16)d;
        const float *row = rows + max(o, 0) * kEncIn;
#pragma unroll
        for (int k = 0; k < kEncIn; ++k) acc[k] = fmaf(row[k], db, acc[k]);
        bias += d;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    // the block's sum, wave after wave
    __syncthreads();
    float *red = s_rows;  // [65 + 1][64]
    for (int w = 0; w < nw; ++w) {
        if (wave == w) {
#pragma unroll
            for (int k = 0; k < kEncIn; ++k) red[k * 64 + lane] = w == 0 ? acc[k] : red[k * 64 + lane] + acc[k];
            red[kEncIn * 64 + lane] = w == 0 ? bias : red[kEncIn * 64 + lane] + bias;
        }
        __syncthreads();
    }
    float *out = a.part + (int64_t)blockIdx.x * (kEncIn + 1) * 64;
    for (int i = threadIdx.x; i < (kEncIn + 1) * 64; i += blockDim.x) out[i] = red[i];
}

// ---- trunk: four hidden layers and the head in one launch --------------------
// A block of 16 waves takes 16 RT rows through all layers; their activations pass
// from layer to layer in LDS as the bfloat16 operand (pre-activations and
// activations are kept in FP32 for the backward pass).  A wave takes 16 columns
// of every layer with their weights (all of K) in 64 registers; the next layer's
// are fetched behind its products, ahead of the results and the barrier.  Bound
// by the five weight fetches' latency, then by every block reading the 0.86 MB of
// weights through its CU (6 us at 64 bytes a clock), so rows per block stay small
// while there are CUs for them.  With four waves and four tiles each in turn the
// forward trunk took 35 us, the backward chain 70.
constexpr int kActLd = kWidth + 8;
constexpr int kTrunkThreads = 1024;

// Columns n (clamped) of B(k, n) = W[k N + n], every k = 32 s + 8 (l / 16) + e.
template <int K>
__device__ __forceinline__ void load_cols(const float *W, int N, int n0, float (&b)[kWidth / 4]) {
    const int lane = threadIdx.x & 63, n = min(n0 + (lane & 15), N - 1), kq = (lane >> 4) * 8;
#pragma unroll
    for (int s = 0; s < K / 32; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) b[8 * s + e] = W[(int64_t)(32 * s + kq + e) * N + n];
}
// Columns n (clamped) of B(k, n) = W[n ld + k]; k from KR on reads as zero (KR a
// multiple of 8).
template <int K, int KR>
__device__ __forceinline__ void load_rows(const float *W, int ld, int N, int n0, float (&b)[kWidth / 4]) {
    const int lane = threadIdx.x & 63, n = min(n0 + (lane & 15), N - 1), kq = (lane >> 4) * 8;
#pragma unroll
    for (int s = 0; s < K / 32; ++s) {
        const int k = 32 * s + kq;
        const float4 *src = (const float4 *)(W + (int64_t)n * ld + (K == KR ? k : min(k, KR - 8)));
        const float4 u = src[0], v = src[1];
        const bool in = K == KR || k < KR;
        b[8 * s] = in ? u.x : 0.f;
        b[8 * s + 1] = in ? u.y : 0.f;
        b[8 * s + 2] = in ? u.z : 0.f;
        b[8 * s + 3] = in ? u.w : 0.f;
        b[8 * s + 4] = in ? v.x : 0.f;
        b[8 * s + 5] = in ? v.y : 0.f;
        b[8 * s + 6] = in ? v.z : 0.f;
        b[8 * s + 7] = in ? v.w : 0.f;
    }
}
template <int K, int RT>
__device__ __forceinline__ void mma_cols(const __bf16 (*X)[kActLd], const float (&b)[kWidth / 4], f32x4 (&acc)[RT]) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
    for (int i = 0; i < RT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < K / 32; ++s) {
        bf16x8 w;
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = (__bf16)b[8 * s + e];
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const bf16x8 u = *(const bf16x8 *)&X[16 * i + r16][32 * s + kq];
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u, w, acc[i], 0, 0, 0);
        }
    }
}

struct TrunkArgs {
    const float *x0, *W[6], *bias[6];  // [1 .. 4] hidden layers, [5] the head
    float *pre[5], *h[5], *z, *z_out;
    int M;
};

template <int RT>
__global__ __launch_bounds__(kTrunkThreads) void k_trunk(TrunkArgs a) {
    __shared__ __attribute__((aligned(16))) __bf16 H[2][16 * RT][kActLd];
    const int64_t m0 = (int64_t)blockIdx.x * 16 * RT;
    const int lane = threadIdx.x & 63, n0 = 16 * (threadIdx.x >> 6), n = n0 + (lane & 15), r0 = (lane >> 4) * 4;
    const int rows = (int)min((int64_t)16 * RT, a.M - m0);
    float b[kWidth / 4];
    f32x4 acc[RT];
    load_cols<kDin>(a.W[1], kWidth, n0, b);
    for (int i = threadIdx.x; i < 16 * RT * kDin; i += kTrunkThreads) {
        const int r = i / kDin, k = i - r * kDin;
        H[0][r][k] = (__bf16)(r < rows ? a.x0[(m0 + r) * kDin + k] : 0.f);
    }
    float bias = a.bias[1][n];
    __syncthreads();
#pragma unroll
    for (int l = 1; l <= 4; ++l) {
        if (l == 1) mma_cols<kDin, RT>(H[0], b, acc);
        else mma_cols<kWidth, RT>(H[(l + 1) & 1], b, acc);
        const float bn = bias;
        if (l < 4) {
            load_cols<kWidth>(a.W[l + 1], kWidth, n0, b);
            bias = a.bias[l + 1][n];
        } else if (n0 < kOut) {
            load_cols<kWidth>(a.W[5], kOut, n0, b);
            bias = a.bias[5][min(n, kOut - 1)];
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = 16 * i + r0 + q;
                const float v = acc[i][q] + bn, g = gelu_f(v);
                H[l & 1][r][n] = (__bf16)g;
                if (r < rows) {
                    a.pre[l][(m0 + r) * kWidth + n] = v;
                    a.h[l][(m0 + r) * kWidth + n] = g;
                }
            }
        __syncthreads();
    }
    if (n0 >= kOut) return;
    mma_cols<kWidth, RT>(H[0], b, acc);
    if (n >= kOut) return;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * i + r0 + q;
            if (r >= rows) continue;
            const float v = acc[i][q] + bias;
            a.z[(m0 + r) * kOut + n] = v;
            if (a.z_out) a.z_out[(m0 + r) * kOut + n] = v;
        }
}

// ---- backward chain: dpre_l and dx0, the trunk's shape run in reverse ----------
struct ChainArgs {
    const float *dz, *W[6], *pre[5];
    float *dpre[5], *dx0;
    int M;
};
constexpr int kOutPad = (kOut + 31) / 32 * 32;

template <int RT>
__global__ __launch_bounds__(kTrunkThreads) void k_chain(ChainArgs a) {
    __shared__ __attribute__((aligned(16))) __bf16 H[2][16 * RT][kActLd];
    const int64_t m0 = (int64_t)blockIdx.x * 16 * RT;
    const int lane = threadIdx.x & 63, n0 = 16 * (threadIdx.x >> 6), n = n0 + (lane & 15), r0 = (lane >> 4) * 4;
    const int rows = (int)min((int64_t)16 * RT, a.M - m0);
    float b[kWidth / 4], pre[4 * RT];
    f32x4 acc[RT];
    // the pre-activations of the wave's columns, with the weights (clamped rows)
    auto load_pre = [&](int l) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                pre[4 * i + q] = a.pre[l][(m0 + min(16 * i + r0 + q, rows - 1)) * kWidth + n];
    };
    load_rows<kOutPad, kOut>(a.W[5], kOut, kWidth, n0, b);
    load_pre(4);
    for (int i = threadIdx.x; i < 16 * RT * kOutPad; i += kTrunkThreads) {
        const int r = i / kOutPad, k = i - r * kOutPad;
        H[0][r][k] = (__bf16)(r < rows && k < kOut ? a.dz[(m0 + r) * kOut + k] : 0.f);
    }
    __syncthreads();
    // dpre_l = (dpre_{l+1} W_{l+1}^T) gelu'(pre_l)
#pragma unroll
    for (int l = 4; l >= 1; --l) {
        if (l == 4) mma_cols<kOutPad, RT>(H[0], b, acc);
        else mma_cols<kWidth, RT>(H[l & 1], b, acc);
        if (l > 1) load_rows<kWidth, kWidth>(a.W[l], kWidth, kWidth, n0, b);
        else if (n0 < kDin) load_rows<kWidth, kWidth>(a.W[1], kWidth, kDin, n0, b);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = 16 * i + r0 + q;
                const float v = r < rows ? acc[i][q] * gelu_grad_f(pre[4 * i + q]) : 0.f;
                H[(l + 1) & 1][r][n] = (__bf16)v;
                if (r < rows) a.dpre[l][(m0 + r) * kWidth + n] = v;
            }
        if (l > 1) load_pre(l - 1);
        __syncthreads();
    }
    if (n0 >= kDin) return;
    mma_cols<kWidth, RT>(H[0], b, acc);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * i + r0 + q;
            if (r < rows) a.dx0[(m0 + r) * kDin + n] = acc[i][q];
        }
}

// Rows per block of the two: 16 up to 4096 rows (a block per CU), then 32 (fewer
// passes over the weights).
static int trunk_tiles(int M) { return M <= 4096 ? 1 : 2; }

// ---- weight gradients ---------------------------------------------------------
// dW = X^T D, X [M][m], D [M][n], reduced over the examples: block tile 64 x 64,
// k step 32, the reduction split over enough blocks to fill the device; the
// splits' products are added in split order by k_sums.  One launch covers every
// layer (block -> layer by the first-block table).
struct GradArgs {
    const float *A, *B;   // X, D
    float *C;             // the gradient (one split) or the splits' products
    int M, N, K, kc;      // rows and columns of the gradient, examples, examples per split
    int gx, gy, first;    // grid of the layer, its first block
};
constexpr int kLayers = 5;
struct GradGroup {
    GradArgs g[kLayers];
};

constexpr int kBK = 32, kLdsK = kBK + 8;  // LDS row: 32 bf16 + 16 bytes of padding

// thread: k t / 8, columns 8 (t % 8) .. + 7 of a [K][ld] matrix (ld a multiple of
// 4, rows 16-byte aligned)
__device__ __forceinline__ void grad_load(const float *X, int ld, int c0, int k0, int k1, float (&r)[8]) {
    const int t = threadIdx.x;
    const int k = k0 + (t >> 3), c = c0 + (t & 7) * 8;
    const float *src = X + (int64_t)k * ld + c;
    if (k < k1 && c + 8 <= ld) {
        const float4 u = *(const float4 *)src, v = *(const float4 *)(src + 4);
        r[0] = u.x; r[1] = u.y; r[2] = u.z; r[3] = u.w;
        r[4] = v.x; r[5] = v.y; r[6] = v.z; r[7] = v.w;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = (k < k1 && c + e < ld) ? src[e] : 0.f;
    }
}
__device__ __forceinline__ void grad_store(__bf16 (*s)[kLdsK], const float (&r)[8]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int e = 0; e < 8; ++e) s[(t & 7) * 8 + e][t >> 3] = (__bf16)r[e];
}

__global__ __launch_bounds__(256) void k_grads(GradGroup a) {
    __shared__ __attribute__((aligned(16))) __bf16 sA[64][kLdsK], sB[64][kLdsK];
    int l = 0;
    while (l + 1 < kLayers && (int)blockIdx.x >= a.g[l + 1].first) ++l;
    const GradArgs &g = a.g[l];
    const int bid = blockIdx.x - g.first, bx = bid % g.gx, by = bid / g.gx % g.gy, bz = bid / (g.gx * g.gy);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = by * 64, n0 = bx * 64;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int kb = bz * g.kc, ke = min(g.K, kb + g.kc);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int r16 = lane & 15, kq = (lane >> 4) * 8;
    float ra[8], rb[8];
    if (kb < ke) {
        grad_load(g.A, g.M, m0, kb, ke, ra);
        grad_load(g.B, g.N, n0, kb, ke, rb);
    }
    for (int k0 = kb; k0 < ke; k0 += kBK) {
        grad_store(sA, ra);
        grad_store(sB, rb);
        __syncthreads();
        if (k0 + kBK < ke) {
            grad_load(g.A, g.M, m0, k0 + kBK, ke, ra);
            grad_load(g.B, g.N, n0, k0 + kBK, ke, rb);
        }
        bf16x8 u[2], w[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) u[i] = *(const bf16x8 *)&sA[wm + 16 * i + r16][kq];
#pragma unroll
        for (int j = 0; j < 2; ++j) w[j] = *(const bf16x8 *)&sB[wn + 16 * j + r16][kq];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[i], w[j], acc[i][j], 0, 0, 0);
        __syncthreads();
    }
    float *C = g.C + (int64_t)bz * g.M * g.N;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn + 16 * j + r16;
            if (n >= g.N) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + (lane >> 4) * 4 + r;
                if (m < g.M) C[(int64_t)m * g.N + n] = acc[i][j][r];
            }
        }
}

// Split factor of a weight gradient (K examples): enough blocks to fill the
// device, at least 256 k per split, at most kMaxSplits splits.
constexpr int kMaxSplits = 256;
constexpr int kMaxColSplits = 1024;  // row chunks of a bias column sum at most
static int gemm_splits(int M, int N, int64_t K, int *kc) {
    const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
    int64_t S = std::min<int64_t>((2048 + tiles - 1) / tiles, K / 256);
    S = std::max<int64_t>(1, std::min<int64_t>(S, kMaxSplits));
    int64_t c = (K + S - 1) / S;
    c = (c + kBK - 1) / kBK * kBK;
    *kc = (int)c;
    return (int)((K + c - 1) / c);
}

// ---- bias gradients: column sums in two deterministic passes --------------------
// Block (x, z) of a layer sums columns 64 x .. + 63 over rows [z rc, (z + 1) rc)
// (four row phases per column, combined in LDS) into part[z N + n]; k_sums adds
// the chunks.
struct ColGroup {
    const float *X[kLayers];
    float *part[kLayers];
    int N[kLayers];
    int M, rc;
};
__global__ __launch_bounds__(256) void k_colsums(ColGroup a) {
    __shared__ float red[4][64];
    const int l = blockIdx.z, N = a.N[l];
    const float *X = a.X[l];
    const int c = threadIdx.x & 63, ph = threadIdx.x >> 6;
    const int n = blockIdx.x * 64 + c;
    const int r0 = blockIdx.y * a.rc, r1 = min(a.M, r0 + a.rc);
    float s = 0.f;
    if (n < N)
        for (int m = r0 + ph; m < r1; m += 4) s += X[(int64_t)m * N + n];
    red[ph][c] = s;
    __syncthreads();
    if (ph == 0 && n < N) a.part[l][(int64_t)blockIdx.y * N + n] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

// ---- sums of the splits -----------------------------------------------------------
// out[i] = sum over z of part[z n + i], n a multiple of 4: a block takes 256
// outputs of a segment, thread (o, g) sums the splits z = g (mod 16) of four
// outputs in order, and the 16 group sums are added in group order
// (deterministic for given n and S).  (With 16 or 64 outputs per block the
// blocks of a 4096-row step were many enough to take 18 us.)
constexpr int kMaxSegments = 2 * kLayers + 1;
struct SumGroup {
    const float *part[kMaxSegments];
    float *out[kMaxSegments];
    int n[kMaxSegments], S[kMaxSegments], first[kMaxSegments];
    int count;
};
__global__ __launch_bounds__(1024) void k_sums(SumGroup a) {
    __shared__ f32x4 red[16][64];
    int k = 0;
    while (k + 1 < a.count && (int)blockIdx.x >= a.first[k + 1]) ++k;
    const float *part = a.part[k];
    const int n = a.n[k], S = a.S[k];
    const int o = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int i = (blockIdx.x - a.first[k]) * 256 + 4 * o;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (i < n) {
#pragma unroll 8
        for (int z = g; z < S; z += 16) s += *(const f32x4 *)(part + (int64_t)z * n + i);
    }
    red[g][o] = s;
    __syncthreads();
    if (g == 0 && i < n) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 16; ++q) t += red[q][o];
        *(f32x4 *)(a.out[k] + i) = t;
    }
}

// Reductions over the kComp lanes of one example (groups of 8 lanes).
__device__ __forceinline__ float group_max(float v) {
#pragma unroll
    for (int o = 1; o < kComp; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, kComp));
    return v;
}
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
    for (int o = 1; o < kComp; o <<= 1) v += __shfl_xor(v, o, kComp);
    return v;
}

// Mixture NLL of the path states plus the arrival-bin cross-entropy, and
// dL/dz, the mean over examples folded into dz.  One group of kComp lanes per
// example: lane c owns mixture component c (its means, log standard
// deviations and their gradients, in registers) and arrival bins c, c + 8,
// c + 16, c + 24; the per-state log-sum-exp over components is a reduction
// inside the group.
__global__ __launch_bounds__(256) void k_loss(int M, int K, const float *z, const float *y, const float *ymask,
                                              const float *dmask, const int32_t *ubin, float *dz, float *loss_per) {
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = gid / kComp, c = gid % kComp;
    if (m >= M) return;  // whole groups leave together
    const float *zr = z + (int64_t)m * kOut;
    float *dr = dz + (int64_t)m * kOut;
    const float *dm = dmask + m * kDim;
    float mu[kDim], lsv[kDim], isg[kDim];
    bool on[kDim];
#pragma unroll
    for (int j = 0; j < kDim; ++j) {
        mu[j] = zr[kComp + c * kDim + j];
        lsv[j] = zr[kComp + kComp * kDim + c * kDim + j];
        isg[j] = __expf(-lsv[j]);
        on[j] = dm[j] > 0.f;
    }
    const float zc = zr[c];
    const float lmax = group_max(zc);
    const float lse = lmax + __logf(group_sum(__expf(zc - lmax)));
    float cnt = 0.f;
    for (int k = 0; k < K; ++k) cnt += ymask[m * K + k];
    cnt = fmaxf(cnt, 1.f);
    const float inv = 1.f / (cnt * (float)M);
    float nll = 0.f, rsum = 0.f, gmu[kDim], gls[kDim];
#pragma unroll
    for (int j = 0; j < kDim; ++j) gmu[j] = gls[j] = 0.f;
    for (int k = 0; k < K; ++k) {
        const float wk = ymask[m * K + k];
        if (!(wk > 0.f)) continue;  // the same for the whole group
        const float *yk = y + ((int64_t)m * K + k) * kDim;
        float s = zc - lse, df[kDim];
#pragma unroll
        for (int j = 0; j < kDim; ++j) {
            df[j] = (yk[j] - mu[j]) * isg[j];
            if (on[j]) s += -0.5f * df[j] * df[j] - lsv[j] - 0.91893853320467274f;
        }
        const float jmax = group_max(s);
        const float lp = jmax + __logf(group_sum(__expf(s - jmax)));
        nll -= wk * lp;
        const float r = __expf(s - lp) * wk * inv;
        rsum += r;
#pragma unroll
        for (int j = 0; j < kDim; ++j) {
            if (on[j]) {
                gmu[j] -= r * df[j] * isg[j];
                gls[j] -= r * (df[j] * df[j] - 1.f);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kDim; ++j) {
        dr[kComp + c * kDim + j] = gmu[j];
        dr[kComp + kComp * kDim + c * kDim + j] = gls[j];
    }
    const float rtot = group_sum(rsum);
    dr[c] = -(rsum - __expf(zc - lse) * rtot);
    const float *hist = zr + kComp * (1 + 2 * kDim);
    float hb[kBins / kComp];
    float hm = -INFINITY;
#pragma unroll
    for (int i = 0; i < kBins / kComp; ++i) {
        hb[i] = hist[c + kComp * i];
        hm = fmaxf(hm, hb[i]);
    }
    const float hmax = group_max(hm);
    float hs = 0.f;
#pragma unroll
    for (int i = 0; i < kBins / kComp; ++i) hs += __expf(hb[i] - hmax);
    const float hl = hmax + __logf(group_sum(hs));
    const int ub = ubin[m];
#pragma unroll
    for (int i = 0; i < kBins / kComp; ++i) {
        const int bin = c + kComp * i;
        dr[kComp * (1 + 2 * kDim) + bin] = (__expf(hb[i] - hl) - (bin == ub ? 1.f : 0.f)) / (float)M;
    }
    if (c == 0) loss_per[m] = nll / cnt + (hl - hist[ub]);
}

__global__ void k_adam(int64_t n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace st

using namespace st;

struct st_mlp {
    MlpLayout lay;
    int max_M = 0, max_O = 0;
    float *param = nullptr, *grad = nullptr, *am = nullptr, *av = nullptr;
    // kept by the last forward pass
    float *xo = nullptr, *pre_sel = nullptr, *x0 = nullptr, *pre[5] = {}, *h[5] = {}, *z = nullptr;
    int32_t *arg = nullptr;
    // gradients of activations
    float *dz = nullptr, *dpre[5] = {}, *dx0 = nullptr, *loss_per = nullptr;
    // the weight gradients' split products, the bias sums' chunks, the encoder's
    // block sums
    float *ws = nullptr;
    int M = 0, O = 0;
    int64_t step = 0;
};

namespace st {
static void mlp_free(st_mlp *n) {
    void *b[] = {n->param, n->grad, n->am, n->av, n->xo, n->pre_sel, n->x0, n->z, n->arg, n->dz,
                 n->dx0, n->loss_per, n->ws};
    for (void *x : b)
        if (x) (void)hipFree(x);
    for (int l = 0; l < 5; ++l) {
        if (n->pre[l]) (void)hipFree(n->pre[l]);
        if (n->h[l]) (void)hipFree(n->h[l]);
        if (n->dpre[l]) (void)hipFree(n->dpre[l]);
    }
    delete n;
}

// rows and columns of the dense layers' weights, layer 1 .. 5
static const int kLayerIn[kLayers] = {kDin, kWidth, kWidth, kWidth, kWidth};
static const int kLayerOut[kLayers] = {kWidth, kWidth, kWidth, kWidth, kOut};
constexpr int kEncBlocks = 512;  // blocks of the encoder's gradient at most
constexpr int64_t kEncPart = (int64_t)(kEncIn + 1) * kEncOut;

static int col_splits(int64_t M) { return (int)std::max<int64_t>(1, std::min<int64_t>(kMaxColSplits, M / 64)); }

// Floats of the workspace for up to M examples (both split counts grow with M).
static int64_t ws_floats(int64_t M) {
    int64_t need = kEncBlocks * kEncPart;
    for (int l = 0; l < kLayers; ++l) {
        // S = min(device's, M / 256): the largest over all batches up to M
        const int64_t tiles = (int64_t)((kLayerIn[l] + 63) / 64) * ((kLayerOut[l] + 63) / 64);
        const int64_t S = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>((2048 + tiles - 1) / tiles, kMaxSplits),
                                                                 M / 256));
        need += S * kLayerIn[l] * kLayerOut[l] + (int64_t)col_splits(M) * kLayerOut[l];
    }
    return need;
}
}  // namespace st

extern "C" {

int st_mlp_create(int32_t max_batch, int32_t max_obstacles, st_mlp **out) {
    if (!out || max_batch < 1 || max_obstacles < 1 || max_obstacles > ST_MAX_OBSTACLES) {
        set_error("st_mlp_create: bad arguments");
        return ST_EINVAL;
    }
    st_mlp *n = new (std::nothrow) st_mlp();
    if (!n) {
        set_error("st_mlp_create: out of host memory");
        return ST_ENOMEM;
    }
    n->max_M = max_batch;
    n->max_O = max_obstacles;
    const int64_t P = n->lay.total, M = max_batch, MO = (int64_t)max_batch * max_obstacles;
    auto al = [&](float **p, int64_t cnt) { return hipMalloc((void **)p, (size_t)std::max<int64_t>(cnt, 1) * 4); };
    hipError_t e = hipSuccess;
    for (float **p : {&n->param, &n->grad, &n->am, &n->av})
        if (e == hipSuccess) e = al(p, P);
    if (e == hipSuccess) e = al(&n->xo, MO * kEncIn);
    if (e == hipSuccess) e = al(&n->pre_sel, M * kEncOut);
    if (e == hipSuccess) e = al(&n->x0, M * kDin);
    if (e == hipSuccess) e = al(&n->dx0, M * kDin);
    for (int l = 1; l <= 4 && e == hipSuccess; ++l) {
        e = al(&n->pre[l], M * kWidth);
        if (e == hipSuccess) e = al(&n->h[l], M * kWidth);
        if (e == hipSuccess) e = al(&n->dpre[l], M * kWidth);
    }
    if (e == hipSuccess) e = al(&n->z, M * kOut);
    if (e == hipSuccess) e = al(&n->dz, M * kOut);
    if (e == hipSuccess) e = al(&n->loss_per, M);
    if (e == hipSuccess) e = al(&n->ws, ws_floats(M));
    if (e == hipSuccess) e = hipMalloc((void **)&n->arg, (size_t)M * kEncOut * 4);
    if (e == hipSuccess) e = hipMemset(n->am, 0, (size_t)P * 4);
    if (e == hipSuccess) e = hipMemset(n->av, 0, (size_t)P * 4);
    if (e == hipSuccess) e = hipMemset(n->param, 0, (size_t)P * 4);
    if (e != hipSuccess) {
        set_error("st_mlp_create: %s", hipGetErrorString(e));
        mlp_free(n);
        return ST_EHIP;
    }
    *out = n;
    return ST_OK;
}

void st_mlp_destroy(st_mlp *n) {
    if (n) mlp_free(n);
}

int64_t st_mlp_param_count(void) { return MlpLayout().total; }

int st_mlp_params(st_mlp *n, const float *host_in, float *host_out) {
    if (!n) {
        set_error("st_mlp_params: null network");
        return ST_EINVAL;
    }
    const size_t bytes = (size_t)n->lay.total * 4;
    if (host_in) {
        ST_HIP(hipMemcpy(n->param, host_in, bytes, hipMemcpyHostToDevice));
        ST_HIP(hipMemset(n->am, 0, bytes));
        ST_HIP(hipMemset(n->av, 0, bytes));
        n->step = 0;
    }
    if (host_out) ST_HIP(hipMemcpy(host_out, n->param, bytes, hipMemcpyDeviceToHost));
    return ST_OK;
}

int st_mlp_grads(st_mlp *n, float *host_out) {
    if (!n || !host_out) {
        set_error("st_mlp_grads: bad arguments");
        return ST_EINVAL;
    }
    ST_HIP(hipDeviceSynchronize());
    ST_HIP(hipMemcpy(host_out, n->grad, (size_t)n->lay.total * 4, hipMemcpyDeviceToHost));
    return ST_OK;
}

int st_mlp_forward(st_mlp *n, int32_t M, int32_t O, const float *core, const float *obs, const float *mask,
                   float *z_out, void *stream) {
    if (!n || M < 1 || M > n->max_M || O < 1 || O > n->max_O || !core || !obs || !mask) {
        set_error("st_mlp_forward: bad arguments");
        return ST_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    n->M = M;
    n->O = O;
    const MlpLayout &L = n->lay;
    const float *P = n->param;
    EncArgs ea{obs, mask, core, P + L.off[0], P + L.off[1], n->xo, n->x0, n->pre_sel, n->arg, M, O, std::max(1, 64 / O)};
    const int tiles = (M + ea.ex - 1) / ea.ex;
    k_encode<<<std::min(tiles, 768), 256, 0, s>>>(ea);  // three blocks per CU
    ST_HIP(hipGetLastError());
    TrunkArgs ta{};
    ta.x0 = n->x0;
    for (int l = 1; l <= 5; ++l) {
        ta.W[l] = P + L.off[2 * l];
        ta.bias[l] = P + L.off[2 * l + 1];
    }
    for (int l = 1; l <= 4; ++l) {
        ta.pre[l] = n->pre[l];
        ta.h[l] = n->h[l];
    }
    ta.z = n->z;
    ta.z_out = z_out;
    ta.M = M;
    if (trunk_tiles(M) == 1) k_trunk<1><<<(M + 15) / 16, kTrunkThreads, 0, s>>>(ta);
    else k_trunk<2><<<(M + 31) / 32, kTrunkThreads, 0, s>>>(ta);
    ST_HIP(hipGetLastError());
    return ST_OK;
}

int st_mlp_loss(st_mlp *n, int32_t K, const float *y, const float *ymask, const float *dmask, const int32_t *ubin,
                float *loss_per_out, void *stream) {
    if (!n || n->M < 1 || K < 1 || !y || !ymask || !dmask || !ubin) {
        set_error("st_mlp_loss: bad arguments (run st_mlp_forward first)");
        return ST_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    k_loss<<<(n->M * kComp + 255) / 256, 256, 0, s>>>(n->M, K, n->z, y, ymask, dmask, ubin, n->dz,
                                                      loss_per_out ? loss_per_out : n->loss_per);
    ST_HIP(hipGetLastError());
    return ST_OK;
}

int st_mlp_backward(st_mlp *n, void *stream) {
    if (!n || n->M < 1) {
        set_error("st_mlp_backward: run st_mlp_forward and st_mlp_loss first");
        return ST_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    const MlpLayout &L = n->lay;
    const float *P = n->param;
    float *G = n->grad;
    const int M = n->M, O = n->O;
    ChainArgs ca{};
    ca.dz = n->dz;
    for (int l = 1; l <= 5; ++l) ca.W[l] = P + L.off[2 * l];
    for (int l = 1; l <= 4; ++l) {
        ca.pre[l] = n->pre[l];
        ca.dpre[l] = n->dpre[l];
    }
    ca.dx0 = n->dx0;
    ca.M = M;
    if (trunk_tiles(M) == 1) k_chain<1><<<(M + 15) / 16, kTrunkThreads, 0, s>>>(ca);
    else k_chain<2><<<(M + 31) / 32, kTrunkThreads, 0, s>>>(ca);
    ST_HIP(hipGetLastError());
    // dW_l = x_{l-1}^T dpre_l and db_l = sum dpre_l of every layer (the head's dz)
    GradGroup gg;
    ColGroup cg;
    SumGroup sg;
    sg.count = 0;
    float *ws = n->ws;
    int blocks = 0;
    auto sum = [&](const float *part, float *out, int cnt, int S) {
        sg.part[sg.count] = part;
        sg.out[sg.count] = out;
        sg.n[sg.count] = cnt;
        sg.S[sg.count] = S;
        sg.first[sg.count] = sg.count == 0 ? 0 : sg.first[sg.count - 1] + (sg.n[sg.count - 1] + 255) / 256;
        sg.count++;
    };
    const int SC = col_splits(M);
    cg.M = M;
    cg.rc = (M + SC - 1) / SC;
    for (int i = 0; i < kLayers; ++i) {
        const int l = i + 1;
        GradArgs &g = gg.g[i];
        g.A = l == 1 ? n->x0 : n->h[l - 1];
        g.B = l == 5 ? n->dz : n->dpre[l];
        g.M = kLayerIn[i];
        g.N = kLayerOut[i];
        g.K = M;
        const int S = gemm_splits(g.M, g.N, M, &g.kc);
        g.gx = (g.N + 63) / 64;
        g.gy = (g.M + 63) / 64;
        g.first = blocks;
        blocks += g.gx * g.gy * S;
        g.C = G + L.off[2 * l];
        if (S > 1) {
            g.C = ws;
            sum(ws, G + L.off[2 * l], g.M * g.N, S);
            ws += (int64_t)S * g.M * g.N;
        }
        cg.X[i] = g.B;
        cg.N[i] = g.N;
        cg.part[i] = ws;
        sum(ws, G + L.off[2 * l + 1], g.N, SC);
        ws += (int64_t)SC * g.N;
    }
    k_grads<<<blocks, 256, 0, s>>>(gg);
    ST_HIP(hipGetLastError());
    k_colsums<<<dim3((kWidth + 63) / 64, SC, kLayers), 256, 0, s>>>(cg);
    ST_HIP(hipGetLastError());
    // encoder: We and be lie next to each other, as a block's sums do; the rows
    // of a block's waves stay within 64 KB of LDS
    const int waves = O <= 56 ? 4 : 2, enc = std::min(kEncBlocks, (M + waves - 1) / waves);
    const size_t lds = std::max<size_t>((size_t)waves * O * kEncIn, (size_t)kEncPart) * sizeof(float);
    EncBackArgs eb{n->xo, n->dx0, n->pre_sel, n->arg, ws, M, O};
    k_encode_back<<<enc, 64 * waves, lds, s>>>(eb);
    ST_HIP(hipGetLastError());
    sum(ws, G + L.off[0], (int)kEncPart, enc);
    const int last = sg.count - 1;
    k_sums<<<sg.first[last] + (sg.n[last] + 255) / 256, 1024, 0, s>>>(sg);
    ST_HIP(hipGetLastError());
    return ST_OK;
}

int st_mlp_adam(st_mlp *n, float lr, void *stream) {
    if (!n || !(lr > 0.f)) {
        set_error("st_mlp_adam: bad arguments");
        return ST_EINVAL;
    }
    n->step++;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)n->step), c2 = 1.f - powf(b2, (float)n->step);
    const int64_t P = n->lay.total;
    k_adam<<<(int)((P + 255) / 256), 256, 0, (hipStream_t)stream>>>(P, n->param, n->grad, n->am, n->av, lr, b1, b2,
                                                                    1e-8f, c1, c2);
    ST_HIP(hipGetLastError());
    return ST_OK;
}

}  // extern "C"
