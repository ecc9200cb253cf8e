// Rank predictor for the admissible blocks: an MLP 8 -> 64 -> 64 -> 64 -> 1
// (ReLU) on geometric block features, trained on the ranks the adaptive ACA
// produces, used to size each block's ACA up front.
//
// Parameters are one float array packed as W1 (64x8, row-major), b1, W2
// (64x64), b2, W3 (64x64), b3, W4 (1x64), b4.  Inputs are standardised with a
// fixed per-feature mean / scale.  Training minimises the pinball (quantile)
// loss with Adam.  Every sum has a fixed order, so forward, backward and updates
// are deterministic.
#include "hmx_internal.h"

namespace hmx {

namespace {

constexpr int kIn = 8;
constexpr int kH = 64;
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + kH * kIn, kOffW2 = kOffB1 + kH,
                  kOffB2 = kOffW2 + kH * kH, kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH * kH,
                  kOffW4 = kOffB3 + kH, kOffB4 = kOffW4 + kH, kNParam = kOffB4 + 1;

// Forward, and with GRAD forward, loss and backward, of tiles of 64 samples in
// one kernel (eight waves, a tile's activations and deltas in LDS, transposed:
// row k holds unit k of the 64 samples).
//   * Forward layers: a lane per sample, eight outputs a wave, the weights in
//     scalar registers; each output is its bias plus the products in unit
//     order, in the vector units (the prediction decides the side of the
//     pinball loss, and keeps the bits of that order).
//   * Backward: the 64 x 64 x 64 contractions dZ' = W^T dZ and gW = dZ A^T on the
//     16x16x4 FP32 matrix instructions; the weight gradients accumulate in
//     registers over a workgroup's tiles and leave it once, as one row of
//     part, which grad_reduce_kernel adds in order.
// Bound by latency: a tile is about 25 us of work of one compute unit whatever
// the batch, up to 64 x kMlpGroups samples.  B = 16384: the forward pass 276 us as
// four launches of a thread per output, now 12 us; loss and gradient 860 us
// as 17 launches, now 33 us.
constexpr int kMT = 64;            // samples per tile
constexpr int kMP = kMT + 4;       // row stride of a tile: 4 i + g over all 64 banks
constexpr int kMW = 8;             // waves
constexpr int kMlpGroups = 256;    // workgroups (rows of part) at most

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct MlpTile {
    float x[kIn * kMP];
    float a1[kH * kMP], a2[kH * kMP], a3[kH * kMP];
    float d0[kH * kMP], d1[kH * kMP];
    float dout[kMT];
};

// out row i = relu(bias_i + sum_k W[i, k] in row k), eight rows a wave; zero for a
// lane that has no sample (live false): what the biases make of no input may be
// infinite, and infinity times its zero delta is no zero
template <int IN>
__device__ __forceinline__ void tile_layer(const float* __restrict__ W, const float* __restrict__ bias,
                                           const float* in, float* out, int wave, int lane,
                                           bool live) {
    const int i0 = wave * 8;
    float s[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] = bias[i0 + u];
#pragma unroll 8
    for (int k = 0; k < IN; ++k) {
        const float x = in[k * kMP + lane];
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] = __builtin_fmaf(W[(i0 + u) * IN + k], x, s[u]);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) out[(i0 + u) * kMP + lane] = live && s[u] > 0.f ? s[u] : 0.f;
}

// dp row k = [a row k > 0] sum_j W[j, k] d row j: wave w forms rows 16 (w / 2)
// .. + 15 of samples 32 (w % 2) .. + 31
__device__ __forceinline__ void tile_delta(const float* __restrict__ W, const float* d,
                                           const float* a, float* dp, int wave, int lane) {
    const int k0 = (wave >> 1) * 16, b0 = (wave & 1) * 32, l = lane & 15, g = lane >> 4;
    f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll 4
    for (int j = 0; j < kH; j += 4) {
        const float wv = W[(j + g) * kH + k0 + l];
        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, d[(j + g) * kMP + b0 + l], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, d[(j + g) * kMP + b0 + 16 + l], c1, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int e = (k0 + 4 * g + v) * kMP + b0 + l;
        dp[e] = a[e] > 0.f ? c0[v] : 0.f;
        dp[e + 16] = a[e + 16] > 0.f ? c1[v] : 0.f;
    }
}

// acc += rows 16 (w / 2) .. of d times rows 32 (w % 2) .. + 31 of a, summed over
// the samples: gW[i, k] += sum_b d[i, b] a[k, b]
__device__ __forceinline__ void tile_wgrad(const float* d, const float* a, f32x4 (&acc)[2], int wave,
                                           int lane) {
    const int i0 = (wave >> 1) * 16, k0 = (wave & 1) * 32, l = lane & 15, g = lane >> 4;
#pragma unroll 4
    for (int b = 0; b < kMT; b += 4) {
        const float dv = d[(i0 + l) * kMP + b + g];
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, a[(k0 + l) * kMP + b + g], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, a[(k0 + 16 + l) * kMP + b + g], acc[1], 0,
                                                     0, 0);
    }
}

// this thread's eighth of sum_b d[i, b] f[b] (f null: 1), i = thread / 8: the
// eight threads of a row hold its total afterwards
__device__ __forceinline__ float tile_row_sum(const float* d, const float* f, int tid) {
    const float* r = d + (tid >> 3) * kMP;
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int b = (tid & 7) + 8 * q;
        s += f ? r[b] * f[b] : r[b];
    }
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 4, 64);
    return s;
}

// part: gridDim.x rows of kNParam gradients; lpart: their loss sums (FP64)
template <bool GRAD>
__global__ __launch_bounds__(kMW * 64) void mlp_tile_kernel(
    const float* __restrict__ X, const float* __restrict__ y, int64_t B, float q,
    const float* __restrict__ w, const float* __restrict__ mean, const float* __restrict__ scale,
    float* __restrict__ out, float* __restrict__ part, double* __restrict__ lpart) {
    extern __shared__ __align__(16) unsigned char mlp_lds[];
    MlpTile& T = *reinterpret_cast<MlpTile*>(mlp_lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = lane & 15, g = lane >> 4;
    const int64_t ntiles = (B + kMT - 1) / kMT;
    f32x4 g1 = {0.f, 0.f, 0.f, 0.f}, g2[2] = {g1, g1}, g3[2] = {g1, g1};
    float b1 = 0.f, b2 = 0.f, b3 = 0.f, g4 = 0.f, b4 = 0.f;  // rows tid / 8
    double lsum = 0.0;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t s0 = t * kMT;
        const bool live = !GRAD || s0 + lane < B;
        {
            const int b = tid >> 3, k = tid & 7;
            const int64_t sb = s0 + b;
            T.x[k * kMP + b] = sb < B ? (X[sb * kIn + k] - mean[k]) * scale[k] : 0.f;
        }
        __syncthreads();
        tile_layer<kIn>(w + kOffW1, w + kOffB1, T.x, T.a1, wave, lane, live);
        __syncthreads();
        tile_layer<kH>(w + kOffW2, w + kOffB2, T.a1, T.a2, wave, lane, live);
        __syncthreads();
        tile_layer<kH>(w + kOffW3, w + kOffB3, T.a2, T.a3, wave, lane, live);
        __syncthreads();
        if (wave == 0) {
            float o = w[kOffB4];
#pragma unroll 8
            for (int k = 0; k < kH; ++k)
                o = __builtin_fmaf(w[kOffW4 + k], T.a3[k * kMP + lane], o);
            const bool in = s0 + lane < B;
            if constexpr (GRAD) {
                // pinball loss rho_q(y - o) and its derivative by o over B
                const float u = in ? y[s0 + lane] - o : 0.f;
                const float ind = u < 0.f ? 1.f : 0.f;
                T.dout[lane] = in ? -(q - ind) / (float)B : 0.f;
                if (in) lsum += u * (q - ind);
            } else if (in) {
                out[s0 + lane] = o;
            }
        }
        __syncthreads();
        if constexpr (GRAD) {
            // output layer, and the deltas of the third
            g4 += tile_row_sum(T.a3, T.dout, tid);
            if (tid < 64) {
                float s = T.dout[lane];
#pragma unroll
                for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
                b4 += s;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = wave * 8 + u;
                T.d0[k * kMP + lane] =
                    T.a3[k * kMP + lane] > 0.f ? w[kOffW4 + k] * T.dout[lane] : 0.f;
            }
            __syncthreads();
            tile_wgrad(T.d0, T.a2, g3, wave, lane);
            b3 += tile_row_sum(T.d0, nullptr, tid);
            tile_delta(w + kOffW3, T.d0, T.a2, T.d1, wave, lane);
            __syncthreads();
            tile_wgrad(T.d1, T.a1, g2, wave, lane);
            b2 += tile_row_sum(T.d1, nullptr, tid);
            tile_delta(w + kOffW2, T.d1, T.a1, T.d0, wave, lane);
            __syncthreads();
            b1 += tile_row_sum(T.d0, nullptr, tid);
            if (wave < 4) {  // 64 x 8: the lanes of inputs 8 .. 15 repeat input 7
#pragma unroll 4
                for (int b = 0; b < kMT; b += 4)
                    g1 = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        T.d0[(wave * 16 + l) * kMP + b + g],
                        T.x[(l < kIn ? l : kIn - 1) * kMP + b + g], g1, 0, 0, 0);
            }
            __syncthreads();  // the tile's rows are refilled by the next
        }
    }
    if constexpr (GRAD) {
        float* __restrict__ P = part + (int64_t)blockIdx.x * kNParam;
        const int i0 = (wave >> 1) * 16, k0 = (wave & 1) * 32;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + 4 * g + v;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                P[kOffW2 + i * kH + k0 + 16 * h + l] = g2[h][v];
                P[kOffW3 + i * kH + k0 + 16 * h + l] = g3[h][v];
            }
            if (wave < 4 && l < kIn) P[kOffW1 + (wave * 16 + 4 * g + v) * kIn + l] = g1[v];
        }
        if ((tid & 7) == 0) {
            const int i = tid >> 3;
            P[kOffB1 + i] = b1;
            P[kOffB2 + i] = b2;
            P[kOffB3 + i] = b3;
            P[kOffW4 + i] = g4;
        }
        if (wave == 0) {
            lsum = wave_sum(lsum);
            if (lane == 0) {
                P[kOffB4] = b4;
                lpart[blockIdx.x] = lsum;
            }
        }
    }
}

// grad[p] = the rows of part summed (each wave a quarter of them in order, the
// four added in order), *loss = the loss sums over B
__global__ __launch_bounds__(256) void grad_reduce_kernel(const float* __restrict__ part,
                                                          const double* __restrict__ lpart,
                                                          int rows, int64_t B,
                                                          float* __restrict__ grad,
                                                          double* __restrict__ loss) {
    __shared__ float sh[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    const int per = (rows + 3) / 4, r0 = w * per, r1 = r0 + per < rows ? r0 + per : rows;
    float s = 0.f;
    if (p < kNParam) {
#pragma unroll 8
        for (int r = r0; r < r1; ++r) s += part[(int64_t)r * kNParam + p];
    }
    sh[w][lane] = s;
    __syncthreads();
    if (w == 0 && p < kNParam) grad[p] = ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
    if (blockIdx.x == 0 && w == 1 && loss) {
        double t = 0.0;
        for (int r = lane; r < rows; r += 64) t += lpart[r];
        t = wave_sum(t);
        if (lane == 0) *loss = t / (double)B;
    }
}

// Adam step t >= 1 on n parameters (bias-corrected), FP32
__global__ void adam_kernel(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, int64_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// per-feature mean and 1 / std over n samples (FP64 sums, one workgroup per feature)
__global__ void norm_kernel(const float* __restrict__ X, int64_t n, float* __restrict__ mean,
                            float* __restrict__ scale) {
    __shared__ double sh[2][4];
    const int k = blockIdx.x;
    double s = 0.0, s2 = 0.0;
    for (int64_t b = threadIdx.x; b < n; b += blockDim.x) {
        const double v = X[b * kIn + k];
        s += v;
        s2 += v * v;
    }
    s = wave_sum(s);
    s2 = wave_sum(s2);
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = s;
        sh[1][threadIdx.x >> 6] = s2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double S = sh[0][0] + sh[0][1] + sh[0][2] + sh[0][3];
        const double S2 = sh[1][0] + sh[1][1] + sh[1][2] + sh[1][3];
        const double mu = S / (double)n;
        const double var = S2 / (double)n - mu * mu;
        mean[k] = (float)mu;
        scale[k] = (float)(var > 1e-12 ? 1.0 / sqrt(var) : 1.0);
    }
}

// gather a batch of samples by index (indices outside [0, n) are clamped)
__global__ void gather_batch_kernel(const float* __restrict__ X, const float* __restrict__ y,
                                    int64_t n, const int64_t* __restrict__ idx, int64_t B,
                                    float* __restrict__ Xb, float* __restrict__ yb) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b >= B) return;
    int64_t s = idx[b];
    s = s < 0 ? 0 : (s >= n ? n - 1 : s);
    for (int k = 0; k < kIn; ++k) Xb[b * kIn + k] = X[s * kIn + k];
    yb[b] = y[s];
}

// Block features (FP64, cast to float): [log2 m, log2 n, diam_t / l,
// diam_s / l, dist / l, min(diam) / max(dist, 1e-12), d, log10 l^2], from the
// boxes of the block's two clusters (node ids t, s; boxes d-major per node)
// (d: box stride, dfeat: the problem's dimension, feature 6; boxes of a
// batched build are padded to 3 dimensions with zeros, which add exact zeros)
__device__ void block_features(int4 bl, int64_t t, int64_t s, const double* __restrict__ bmin,
                               const double* __restrict__ bmax, int d, int dfeat, double ell,
                               float* f) {
    double dt = 0.0, ds = 0.0, dist2 = 0.0;
    for (int k = 0; k < d; ++k) {
        const double ta = bmin[t * d + k], tb = bmax[t * d + k];
        const double sa = bmin[s * d + k], sb = bmax[s * d + k];
        dt += (tb - ta) * (tb - ta);
        ds += (sb - sa) * (sb - sa);
        double g1 = ta - sb, g2 = sa - tb;
        g1 = g1 < 0.0 ? 0.0 : g1;
        g2 = g2 < 0.0 ? 0.0 : g2;
        dist2 += g1 * g1 + g2 * g2;
    }
    const double Dt = sqrt(dt), Ds = sqrt(ds), dist = sqrt(dist2);
    f[0] = (float)log2((double)(bl.y - bl.x));
    f[1] = (float)log2((double)(bl.w - bl.z));
    f[2] = (float)(Dt / ell);
    f[3] = (float)(Ds / ell);
    f[4] = (float)(dist / ell);
    f[5] = (float)((Dt < Ds ? Dt : Ds) / (dist > 1e-12 ? dist : 1e-12));
    f[6] = (float)dfeat;
    f[7] = (float)log10(ell * ell);
}

// training pairs: features of every block and (optionally) its ACA rank as float
__global__ void features_kernel(const int4* __restrict__ blocks, const int2* __restrict__ ids,
                                int64_t nb, const double* __restrict__ bmin,
                                const double* __restrict__ bmax, int d, double ell,
                                const int32_t* __restrict__ rank, float* __restrict__ F,
                                float* __restrict__ y) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b >= nb) return;
    float f[kIn];
    block_features(blocks[b], ids[b].x, ids[b].y, bmin, bmax, d, d, ell, f);
    for (int k = 0; k < kIn; ++k) F[b * kIn + k] = f[k];
    if (y) y[b] = (float)rank[b];
}

// Fused rank prediction, one thread per admissible block: features, input
// standardisation, the four layers with the weights staged in LDS (every lane
// reads the same weight at the same time, so LDS broadcasts), and the ACA
// target clamp(ceil(pred) + 1, 1, min(kmax, m, n)).  The sums run in the same
// order as in mlp_tile_kernel.
constexpr int kInferThreads = 256;

__global__ __launch_bounds__(kInferThreads) void rank_predict_kernel(
    const int4* __restrict__ blocks, const int2* __restrict__ ids, int64_t nb,
    const double* __restrict__ bmin, const double* __restrict__ bmax, int d, double ell,
    const float* __restrict__ w, const float* __restrict__ mean, const float* __restrict__ scale,
    int kmax, float* __restrict__ pred_out, int32_t* __restrict__ target,
    const int64_t* __restrict__ pbase, int np, const double* __restrict__ ell_p,
    const int32_t* __restrict__ dim_p) {
    __shared__ float sw[kNParam];
    for (int i = threadIdx.x; i < kNParam; i += kInferThreads) sw[i] = w[i];
    __syncthreads();
    const int64_t b = blockIdx.x * (int64_t)kInferThreads + threadIdx.x;
    if (b >= nb) return;
    const int4 bl = blocks[b];
    float x[kIn];
    if (pbase) {  // many problems: the block's problem gives l and d
        const int p = problem_of(pbase, np, bl.x);
        block_features(bl, ids[b].x, ids[b].y, bmin, bmax, 3, dim_p[p], ell_p[p], x);
    } else {
        block_features(bl, ids[b].x, ids[b].y, bmin, bmax, d, d, ell, x);
    }
    for (int k = 0; k < kIn; ++k) x[k] = (x[k] - mean[k]) * scale[k];
    float h1[kH], h2[kH];
#pragma unroll
    for (int i = 0; i < kH; ++i) {
        float s = sw[kOffB1 + i];
        for (int k = 0; k < kIn; ++k) s += sw[kOffW1 + i * kIn + k] * x[k];
        h1[i] = s > 0.f ? s : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kH; ++i) {
        float s = sw[kOffB2 + i];
#pragma unroll
        for (int k = 0; k < kH; ++k) s += sw[kOffW2 + i * kH + k] * h1[k];
        h2[i] = s > 0.f ? s : 0.f;
    }
    float o = sw[kOffB4];
#pragma unroll
    for (int i = 0; i < kH; ++i) {
        float s = sw[kOffB3 + i];
#pragma unroll
        for (int k = 0; k < kH; ++k) s += sw[kOffW3 + i * kH + k] * h2[k];
        h1[i] = s > 0.f ? s : 0.f;  // third hidden layer reuses h1
    }
    for (int k = 0; k < kH; ++k) o += sw[kOffW4 + k] * h1[k];
    if (pred_out) pred_out[b] = o;
    if (target) {
        int R = kmax;
        R = (bl.y - bl.x) < R ? (bl.y - bl.x) : R;
        R = (bl.w - bl.z) < R ? (bl.w - bl.z) : R;
        int r;
        if (!(o == o)) {
            r = R;  // NaN prediction: full capacity
        } else {
            const float c = ceilf(o) + 1.f;
            r = c < 1.f ? 1 : (c > (float)R ? R : (int)c);
        }
        target[b] = r;
    }
}

// ---- fallback lists of the one-shot ACA ----
__global__ void fail_flags_kernel(const int32_t* __restrict__ rank, int64_t nb,
                                  int64_t* __restrict__ flag) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b < nb) flag[b] = rank[b] < 0 ? 1 : 0;
}

__global__ void over_flags_kernel(const int32_t* __restrict__ rank, const int32_t* __restrict__ rt,
                                  int64_t nb, int64_t* __restrict__ flag) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b < nb) flag[b] = rt[b] > 0 && rank[b] > rt[b] ? 1 : 0;
}

__global__ void gather_failed_kernel(const int32_t* __restrict__ rank,
                                     const int64_t* __restrict__ pos, int64_t nb,
                                     const int4* __restrict__ blocks,
                                     const int32_t* __restrict__ level,
                                     const int32_t* __restrict__ rt, int32_t* __restrict__ list,
                                     int4* __restrict__ blocks_out,
                                     int32_t* __restrict__ level_out,
                                     int32_t* __restrict__ rt_out) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b >= nb || rank[b] >= 0) return;
    const int64_t i = pos[b];
    list[i] = (int32_t)b;
    blocks_out[i] = blocks[b];
    level_out[i] = level[b];
    rt_out[i] = rt[b];
}

__global__ void scatter_i32_kernel(const int32_t* __restrict__ list, int64_t nl,
                                   const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                   int add) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nl) return;
    const int32_t b = list[i];
    dst[b] = add ? dst[b] + src[i] : src[i];
}

__global__ void scatter_i64_kernel(const int32_t* __restrict__ list, int64_t nl,
                                   const int64_t* __restrict__ src, int64_t* __restrict__ dst) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < nl) dst[list[i]] = src[i];
}

unsigned g1d(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

int64_t mlp_nparams() { return kNParam; }

namespace {
unsigned mlp_groups(int64_t B) {
    const int64_t t = (B + kMT - 1) / kMT;
    return (unsigned)(t < kMlpGroups ? t : kMlpGroups);
}
}  // namespace

// out[b] for the B samples of X (which must not overlap out)
hipError_t mlp_forward(const float* w, const float* mean, const float* scale, const float* X,
                       int64_t B, float* out, hipStream_t st) {
    if (B == 0) return hipSuccess;
    const int64_t t = (B + kMT - 1) / kMT;
    hipLaunchKernelGGL(mlp_tile_kernel<false>, dim3((unsigned)(t < (1 << 20) ? t : (1 << 20))),
                       dim3(kMW * 64), sizeof(MlpTile), st, X, nullptr, B, 0.f, w, mean, scale, out,
                       nullptr, nullptr);
    return hipGetLastError();
}

size_t mlp_grad_scratch_bytes(int64_t B) {
    return (size_t)mlp_groups(B) * (kNParam * sizeof(float) + sizeof(double)) + 16;
}

// loss (device double, optional) and gradient of the mean pinball loss over the
// batch; scratch: mlp_grad_scratch_bytes(B)
hipError_t mlp_loss_grad(const float* w, const float* mean, const float* scale, const float* X,
                         const float* y, int64_t B, float q, float* grad, void* scratch,
                         double* loss, hipStream_t st) {
    if (B == 0) return hipSuccess;
    const unsigned groups = mlp_groups(B);
    double* lpart = (double*)scratch;
    float* part = (float*)(lpart + groups);
    hipLaunchKernelGGL(mlp_tile_kernel<true>, dim3(groups), dim3(kMW * 64), sizeof(MlpTile), st, X,
                       y, B, q, w, mean, scale, nullptr, part, lpart);
    hipLaunchKernelGGL(grad_reduce_kernel, dim3((unsigned)((kNParam + 63) / 64)), dim3(256), 0, st,
                       part, lpart, (int)groups, B, grad, loss);
    return hipGetLastError();
}

hipError_t mlp_adam(float* w, float* m, float* v, const float* g, int64_t t, float lr, float b1,
                    float b2, float eps, hipStream_t st) {
    const float c1 = (float)(1.0 - pow((double)b1, (double)t));
    const float c2 = (float)(1.0 - pow((double)b2, (double)t));
    hipLaunchKernelGGL(adam_kernel, dim3(g1d(kNParam)), dim3(256), 0, st, w, m, v, g, kNParam, lr,
                       b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t mlp_norm(const float* X, int64_t n, float* mean, float* scale, hipStream_t st) {
    hipLaunchKernelGGL(norm_kernel, dim3(kIn), dim3(256), 0, st, X, n, mean, scale);
    return hipGetLastError();
}

hipError_t mlp_gather_batch(const float* X, const float* y, int64_t n, const int64_t* idx,
                            int64_t B, float* Xb, float* yb, hipStream_t st) {
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_batch_kernel, dim3(g1d(B)), dim3(256), 0, st, X, y, n, idx, B, Xb,
                       yb);
    return hipGetLastError();
}

hipError_t launch_features(const int4* blocks, const int2* ids, int64_t nb, const double* bmin,
                           const double* bmax, int d, double ell, const int32_t* rank, float* F,
                           float* y, hipStream_t st) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(features_kernel, dim3(g1d(nb)), dim3(256), 0, st, blocks, ids, nb, bmin,
                       bmax, d, ell, rank, F, y);
    return hipGetLastError();
}

hipError_t launch_rank_predict(const int4* blocks, const int2* ids, int64_t nb, const double* bmin,
                               const double* bmax, int d, double ell, const float* w,
                               const float* mean, const float* scale, int kmax, float* pred,
                               int32_t* target, hipStream_t st, const int64_t* pbase, int np,
                               const double* ell_p, const int32_t* dim_p) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(rank_predict_kernel, dim3(g1d(nb, kInferThreads)), dim3(kInferThreads), 0,
                       st, blocks, ids, nb, bmin, bmax, d, ell, w, mean, scale, kmax, pred, target,
                       pbase, np, ell_p, dim_p);
    return hipGetLastError();
}

hipError_t launch_fail_flags(const int32_t* rank, int64_t nb, int64_t* flag, hipStream_t st) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(fail_flags_kernel, dim3(g1d(nb)), dim3(256), 0, st, rank, nb, flag);
    return hipGetLastError();
}

hipError_t launch_over_flags(const int32_t* rank, const int32_t* rt, int64_t nb, int64_t* flag,
                             hipStream_t st) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(over_flags_kernel, dim3(g1d(nb)), dim3(256), 0, st, rank, rt, nb, flag);
    return hipGetLastError();
}

hipError_t launch_gather_failed(const int32_t* rank, const int64_t* pos, int64_t nb,
                                const int4* blocks, const int32_t* level, const int32_t* rt,
                                int32_t* list, int4* blocks_out, int32_t* level_out,
                                int32_t* rt_out, hipStream_t st) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_failed_kernel, dim3(g1d(nb)), dim3(256), 0, st, rank, pos, nb,
                       blocks, level, rt, list, blocks_out, level_out, rt_out);
    return hipGetLastError();
}

hipError_t launch_scatter_i32(const int32_t* list, int64_t nl, const int32_t* src, int32_t* dst,
                              int add, hipStream_t st) {
    if (nl == 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_i32_kernel, dim3(g1d(nl)), dim3(256), 0, st, list, nl, src, dst,
                       add);
    return hipGetLastError();
}

hipError_t launch_scatter_i64(const int32_t* list, int64_t nl, const int64_t* src, int64_t* dst,
                              hipStream_t st) {
    if (nl == 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_i64_kernel, dim3(g1d(nl)), dim3(256), 0, st, list, nl, src, dst);
    return hipGetLastError();
}

}  // namespace hmx
