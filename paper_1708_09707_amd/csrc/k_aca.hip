// Batched adaptive cross approximation (Algorithm 2, Section 5.4.1).
//
// One workgroup per admissible block, each running its own rank loop, so
// blocks stop independently (no global "voting" bounded by the slowest
// block).  The blocks of a chunk are grouped by the larger side's points
// (kAcaClassRows), each size class one launch, the classes concurrent:
//   * up to 512 points (1024 in FP32): aca_lds_kernel, one pass of 1 to 4 rows
//     a thread, the first eight columns of U and V in LDS;
//   * above: aca_kernel, several passes, the columns in memory (the very
//     largest run on many workgroups each, k_aca_split.hip).
// Both are bound by the issue of vector instructions in the small classes
// (registers, LDS and L2 hold the data; the FP64 inner products and their
// reductions are most of the work) and by the latency of the columns' loads in
// the large ones.  The start of this form (256-row passes of one wave, every
// product a reduction of its own, columns in memory) spent 10200 vector
// instructions on an average one-wave block of N = 2 10^5, d = 3; the one-wave
// classes that replace it 3443, 5728 and 8872 (to 64, 128 and 256 points).  ACA phase before and after: N = 200003
// 3-d BF16 eps 3e-3 32.0 -> 14.3 ms, N = 100003 3-d FP32 eps 1e-5 53 -> 27 ms,
// N = 2^20 2-d FP32 33.0 -> 29.5 ms, N = 2^19 2-d FP64 33.5 -> 27.6 ms, N = 4096
// 2-d FP64 0.69 -> 0.43 ms.
// Per step r:
//   1. residual column  u^ = A[:, j] - sum_{l<r} u_l (v_l)_j   (rows over threads)
//   2. row pivot        i  = argmax over unused rows |u^_i| (lowest index on ties)
//      a column whose largest residual entry is <= eps0 times the column's own
//      largest |entry| adds no rank (zero or rounding-noise residual); the
//      lowest unused column is tried next, and kmax such columns end the block
//   3. u_r = u^ / u^_i,  v_r = A[i, :]^T - sum_{l<r} (u_l)_i v_l  (cols over threads)
//   4. |S_r|_F^2 += 2 sum_{l<r} (u_r.u_l)(v_r.v_l) + |u_r|^2 |v_r|^2   in FP64
//   5. stop if |u_r| |v_r| <= eps (1 - aca_eta) / (1 + eps) |S_r|_F
//   6. next column pivot j = argmax over unused columns |(v_r)_j|
// The inner products of step 4 are FP64.  In aca_kernel, with the test applied
// every step, term r's products with the earlier terms are gathered during the residual
// passes of step r + 1, which read those columns anyway (term r + 1 is then
// speculative and dropped if term r's test passes); otherwise the whole
// workgroup computes them after the row, eight previous columns per pass.
// Every pass issues the loads of several previous columns before using them.
// Learned rank sizing gives every block a predicted target: storage for that
// many columns with the test in 5 applied every step (sizing form), or
// exactly that many steps with the test applied to the last term only
// (one-shot form).  A block that reaches its target unfinished continues
// adaptively (the fallback), or, when its storage holds only the target,
// reports rank -1 to be approximated again with k_max columns.
// The first column is the sigma point nearest (FP64, no contraction) to the
// centre of tau's bounding box, so the first cross runs through the block's
// largest entries.
// Used rows/columns are bitmasks in LDS.  U (m x cap) and V (n x cap) are
// column-major in a capacity pool; column r of U doubles as the scratch for
// the residual column.  All reductions have a fixed tree, so the result is
// bit-reproducible from run to run.
#include <climits>

#include "hmx_internal.h"

#include <algorithm>

namespace hmx {

namespace {

constexpr int kDotCols = 8;     // previous columns per inner-product pass
constexpr int kLU = 8;          // previous columns whose loads are in flight together

template <typename T>
struct Arg {
    T best;  // |value|; -1 = none
    int idx;
    T val;   // signed value
};

template <typename T>
__device__ __forceinline__ void arg_combine(Arg<T>& a, const Arg<T>& b) {
    if (b.best > a.best || (b.best == a.best && b.idx < a.idx)) a = b;
}

// ---------------------------------------------------------------------------
// Wave reductions on the DPP crossbar: the quad swaps (lane i with i ^ 1, then
// i ^ 2), the half-row mirror (i with 7 - i) and the row mirror (i with
// 15 - i) leave every lane of a row of 16 holding the row's total; the four
// rows are then combined from scalar reads.  The result is the same on every
// lane and needs no permute indices or LDS traffic.
constexpr int kDppXor1 = 0xB1;        // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;
constexpr int kDppRor8 = 0x128;       // lane i of a row of 16 with lane i ^ 8

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
    return dpp_i<CTRL>(v);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, dpp_i<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)dpp_i<CTRL>((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)dpp_i<CTRL>((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int lane_read(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_read(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double lane_read(double v, int l) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// sum over the wave, (row 0 + row 1) + (row 2 + row 3)
__device__ __forceinline__ double wave_total(double v) {
    v += dpp<kDppXor1>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppHalfMirror>(v);
    v += dpp<kDppMirror>(v);
    return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}

__device__ __forceinline__ double wave_max(double v) {
    double u = dpp<kDppXor1>(v);
    v = u > v ? u : v;
    u = dpp<kDppXor2>(v);
    v = u > v ? u : v;
    u = dpp<kDppHalfMirror>(v);
    v = u > v ? u : v;
    u = dpp<kDppMirror>(v);
    v = u > v ? u : v;
    double r = lane_read(v, 0);
#pragma unroll
    for (int q = 16; q < 64; q += 16) {
        const double t = lane_read(v, q);
        r = t > r ? t : r;
    }
    return r;
}

// v of the lane 32 (16) away added to (maximised with) the own one: the swap
// of the wave's halves (of its odd and even rows of 16) with itself gives
// every lane both values, in the same order on both lanes
template <int N>
__device__ __forceinline__ void lane_swap(uint32_t v, uint32_t& a, uint32_t& b) {
    static_assert(N == 16 || N == 32, "rows of 16 or halves of 32 lanes");
    const auto r = N == 32 ? __builtin_amdgcn_permlane32_swap(v, v, false, false)
                           : __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0];
    b = r[1];
}
template <int N>
__device__ __forceinline__ void lane_pair(float v, float& x, float& y) {
    uint32_t a, b;
    lane_swap<N>(__builtin_bit_cast(uint32_t, v), a, b);
    x = __builtin_bit_cast(float, a);
    y = __builtin_bit_cast(float, b);
}
template <int N>
__device__ __forceinline__ void lane_pair(double v, double& x, double& y) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    uint32_t al, bl, ah, bh;
    lane_swap<N>((uint32_t)u, al, bl);
    lane_swap<N>((uint32_t)(u >> 32), ah, bh);
    x = __builtin_bit_cast(double, ((uint64_t)ah << 32) | al);
    y = __builtin_bit_cast(double, ((uint64_t)bh << 32) | bl);
}

// the largest value of the wave, on every lane
template <typename T>
__device__ __forceinline__ T wave_max_t(T v) {
    T u = dpp<kDppXor1>(v);
    v = u > v ? u : v;
    u = dpp<kDppXor2>(v);
    v = u > v ? u : v;
    u = dpp<kDppHalfMirror>(v);
    v = u > v ? u : v;
    u = dpp<kDppMirror>(v);
    v = u > v ? u : v;
    T a, b;
    lane_pair<16>(v, a, b);
    v = a > b ? a : b;
    lane_pair<32>(v, a, b);
    return a > b ? a : b;
}

// The wave totals of eight values per lane.  The first three exchanges halve
// the values that a lane keeps: a swap of the wave's halves (of its odd and
// even rows of 16) between two values leaves each half (row) with both parts
// of one of them, so their sum needs no selection.  Eight totals take 34
// instructions instead of the 200 of eight separate butterflies; afterwards
// lane i holds the total of value wave_col8(i), the same bits on every lane of
// that value.
__device__ __forceinline__ int wave_col8(int lane) {
    return ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
}
// the first lane that holds the total of value c
__device__ __forceinline__ int wave_lane8(int c) {
    return ((c >> 2) & 1) * 32 + ((c >> 1) & 1) * 16 + (c & 1) * 8;
}

// per half (row) the sum of the two parts of u (first half, even rows) or v
template <int N>
__device__ __forceinline__ double lane_fold(double u, double v) {
    static_assert(N == 16 || N == 32, "rows of 16 or halves of 32 lanes");
    const uint64_t a = __builtin_bit_cast(uint64_t, u), b = __builtin_bit_cast(uint64_t, v);
    const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b,
                   bh = (uint32_t)(b >> 32);
    const auto lo = N == 32 ? __builtin_amdgcn_permlane32_swap(al, bl, false, false)
                            : __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto hi = N == 32 ? __builtin_amdgcn_permlane32_swap(ah, bh, false, false)
                            : __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

__device__ __forceinline__ double wave_total8(const double (&v)[8], int lane) {
    double a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = lane_fold<32>(v[i], v[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; ++i) b[i] = lane_fold<16>(a[i], a[i + 2]);
    const bool h = (lane & 8) != 0;
    double c = (h ? b[1] : b[0]) + dpp<kDppRor8>(h ? b[0] : b[1]);
    c += dpp<kDppXor1>(c);
    c += dpp<kDppXor2>(c);
    c += dpp<kDppHalfMirror>(c);
    return c;
}

// sum over the eight values of wave_total8 (one lane of each), on every lane
__device__ __forceinline__ double wave_cols_total(double v) {
    v += dpp<kDppRor8>(v);
    double x, y;
    lane_pair<16>(v, x, y);
    v = x + y;
    lane_pair<32>(v, x, y);
    return x + y;
}

template <typename T, int CTRL>
__device__ __forceinline__ Arg<T> dpp_arg(const Arg<T>& a) {
    return Arg<T>{dpp<CTRL>(a.best), dpp<CTRL>(a.idx), dpp<CTRL>(a.val)};
}

// the largest |value| of the wave, lowest index on ties (the same element
// whatever the order of combination)
template <typename T>
__device__ __forceinline__ Arg<T> wave_argmax_u(Arg<T> a) {
    arg_combine(a, dpp_arg<T, kDppXor1>(a));
    arg_combine(a, dpp_arg<T, kDppXor2>(a));
    arg_combine(a, dpp_arg<T, kDppHalfMirror>(a));
    arg_combine(a, dpp_arg<T, kDppMirror>(a));
    Arg<T> r{lane_read(a.best, 0), lane_read(a.idx, 0), lane_read(a.val, 0)};
#pragma unroll
    for (int q = 16; q < 64; q += 16)
        arg_combine(r, Arg<T>{lane_read(a.best, q), lane_read(a.idx, q), lane_read(a.val, q)});
    return r;
}

template <typename T, int NW>
struct AcaShared {
    T vec[kMaxRankCap];         // broadcast row of V (step 1) / row of U (step 3)
    double gu[kMaxRankCap];     // u_r . u_l
    double gv[kMaxRankCap];     // v_r . v_l
    double part[NW][kDotCols];  // per-wave partial inner products
    T abest[NW];
    T aval[NW];
    int aidx[NW];
    double dsum[2][NW];
    int imin[NW];
    double dkey[NW];
    int dkidx[NW];
    long long ovf;  // overflow offset granted to the block, or -1
    long long uo, vo;  // the block's current storage offsets (moved by an overflow)
};

// overflow storage of the learned sizing pass (see AcaArgs)
struct Overflow {
    unsigned long long* used;
    int64_t cap, u0, v0;
    int64_t* moved;  // per block of the launch: the offset granted, else left as is
};

// the smallest value of the wave, on every lane
__device__ __forceinline__ int wave_min(int v) {
    int u = dpp<kDppXor1>(v);
    v = u < v ? u : v;
    u = dpp<kDppXor2>(v);
    v = u < v ? u : v;
    u = dpp<kDppHalfMirror>(v);
    v = u < v ? u : v;
    u = dpp<kDppMirror>(v);
    v = u < v ? u : v;
    int r = lane_read(v, 0);
#pragma unroll
    for (int q = 16; q < 64; q += 16) {
        const int t = lane_read(v, q);
        r = t < r ? t : r;
    }
    return r;
}

template <typename T, int NW>
__device__ int block_min_int(int v, AcaShared<T, NW>& sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    v = wave_min(v);
    if (lane == 0) sh.imin[w] = v;
    __syncthreads();
    int r = sh.imin[0];
    for (int q = 1; q < NW; ++q) r = sh.imin[q] < r ? sh.imin[q] : r;
    __syncthreads();
    return r;
}

// min (op = 0) or max (op = 1) of a double across the workgroup
template <typename T, int NW>
__device__ double block_minmax(double v, int op, AcaShared<T, NW>& sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double u = __shfl_xor(v, o, 64);
        v = op ? (u > v ? u : v) : (u < v ? u : v);
    }
    if (lane == 0) sh.dkey[w] = v;
    __syncthreads();
    double r = sh.dkey[0];
    for (int q = 1; q < NW; ++q) r = op ? (sh.dkey[q] > r ? sh.dkey[q] : r)
                                        : (sh.dkey[q] < r ? sh.dkey[q] : r);
    __syncthreads();
    return r;
}

// index of the smallest key (lowest index on ties)
template <typename T, int NW>
__device__ int block_argmin_f64(double key, int idx, AcaShared<T, NW>& sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double k2 = __shfl_xor(key, o, 64);
        const int i2 = __shfl_xor(idx, o, 64);
        if (k2 < key || (k2 == key && i2 < idx)) {
            key = k2;
            idx = i2;
        }
    }
    if (lane == 0) {
        sh.dkey[w] = key;
        sh.dkidx[w] = idx;
    }
    __syncthreads();
    double bk = sh.dkey[0];
    int bi = sh.dkidx[0];
    for (int q = 1; q < NW; ++q)
        if (sh.dkey[q] < bk || (sh.dkey[q] == bk && sh.dkidx[q] < bi)) {
            bk = sh.dkey[q];
            bi = sh.dkidx[q];
        }
    __syncthreads();
    return bi;
}

// reduce acc[0..DC) across the workgroup into out[0..nk) (fixed tree)
template <int DC, typename T, int NW>
__device__ void block_sum_cols(double* acc, int nk, double* out, AcaShared<T, NW>& sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < DC; ++k) acc[k] = wave_sum(acc[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < DC; ++k) sh.part[w][k] = acc[k];
    }
    __syncthreads();
    if ((int)threadIdx.x < nk) {
        double s = sh.part[0][threadIdx.x];
        for (int q = 1; q < NW; ++q) s += sh.part[q][threadIdx.x];
        out[threadIdx.x] = s;
    }
    __syncthreads();
}

// first column: the sigma point nearest to the centre 0.5 (a + b) of tau's
// bounding box, squared distance summed in dimension order, all in FP64
// without contraction (the first point where every distance overflows)
template <typename T, int NT>
__device__ int first_column(const double* __restrict__ soa64, int64_t n, int d, int4 bl,
                            AcaShared<T, NT / kWave>& sh) {
    const int m = bl.y - bl.x, nc = bl.w - bl.z;
    double c[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (k >= d) break;
        double mn = INFINITY, mx = -INFINITY;
        for (int i = threadIdx.x; i < m; i += NT) {
            const double v = soa64[(int64_t)k * n + bl.x + i];
            mn = v < mn ? v : mn;
            mx = v > mx ? v : mx;
        }
        mn = block_minmax(mn, 0, sh);
        mx = block_minmax(mx, 1, sh);
        c[k] = __dmul_rn(0.5, __dadd_rn(mn, mx));
    }
    double best = INFINITY;
    int bi = INT_MAX;
    for (int q = threadIdx.x; q < nc; q += NT) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k >= d) break;
            const double t = __dsub_rn(soa64[(int64_t)k * n + bl.z + q], c[k]);
            s = __dadd_rn(s, __dmul_rn(t, t));
        }
        if (s < best) {
            best = s;
            bi = q;
        }
    }
    bi = block_argmin_f64(best, bi, sh);
    return bi == INT_MAX ? 0 : bi;
}

__device__ __forceinline__ bool bit_get(const uint32_t* m, int i) {
    return (m[i >> 5] >> (i & 31)) & 1u;
}

// products of column p of a column-major matrix X (len rows) with its columns
// l < p into out[0..p), eight columns per pass, FP64, fixed reduction tree
template <typename T, int NT, int DC>
__device__ void column_products(const T* __restrict__ X, int len, int p, double* out,
                                AcaShared<T, NT / kWave>& sh) {
    const T* __restrict__ Xp = X + (int64_t)p * len;
    for (int c0 = 0; c0 < p; c0 += DC) {
        const int nk = p - c0 < DC ? p - c0 : DC;
        const T* __restrict__ Xc = X + (int64_t)c0 * len;
        double acc[DC];
#pragma unroll
        for (int k = 0; k < DC; ++k) acc[k] = 0.0;
        for (int ib = 0; ib < len; ib += 4 * NT) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = ib + threadIdx.x + e * NT;
                if (i < len) {
                    const double x = (double)Xp[i];
#pragma unroll
                    for (int k = 0; k < DC; ++k)
                        if (k < nk) acc[k] += x * (double)Xc[k * len + i];
                }
            }
        }
        block_sum_cols<DC>(acc, nk, out + c0, sh);
    }
}

// Rows i0 + k NT (k < KR) of a pass: indices clamped into [0, len) so that
// every load is issued unconditionally (the loads of a batch then overlap
// instead of each waiting behind the branch of its own bounds test).
template <int NT, int KR>
__device__ __forceinline__ void clamp_rows(int i0, int len, int (&ic)[KR], bool (&ok)[KR]) {
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const int i = i0 + k * NT;
        ok[k] = i < len;
        ic[k] = ok[k] ? i : len - 1;
    }
}

// element at a 32-bit byte offset from a wave-uniform base
template <typename T>
__device__ __forceinline__ T ld_at(const T* __restrict__ base, uint32_t byte_off) {
    return *(const T*)((const char*)base + byte_off);
}

template <typename T>
__device__ __forceinline__ void st_at(T* __restrict__ base, uint32_t byte_off, T v) {
    *(T*)((char*)base + byte_off) = v;
}
// v, as a value the compiler knows nothing of: addresses formed from it are
// formed where they are used, not kept over the whole step loop
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Loads through a raw buffer descriptor on a wave-uniform base: the per-lane
// part of the address is one 32-bit offset shared by all columns of a pass,
// the column offset a scalar.  Every index is clamped into its array before
// the load, so the descriptor's range check never applies (its size is the
// largest the field holds).
constexpr int kBufWord3 = 0x00020000;  // 32-bit data format, the raw-buffer form on CDNA

template <typename T>
struct BufView {
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ explicit BufView(const T* base)
        : rs(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, kBufWord3)) {}
    __device__ __forceinline__ T at(uint32_t voff, uint32_t soff) const;
};

template <>
__device__ __forceinline__ float BufView<float>::at(uint32_t voff, uint32_t soff) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, 0));
}

template <>
__device__ __forceinline__ double BufView<double>::at(uint32_t voff, uint32_t soff) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, 0));
}

// coordinates of point first + row (row's byte offset boff) of a d x n SoA array
template <typename T>
__device__ __forceinline__ void load_pt_buf(const BufView<T>& pts, int64_t n, int d, uint32_t boff,
                                            T* p) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
        p[k] = (k < d) ? pts.at(boff, (uint32_t)((int64_t)k * n * (int64_t)sizeof(T))) : (T)0;
}

// phi of K rows against one point, the branch on the kernel's kind outside
// the rows (coordinates padded to three with zeros)
template <typename T, int K>
__device__ __forceinline__ void phi_rows(const KernelEval<T>& Kf, const T (&x)[K][3], const T* p,
                                         T (&out)[K]) {
#define HMX_PHI_ROWS(KIND)                                                  \
    _Pragma("unroll") for (int k = 0; k < K; ++k) out[k] = phi_ordered<KIND>(Kf, x[k], p)
    switch (Kf.kind) {
        case HMX_GAUSSIAN: HMX_PHI_ROWS(HMX_GAUSSIAN); break;
        case HMX_MATERN32: HMX_PHI_ROWS(HMX_MATERN32); break;
        case HMX_MATERN_NU1:
            // one row after the other: the Bessel sums of several rows at
            // once take more registers than the columns leave
            _Pragma("unroll") for (int k = 0; k < K; ++k) {
                out[k] = phi_ordered<HMX_MATERN_NU1>(Kf, x[k], p);
                __builtin_amdgcn_sched_barrier(0);
            }
            break;
        case HMX_TEST_CONST: HMX_PHI_ROWS(HMX_TEST_CONST); break;
        default: HMX_PHI_ROWS(HMX_TEST_LOWRANK); break;
    }
#undef HMX_PHI_ROWS
}

// acc[l0 + q] += the wave totals of sum_k xp[k] val[q][k] for the columns
// l0 + q < p of a batch of kLU
template <typename T, int KR>
__device__ __forceinline__ void add_products(const T (&val)[kLU][KR], const T (&xp)[KR], int l0,
                                             int p, double* acc, int lane) {
    static_assert(kLU == 8, "wave_total8 takes a batch at a time");
    double s[kLU];
#pragma unroll
    for (int q = 0; q < kLU; ++q) s[q] = 0.0;
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const double x = (double)xp[k];
#pragma unroll
        for (int q = 0; q < kLU; ++q) s[q] += x * (double)val[q][k];
    }
    const double tot = wave_total8(s, lane);
    const int l = l0 + wave_col8(lane);
    if ((lane & 7) == 0 && l < p) acc[l] += tot;
}

// a[k] -= X_l[row k] c_l for l = 0, 1, ..., r - 1 in that order (columns of
// the column-major X, leading dimension ld; coefficients c in LDS), kLU
// columns' loads in flight at once; padding columns beyond r weigh zero.
// With pend, also the products of column p's rows xp[k] (zero on rows outside
// the block) with every column l < p, added to acc[l]: the deferred inner
// products of the open term.
template <typename T, int KR>
__device__ __forceinline__ void subtract_columns(const T* __restrict__ X, int64_t ld, int r,
                                                 const T* coef, const int (&ic)[KR],
                                                 T (&a)[KR], bool pend, int p,
                                                 const T (&xp)[KR], double* acc, int lane) {
    // r and p are the same on every lane; saying so keeps the column bases scalar
    r = __builtin_amdgcn_readfirstlane(r);
    p = __builtin_amdgcn_readfirstlane(p);
    uint32_t off[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) off[k] = (uint32_t)ic[k] * (uint32_t)sizeof(T);
    for (int l0 = 0; l0 < r; l0 += kLU) {
        const BufView<T> cols(X + (int64_t)l0 * ld);
        T c[kLU], val[kLU][KR];
#pragma unroll
        for (int q = 0; q < kLU; ++q) {
            const bool in = l0 + q < r;
            const int l = in ? l0 + q : r - 1;
            c[q] = in ? coef[l] : (T)0;
            const uint32_t soff = (uint32_t)((int64_t)(l - l0) * ld * (int64_t)sizeof(T));
#pragma unroll
            for (int k = 0; k < KR; ++k) val[q][k] = cols.at(off[k], soff);
        }
#pragma unroll
        for (int q = 0; q < kLU; ++q)
#pragma unroll
            for (int k = 0; k < KR; ++k) a[k] -= val[q][k] * c[q];
        if (pend && l0 < p) add_products<T, KR>(val, xp, l0, p, acc, lane);
    }
}

// the same products in the order of the deferred accumulation of the step
// loop (per batch of KR rows per thread: the wave totals of kLU columns, added
// to the wave's row of acc; the waves' rows are summed in order by the caller),
// so that a test taken on them decides as the deferred one would
template <typename T, int NT, int KR>
__device__ void column_products_waved(const T* __restrict__ X, int len, int p,
                                      double (*acc)[kMaxRankCap]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    p = __builtin_amdgcn_readfirstlane(p);
    for (int l = lane; l < p; l += kWave) acc[w][l] = 0.0;
    __syncthreads();
    for (int ib = 0; ib < len; ib += KR * NT) {
        int ic[KR];
        bool ok[KR];
        clamp_rows<NT, KR>(ib + threadIdx.x, len, ic, ok);
        uint32_t off[KR];
        T xp[KR];
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            off[k] = (uint32_t)ic[k] * (uint32_t)sizeof(T);
            const T v = ld_at(X + (int64_t)p * len, off[k]);
            xp[k] = ok[k] ? v : (T)0;
        }
        for (int l0 = 0; l0 < p; l0 += kLU) {
            const BufView<T> cols(X + (int64_t)l0 * len);
            T val[kLU][KR];
#pragma unroll
            for (int q = 0; q < kLU; ++q) {
                const int l = l0 + q < p ? l0 + q : p - 1;
                const uint32_t soff = (uint32_t)((int64_t)(l - l0) * len * (int64_t)sizeof(T));
#pragma unroll
                for (int k = 0; k < KR; ++k) val[q][k] = cols.at(off[k], soff);
            }
            add_products<T, KR>(val, xp, l0, p, acc[w], lane);
        }
    }
    __syncthreads();
}

// a value known to be the same on every lane, in scalar registers
__device__ __forceinline__ long long uniform_i64(long long v) {
    const unsigned long long u = (unsigned long long)v;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// A block of the learned sizing pass that reached its target unfinished:
// request R columns of overflow storage (one atomic, by thread 0), copy the
// r columns computed so far and return the offset granted (the same on every
// thread), or -1 when the reserve is exhausted.
template <typename T, int NT>
__device__ __forceinline__ long long aca_overflow_move(const Overflow& ovf, int m, int nc, int R, int r,
                                                    const T* __restrict__ U,
                                                    const T* __restrict__ V,
                                                    T* __restrict__ Upool, T* __restrict__ Vpool,
                                                    int64_t ubase, int64_t vbase, long long* slot) {
    if (threadIdx.x == 0) {
        const unsigned long long need = (unsigned long long)(m > nc ? m : nc) * (unsigned long long)R;
        const unsigned long long old = atomicAdd(ovf.used, need);
        *slot = old + need <= (unsigned long long)ovf.cap ? (long long)old : -1;
    }
    __syncthreads();
    const long long off = *slot;
    if (off < 0) return -1;
    T* __restrict__ Un = Upool + (ovf.u0 + off - ubase);
    T* __restrict__ Vn = Vpool + (ovf.v0 + off - vbase);
    const int t = opaque(threadIdx.x);
    for (int e = t; e < r * m; e += NT) Un[e] = U[e];
    for (int e = t; e < r * nc; e += NT) Vn[e] = V[e];
    __syncthreads();
    return off;
}

// waves per SIMD the compiler must leave room for: four in FP32 (the steps
// wait on loads, and gain from the occupancy: eight rows a thread at two waves
// took 46 ms instead of 29 for the blocks above 4096 points at N = 2^20), two in
// FP64, whose values take twice the registers.  All values of a step fit these
// registers: the runtime has to map a kernel's private memory at its launch, on
// a card that may be full.  Uniform values are said to be (scalar registers), a
// workgroup has one block and no loop around it, addresses are 32-bit offsets or
// formed where they are used.  With 176 bytes a lane in private memory (FP32; FP64
// 48) the ACA phase took 29.7 ms at N = 2^20 2-d FP32, now 29.1; 28.2 and 27.8-28.5
// at N = 2^19 2-d FP64; 27.8 and 27.6 at N = 100003 3-d FP32.
template <typename T>
constexpr int aca_min_waves() {
    return sizeof(T) == 8 ? 2 : 4;
}

template <typename T, int NT, int KR>
__global__ __launch_bounds__(NT, (aca_min_waves<T>())) void aca_kernel(
    const T* __restrict__ soa, const double* __restrict__ soa64, int64_t n, int d, KernelEval<T> K,
    const int4* __restrict__ blocks, const uint32_t* __restrict__ order, int64_t nblocks,
    const int64_t* __restrict__ uoff, const int64_t* __restrict__ voff, int64_t ubase,
    int64_t vbase, int kmax, double eps, double aca_eta, T eps0, int fixed,
    const int32_t* __restrict__ rtarget, int one_shot_mode, int cap_only, Overflow ovf,
    int lds_words, T* __restrict__ Upool, T* __restrict__ Vpool,
    int32_t* __restrict__ rank_out, int32_t* __restrict__ steps_out) {
    constexpr int NW = NT / kWave;
    constexpr int DC = kDotCols;
    extern __shared__ uint32_t smask[];
    __shared__ AcaShared<T, NW> sh;
    __shared__ double accu[NW][kMaxRankCap];  // deferred products, one row per wave
    __shared__ double accv[NW][kMaxRankCap];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const double tol = lane_read(eps * (1.0 - aca_eta) / (1.0 + eps), 0);

    if ((int64_t)blockIdx.x >= nblocks) return;
    const int64_t b = order[blockIdx.x];
    const int4 bl = blocks[b];
    const int m = bl.y - bl.x, nc = bl.w - bl.z;
    int R = kmax;
    R = m < R ? m : R;
    R = nc < R ? nc : R;
    // the block's storage offsets live in LDS and are read at every step
    // (they move once if the block outgrows its target into overflow
    // storage; a loop-carried pointer would cost the loop its hoisting)
    if (tid == 0) {
        sh.uo = uoff[b] - ubase;
        sh.vo = voff[b] - vbase;
    }
    const BufView<T> rows_pts(soa + bl.x), cols_pts(soa + bl.z);
    const int mw = (m + 31) >> 5, nw = (nc + 31) >> 5;
    const bool single = m <= KR * NT;  // one pass covers every row
    if (mw + nw > lds_words) {  // outside this launch's size class (never by construction)
        if (tid == 0) {
            rank_out[b] = 0;
            if (steps_out) steps_out[b] = 0;
        }
        return;
    }
    uint32_t* rmask = smask;
    uint32_t* cmask = smask + mw;
    for (int q = tid; q < mw + nw; q += NT) smask[q] = 0u;
    __syncthreads();

    // rtarget[b] > 0 bounds the block's columns to a predicted target.
    // Sizing form (one_shot_mode = 0): the stopping test runs every step
    // as in the adaptive method.  One-shot form: the target is reached
    // without the test, which then judges the last term.  A block that
    // reaches its target unfinished either continues adaptively (storage
    // for k_max columns) or, with cap_only (storage for the target only),
    // ends with rank -1 to be approximated again with k_max columns.
    const bool sized = rtarget && rtarget[b] > 0;
    bool one_shot = sized && one_shot_mode;
    int target = sized ? (rtarget[b] < R ? rtarget[b] : R) : R;
    bool refused = false;
    double last_p = 0.0;  // |u_r|^2 |v_r|^2 of the last term
    // With the test applied every step, term p's products with the
    // earlier terms are gathered while the passes of term p + 1 read
    // those columns anyway; term p's test is taken once they are
    // complete, and term p + 1 is dropped if it passes (it was computed
    // speculatively).  The decisions are those of the step-by-step order.
    const bool fuse = !fixed && !one_shot;
    bool pending = false;     // term r - 1's test is still open
    double nu2p = 0.0, nv2p = 0.0;

    int r = 0, ncols_used = 0, nfailed = 0, steps = 0;
    int j = first_column<T, NT>(soa64, n, d, bl, sh);  // (its barriers publish sh.uo, sh.vo)
    double S2 = 0.0;
    for (;;) {
        if (r >= target) {
            if (r >= R) break;
            if (one_shot) {
                one_shot = false;
                if (sqrt(last_p) <= tol * sqrt(S2)) break;
            }
            if (pending) {
                // no room for a speculative term: term r - 1's products now,
                // summed in the order of the deferred accumulation
                column_products_waved<T, NT, KR>(Upool + uniform_i64(sh.uo), m, r - 1, accu);
                column_products_waved<T, NT, KR>(Vpool + uniform_i64(sh.vo), nc, r - 1, accv);
                double cross = 0.0;
                for (int l = 0; l < r - 1; ++l) {
                    double gu = accu[0][l], gv = accv[0][l];
#pragma unroll 4
                    for (int q = 1; q < NW; ++q) {
                        gu += accu[q][l];
                        gv += accv[q][l];
                    }
                    cross += gu * gv;
                }
                __syncthreads();  // every wave has read the rows before any clears them
                S2 += 2.0 * cross + nu2p * nv2p;
                last_p = nu2p * nv2p;
                pending = false;
                if (sqrt(last_p) <= tol * sqrt(S2)) break;
            }
            if (cap_only) {
                // storage for the target only: continue in overflow
                // storage for R columns if the reserve has room
                const long long off = uniform_i64(
                    ovf.used ? aca_overflow_move<T, NT>(ovf, m, nc, R, r,
                                                        Upool + uniform_i64(sh.uo),
                                                        Vpool + uniform_i64(sh.vo), Upool,
                                                        Vpool, ubase, vbase, &sh.ovf)
                             : -1);
                if (off < 0) {
                    refused = true;
                    break;
                }
                if (tid == 0) {
                    sh.uo = ovf.u0 + off - ubase;
                    sh.vo = ovf.v0 + off - vbase;
                    ovf.moved[b] = off;
                }
                __syncthreads();
            }
            target = R;
        }
        // the same on every lane; saying so keeps them in scalar registers
        r = __builtin_amdgcn_readfirstlane(r);
        j = __builtin_amdgcn_readfirstlane(j);
        S2 = lane_read(S2, 0);
        nu2p = lane_read(nu2p, 0);
        nv2p = lane_read(nv2p, 0);
        last_p = lane_read(last_p, 0);
        // columns l < r are only read in a step, column r only written
        T* __restrict__ U = Upool + uniform_i64(sh.uo);
        T* __restrict__ V = Vpool + uniform_i64(sh.vo);
        const T* __restrict__ Uread = U;
        const T* __restrict__ Vread = V;
        const int p = r - 1;  // the open term, when pending
        // ---- step 1: residual column j into U[:, r] ----
        for (int l = opaque(tid); l < r; l += NT) sh.vec[l] = V[(int64_t)l * nc + j];
        if (tid == 0) cmask[j >> 5] |= 1u << (j & 31);
        if (pending)
            for (int l = lane; l < p; l += kWave) {
                accu[w][l] = 0.0;
                accv[w][l] = 0.0;
            }
        __syncthreads();
        ++ncols_used;
        ++steps;
        T yj[3];
        load_pt(soa, n, d, (int64_t)bl.z + j, yj);
        Arg<T> am{(T)-1, INT_MAX, (T)0};
        double colmax = 0.0;
        T keep[KR];  // the residual column itself when the block has one pass of rows
        // KR rows per thread per pass; the trip count is the same for
        // every thread of the workgroup
        for (int ib = 0; ib < m; ib += KR * NT) {
            int ic[KR];
            bool ok[KR];
            clamp_rows<NT, KR>(ib + tid, m, ic, ok);
            T xi[KR][3], a[KR], up[KR];
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                const uint32_t off = (uint32_t)ic[k] * (uint32_t)sizeof(T);
                load_pt_buf(rows_pts, n, d, off, xi[k]);
                up[k] = (T)0;
                if (pending) {
                    const T v = ld_at(Uread + (int64_t)p * m, off);
                    up[k] = ok[k] ? v : (T)0;
                }
            }
            phi_rows<T, KR>(K, xi, yj, a);
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                a[k] = ok[k] ? a[k] : (T)0;
                const double aa0 = a[k] < (T)0 ? -(double)a[k] : (double)a[k];
                colmax = aa0 > colmax ? aa0 : colmax;
            }
            subtract_columns(Uread, m, r, sh.vec, ic, a, pending, p, up, accu[w], lane);
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                keep[k] = a[k];
                if (ok[k]) {
                    const int i = ic[k];
                    if (!single)
                            st_at(U + (int64_t)r * m, (uint32_t)i * (uint32_t)sizeof(T), a[k]);
                    const T aa = a[k] < (T)0 ? -a[k] : a[k];
                    if (!bit_get(rmask, i) && aa > am.best) {
                        am.best = aa;
                        am.idx = i;
                        am.val = a[k];
                    }
                }
            }
        }
        // row pivot and the column's largest |entry| in one reduction
        am = wave_argmax_u(am);
        colmax = wave_max(colmax);
        if constexpr (NW > 1) {
            if (lane == 0) {
                sh.abest[w] = am.best;
                sh.aidx[w] = am.idx;
                sh.aval[w] = am.val;
                sh.dkey[w] = colmax;
            }
            __syncthreads();
            am = Arg<T>{sh.abest[0], sh.aidx[0], sh.aval[0]};
            colmax = sh.dkey[0];
#pragma unroll 4
            for (int q = 1; q < NW; ++q) {
                arg_combine(am, Arg<T>{sh.abest[q], sh.aidx[q], sh.aval[q]});
                colmax = sh.dkey[q] > colmax ? sh.dkey[q] : colmax;
            }
            __syncthreads();
        }
        if (am.idx == INT_MAX || (double)am.best <= (double)eps0 * colmax) {
            // no usable pivot in this column: try the lowest unused column
            ++nfailed;
            if (ncols_used >= nc || nfailed >= kmax) break;
            int cand = INT_MAX;
            for (int q = tid; q < nw; q += NT) {
                const uint32_t word = cmask[q];
                if (word != 0xffffffffu) {
                    const int c = (q << 5) + __ffs(~word) - 1;
                    if (c < nc && c < cand) cand = c;
                }
            }
            cand = block_min_int(cand, sh);
            if (cand == INT_MAX) break;
            j = cand;
            continue;
        }
        const int ip = __builtin_amdgcn_readfirstlane(am.idx);
        const T piv = lane_read(am.val, 0);
        // ---- step 3a: u_r = u^ / pivot; |u_r|^2 is reduced with the row's sums ----
        double nu2 = 0.0;
        T* __restrict__ Ur = U + (int64_t)r * m;
        if (single) {
            int ic[KR];
            bool ok[KR];
            clamp_rows<NT, KR>(opaque(tid), m, ic, ok);
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                if (ok[k]) {
                    const T u = keep[k] / piv;
                    st_at(Ur, (uint32_t)ic[k] * (uint32_t)sizeof(T), u);
                    nu2 += (double)u * (double)u;
                }
            }
        } else {
            for (int ib = 0; ib < m; ib += KR * NT) {
                int ic[KR];
                bool ok[KR];
                clamp_rows<NT, KR>(ib + tid, m, ic, ok);
                T u[KR];
#pragma unroll
                for (int k = 0; k < KR; ++k)
                    u[k] = ld_at(Ur, (uint32_t)ic[k] * (uint32_t)sizeof(T));
#pragma unroll
                for (int k = 0; k < KR; ++k) {
                    if (ok[k]) {
                        u[k] = u[k] / piv;
                        st_at(Ur, (uint32_t)ic[k] * (uint32_t)sizeof(T), u[k]);
                        nu2 += (double)u[k] * (double)u[k];
                    }
                }
            }
        }
        if (!fuse && !fixed) column_products<T, NT, DC>(Uread, m, r, sh.gu, sh);
        for (int l = opaque(tid); l < r; l += NT) sh.vec[l] = U[(int64_t)l * m + ip];
        if (tid == 0) rmask[ip >> 5] |= 1u << (ip & 31);
        __syncthreads();
        // ---- step 3b: residual row i_r into V[:, r] ----
        T xp[3];
        load_pt(soa, n, d, (int64_t)bl.x + ip, xp);
        double nv2 = 0.0;
        Arg<T> cm{(T)-1, INT_MAX, (T)0};
        for (int qb = 0; qb < nc; qb += KR * NT) {
            int ic[KR];
            bool ok[KR];
            clamp_rows<NT, KR>(qb + tid, nc, ic, ok);
            T yq[KR][3], a[KR], vp[KR];
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                const uint32_t off = (uint32_t)ic[k] * (uint32_t)sizeof(T);
                load_pt_buf(cols_pts, n, d, off, yq[k]);
                vp[k] = (T)0;
                if (pending) {
                    const T v = ld_at(Vread + (int64_t)p * nc, off);
                    vp[k] = ok[k] ? v : (T)0;
                }
            }
            phi_rows<T, KR>(K, yq, xp, a);
#pragma unroll
            for (int k = 0; k < KR; ++k) a[k] = ok[k] ? a[k] : (T)0;
            subtract_columns(Vread, nc, r, sh.vec, ic, a, pending, p, vp, accv[w], lane);
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                if (ok[k]) {
                    const int q = ic[k];
                    st_at(V + (int64_t)r * nc, (uint32_t)q * (uint32_t)sizeof(T), a[k]);
                    nv2 += (double)a[k] * (double)a[k];
                    const T aa = a[k] < (T)0 ? -a[k] : a[k];
                    if (!bit_get(cmask, q) && aa > cm.best) {
                        cm.best = aa;
                        cm.idx = q;
                        cm.val = a[k];
                    }
                }
            }
        }
        // next column pivot, |u_r|^2, |v_r|^2 and (term p's products being
        // complete) the cross sum of term p, in one reduction; the rows of
        // the deferred products are read before its closing barrier so
        // that no wave clears them for the next step while another reads
        cm = wave_argmax_u(cm);
        nu2 = wave_total(nu2);
        nv2 = wave_total(nv2);
        if constexpr (NW > 1) {
            if (lane == 0) {
                sh.abest[w] = cm.best;
                sh.aidx[w] = cm.idx;
                sh.aval[w] = cm.val;
                sh.dsum[0][w] = nu2;
                sh.dsum[1][w] = nv2;
            }
            __syncthreads();
            cm = Arg<T>{sh.abest[0], sh.aidx[0], sh.aval[0]};
            nu2 = sh.dsum[0][0];
            nv2 = sh.dsum[1][0];
#pragma unroll 4
            for (int q = 1; q < NW; ++q) {
                arg_combine(cm, Arg<T>{sh.abest[q], sh.aidx[q], sh.aval[q]});
                nu2 += sh.dsum[0][q];
                nv2 += sh.dsum[1][q];
            }
        }
        double cross_p = 0.0;
        if (pending) {
            for (int l = 0; l < p; ++l) {
                double gu = accu[0][l], gv = accv[0][l];
#pragma unroll 4
                for (int q = 1; q < NW; ++q) {
                    gu += accu[q][l];
                    gv += accv[q][l];
                }
                cross_p += gu * gv;
            }
        }
        if constexpr (NW > 1) __syncthreads();
        // ---- step 4: the norm recursion and the stopping test ----
        ++r;
        if (!fuse) {
            double cross = 0.0;
            if (!fixed) {
                column_products<T, NT, DC>(Vread, nc, r - 1, sh.gv, sh);
                for (int l = 0; l < r - 1; ++l) cross += sh.gu[l] * sh.gv[l];
            }
            S2 += 2.0 * cross + nu2 * nv2;
            last_p = nu2 * nv2;
            if (!fixed && !one_shot && sqrt(last_p) <= tol * sqrt(S2)) break;
        } else {
            if (pending) {
                // term r - 2 = p, its products summed over the waves in order
                S2 += 2.0 * cross_p + nu2p * nv2p;
                last_p = nu2p * nv2p;
                if (sqrt(last_p) <= tol * sqrt(S2)) {
                    r -= 1;  // the speculative term is dropped
                    break;
                }
            }
            if (r == 1) {  // the first term has no products
                S2 = nu2 * nv2;
                last_p = S2;
                pending = false;
                if (sqrt(last_p) <= tol * sqrt(S2)) break;
            } else {
                pending = true;
                nu2p = nu2;
                nv2p = nv2;
            }
        }
        // ---- step 6: next column pivot ----
        if (cm.idx == INT_MAX) break;
        j = cm.idx;
    }
    if (tid == 0) {
        rank_out[b] = refused ? -1 : r;
        if (steps_out) steps_out[b] = steps;
    }
}

// ---------------------------------------------------------------------------
// Blocks of at most S = 64 NW K points a side: thread t holds rows and columns
// t, t + NT, ... of the block (one pass) with their points' coordinates in
// registers, and the first nl columns of U and V live in LDS (later ones are
// read back from memory).  A step then reads no memory but the columns past nl: a pivot's row
// of U or column of V is one gather, a lane per column, whose values become
// scalar operands of the updates.  The columns not yet computed hold zeros, so
// they are taken in whole batches.  The products of a new term with the
// earlier ones are taken in the same step (each thread reads its own rows),
// eight columns to a reduction, so no term is computed speculatively, and a
// step of several waves has two barriers.  The pivots, the stopping test and
// the order of every residual update are those of the general kernel.
// ---------------------------------------------------------------------------

// the largest best[k] of the wave and the lowest k, then lane, that has it;
// false when no entry is >= 0
template <typename T, int K>
__device__ __forceinline__ bool wave_pivot(const T (&best)[K], T& top, int& k, int& lane) {
    T v = best[0];
#pragma unroll
    for (int q = 1; q < K; ++q) v = best[q] > v ? best[q] : v;
    top = lane_read(wave_max_t(v), 0);
    if (!(top >= (T)0)) return false;
    unsigned long long hit = 0;
    int kk = 0;
#pragma unroll
    for (int q = K - 1; q >= 0; --q) {
        const unsigned long long h = __ballot(best[q] == top);
        hit = h ? h : hit;
        kk = h ? q : kk;
    }
    k = __builtin_amdgcn_readfirstlane(kk);
    lane = __builtin_amdgcn_readfirstlane(__builtin_ctzll(hit));
    return true;
}

template <typename T, int NW>
struct LdsShared {
    T best[2][NW], val[NW], cmax[NW];
    T pt[2][NW][3];  // the pivot candidates' points
    int idx[3][NW];
    double key[2][NW];
    double pu[NW][kMaxRankCap + 8], pv[NW][kMaxRankCap + 8];  // per-wave products
    long long slot;  // overflow offset granted to the block, or -1
};
template <typename T>
struct LdsShared<T, 1> {
    long long slot;
};

constexpr size_t kLdsBytes = 160 * 1024;  // of a compute unit

// dynamic LDS of the kernel: U and V, nl columns of S + 1 entries (the odd
// stride spreads a row's entries over the banks)
template <typename T, int S>
constexpr size_t aca_lds_bytes(int nl) {
    return (size_t)(2 * nl * (S + 1)) * sizeof(T);
}

template <typename T, int NW, int K>
__global__ __launch_bounds__(NW * kWave) void aca_lds_kernel(
    const T* __restrict__ soa, const double* __restrict__ soa64, int64_t n, int d,
    KernelEval<T> Kf, const int4* __restrict__ blocks, const uint32_t* __restrict__ order,
    int64_t nblocks, const int64_t* __restrict__ uoff, const int64_t* __restrict__ voff,
    int64_t ubase, int64_t vbase, int kmax, double eps, double aca_eta, T eps0, int fixed,
    const int32_t* __restrict__ rtarget, int one_shot_mode, int cap_only, Overflow ovf, int nl,
    T* Upool, T* Vpool, int32_t* __restrict__ rank_out, int32_t* __restrict__ steps_out) {
    constexpr int NT = NW * kWave, S = NT * K, P = S + 1;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ LdsShared<T, NW> sh;
    T* const UL = (T*)lds_raw;
    T* const VL = UL + nl * P;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    double tol2 = eps * (1.0 - aca_eta) / (1.0 + eps);
    tol2 *= tol2;
    for (int64_t o = blockIdx.x; o < nblocks; o += gridDim.x) {
        const int64_t b = __builtin_amdgcn_readfirstlane((int)order[o]);
        const int4 bl = blocks[b];
        const int rlo = __builtin_amdgcn_readfirstlane(bl.x);
        const int clo = __builtin_amdgcn_readfirstlane(bl.z);
        const int m = __builtin_amdgcn_readfirstlane(bl.y) - rlo;
        const int nc = __builtin_amdgcn_readfirstlane(bl.w) - clo;
        if (m > S || nc > S) {  // outside this class (never by construction)
            if (tid == 0) {
                rank_out[b] = 0;
                if (steps_out) steps_out[b] = 0;
            }
            continue;
        }
        int R = kmax;
        R = m < R ? m : R;
        R = nc < R ? nc : R;
        long long uo = uniform_i64(uoff[b] - ubase), vo = uniform_i64(voff[b] - vbase);
        int ir[K], ic[K];  // the thread's rows and columns, clamped into the block
        bool rok[K], cok[K];
        T x[K][3], y[K][3];
        {
            const BufView<T> rp(soa + rlo), cp(soa + clo);
            clamp_rows<NT, K>(tid, m, ir, rok);
            clamp_rows<NT, K>(tid, nc, ic, cok);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                load_pt_buf(rp, n, d, (uint32_t)ir[k] * (uint32_t)sizeof(T), x[k]);
                load_pt_buf(cp, n, d, (uint32_t)ic[k] * (uint32_t)sizeof(T), y[k]);
            }
        }
        for (int e = tid; e < 2 * nl * P; e += NT) UL[e] = (T)0;  // (VL follows UL)
        // first column: the sigma point nearest to the centre of tau's box
        // (lowest index on ties), as in first_column
        int j;
        {
            double key[K];
#pragma unroll
            for (int k = 0; k < K; ++k) key[k] = 0.0;
            for (int a = 0; a < d; ++a) {
                double mn = INFINITY, mx = -INFINITY;
#pragma unroll
                for (int k = 0; k < K; ++k) {  // (clamped indices are rows of tau as well)
                    const double v = soa64[(int64_t)a * n + rlo + ir[k]];
                    mn = v < mn ? v : mn;
                    mx = v > mx ? v : mx;
                }
                mx = wave_max_t(mx);
                mn = -wave_max_t(-mn);
                if constexpr (NW > 1) {
                    if (lane == 0) {
                        sh.key[0][w] = mn;
                        sh.key[1][w] = mx;
                    }
                    __syncthreads();
                    for (int q = 0; q < NW; ++q) {
                        mn = sh.key[0][q] < mn ? sh.key[0][q] : mn;
                        mx = sh.key[1][q] > mx ? sh.key[1][q] : mx;
                    }
                    __syncthreads();
                }
                const double c = __dmul_rn(0.5, __dadd_rn(mn, mx));
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const double t = __dsub_rn(soa64[(int64_t)a * n + clo + ic[k]], c);
                    key[k] = __dadd_rn(key[k], __dmul_rn(t, t));
                }
            }
            double v = INFINITY;
            int iv = INT_MAX;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (cok[k] && key[k] < v) {
                    v = key[k];
                    iv = ic[k];
                }
            const double top = -wave_max_t(-v);
            int cand = v == top ? iv : INT_MAX;
#pragma unroll
            for (int s = 32; s > 0; s >>= 1) {
                const int u = __shfl_xor(cand, s, 64);
                cand = u < cand ? u : cand;
            }
            if constexpr (NW > 1) {
                if (lane == 0) {
                    sh.key[0][w] = top;
                    sh.idx[0][w] = cand;
                }
            }
            __syncthreads();  // (publishes the zeroed LDS columns as well)
            if constexpr (NW > 1) {
                double bk = sh.key[0][0];
                cand = sh.idx[0][0];
                for (int q = 1; q < NW; ++q)
                    if (sh.key[0][q] < bk || (sh.key[0][q] == bk && sh.idx[0][q] < cand)) {
                        bk = sh.key[0][q];
                        cand = sh.idx[0][q];
                    }
                __syncthreads();
            }
            cand = cand == INT_MAX ? 0 : cand;
            j = __builtin_amdgcn_readfirstlane(cand);
        }
        T p[3];  // the pivot's point
        load_pt(soa, n, d, (int64_t)clo + j, p);
        const bool sized = rtarget && rtarget[b] > 0;
        bool one_shot = sized && one_shot_mode;
        int target = sized ? (rtarget[b] < R ? rtarget[b] : R) : R;
        target = __builtin_amdgcn_readfirstlane(target);
        bool refused = false;
        double last_p = 0.0, S2 = 0.0;
        unsigned rused = 0, cused = 0;  // bit k: the thread's row / column k is used

        // the coordinates of row or column k of lane l
        auto point = [&](const T (&pts)[K][3], int k, int l) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                p[c] = lane_read(pts[0][c], l);
#pragma unroll
                for (int q = 1; q < K; ++q) {
                    const T t = lane_read(pts[q][c], l);
                    p[c] = k == q ? t : p[c];
                }
            }
        };
        // a -= F c over the columns l < r in order: F's columns in LDS (FL),
        // then in memory (FG, leading dimension fld, rows ix); the
        // coefficients are row at of the other factor (HL, HG, hld), lane l
        // gathering column l's
        auto update = [&](T (&a)[K], const T* FL, const T* FG, int fld, const int (&ix)[K],
                          const T* HL, const T* HG, int hld, int at, int r) {
            for (int l64 = 0; l64 < r; l64 += kWave) {
                const int lg = l64 + lane;
                T cv = (T)0;
                if (lg < r) cv = lg < nl ? HL[lg * P + at] : HG[(int64_t)lg * hld + at];
                const int end = r - l64 < kWave ? r : l64 + kWave;
                int l0 = l64;
                for (; l0 < end && l0 < nl; l0 += 4) {
                    const T* f = FL + l0 * P + tid;
                    T val[4][K];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int k = 0; k < K; ++k) val[q][k] = f[q * P + k * NT];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const T c = lane_read(cv, l0 - l64 + q);
#pragma unroll
                        for (int k = 0; k < K; ++k) a[k] -= val[q][k] * c;
                    }
                }
                for (; l0 < end; l0 += 4) {
                    const BufView<T> cols(FG + (int64_t)l0 * fld);
                    T val[4][K];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int l = l0 + q < r ? q : r - 1 - l0;
                        const uint32_t soff = (uint32_t)(l * fld) * (uint32_t)sizeof(T);
#pragma unroll
                        for (int k = 0; k < K; ++k)
                            val[q][k] = cols.at((uint32_t)ix[k] * (uint32_t)sizeof(T), soff);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const T c = lane_read(cv, l0 - l64 + q);  // (zero past r)
#pragma unroll
                        for (int k = 0; k < K; ++k) a[k] -= val[q][k] * c;
                    }
                }
            }
        };
        // the wave totals of a . (column l0 + q of F), q < 8, l0 + q <= r,
        // column r being a itself
        auto products = [&](const T (&a)[K], const T* FL, const T* FG, int fld, const int (&ix)[K],
                            int l0, int r) -> double {
            double g[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) g[q] = 0.0;
            if (l0 + 8 <= nl) {
                const T* f = FL + l0 * P + tid;
#pragma unroll
                for (int q = 0; q < 8; ++q)
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        g[q] += (double)a[k] * (double)f[q * P + k * NT];
            } else {
                const BufView<T> cols(FG + (int64_t)l0 * fld);
                T val[8][K];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int l = l0 + q < r ? q : (r > l0 ? r - 1 - l0 : 0);
                    const uint32_t soff = (uint32_t)(l * fld) * (uint32_t)sizeof(T);
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        val[q][k] = cols.at((uint32_t)ix[k] * (uint32_t)sizeof(T), soff);
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const T f = l0 + q < r ? val[q][k] : (l0 + q == r ? a[k] : (T)0);
                        g[q] += (double)a[k] * (double)f;
                    }
            }
            return wave_total8(g, lane);
        };

        int r = 0, ncols_used = 0, nfailed = 0, steps = 0;
        for (;;) {
            if (r >= target) {
                if (r >= R) break;
                if (one_shot) {
                    one_shot = false;
                    if (last_p <= tol2 * S2) break;
                }
                if (cap_only) {
                    // storage for the target only: continue in overflow
                    // storage for R columns if the reserve has room
                    const long long off = uniform_i64(
                        ovf.used ? aca_overflow_move<T, NT>(ovf, m, nc, R, r, Upool + uo,
                                                            Vpool + vo, Upool, Vpool, ubase, vbase,
                                                            &sh.slot)
                                 : -1);
                    if (off < 0) {
                        refused = true;
                        break;
                    }
                    uo = ovf.u0 + off - ubase;
                    vo = ovf.v0 + off - vbase;
                    if (tid == 0) ovf.moved[b] = off;
                }
                target = R;
            }
            T* const U = Upool + uo;
            T* const V = Vpool + vo;
            // (several waves: the barrier that ended the last step orders its
            // stores; one wave needs it only to read columns back)
            if (NW == 1 && r > nl) __syncthreads();
            // ---- the residual column j ----
            ++ncols_used;
            ++steps;
            {
                const int kj = K == 1 ? 0 : j / NT;
                if (tid == j - kj * NT) cused |= 1u << kj;
            }
            T a[K];
            phi_rows<T, K>(Kf, x, p, a);
            T cm = (T)0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                a[k] = rok[k] ? a[k] : (T)0;
                const T aa = a[k] < (T)0 ? -a[k] : a[k];
                cm = aa > cm ? aa : cm;
            }
            update(a, UL, U, m, ir, VL, V, nc, j, r);
            // ---- the row pivot ----
            T best[K], top = (T)-1, piv = (T)0;
            int kp = 0, lp = 0, ip = INT_MAX;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const T aa = a[k] < (T)0 ? -a[k] : a[k];
                best[k] = rok[k] && !((rused >> k) & 1u) && aa > (T)-1 ? aa : (T)-1;
            }
            cm = lane_read(wave_max_t(cm), 0);
            if (wave_pivot(best, top, kp, lp)) {
                ip = kp * NT + w * kWave + lp;
                piv = lane_read(a[0], lp);
#pragma unroll
                for (int k = 1; k < K; ++k) {
                    const T t = lane_read(a[k], lp);
                    piv = kp == k ? t : piv;
                }
                point(x, kp, lp);
            }
            if constexpr (NW > 1) {
                if (lane == 0) {
                    sh.best[0][w] = top;
                    sh.idx[0][w] = ip;
                    sh.val[w] = piv;
                    sh.cmax[w] = cm;
#pragma unroll
                    for (int c = 0; c < 3; ++c) sh.pt[0][w][c] = p[c];
                }
                __syncthreads();
                Arg<T> am{sh.best[0][0], sh.idx[0][0], (T)0};
                cm = sh.cmax[0];
                int wq = 0;
#pragma unroll
                for (int q = 1; q < NW; ++q) {
                    const Arg<T> other{sh.best[0][q], sh.idx[0][q], (T)0};
                    wq = other.best > am.best || (other.best == am.best && other.idx < am.idx) ? q
                                                                                               : wq;
                    arg_combine(am, other);
                    cm = sh.cmax[q] > cm ? sh.cmax[q] : cm;
                }
                top = am.best;
                ip = __builtin_amdgcn_readfirstlane(am.idx);
                piv = sh.val[wq];
#pragma unroll
                for (int c = 0; c < 3; ++c) p[c] = sh.pt[0][wq][c];
            }
            if (ip == INT_MAX || (double)top <= (double)eps0 * (double)cm) {
                // no usable pivot in this column: try the lowest unused column
                ++nfailed;
                if (ncols_used >= nc || nfailed >= kmax) break;
                int cand = INT_MAX;
#pragma unroll
                for (int k = K - 1; k >= 0; --k) {
                    const unsigned long long h = __ballot(cok[k] && !((cused >> k) & 1u));
                    cand = h ? k * NT + w * kWave + __builtin_ctzll(h) : cand;
                }
                if constexpr (NW > 1) {
                    if (lane == 0) sh.idx[2][w] = cand;
                    __syncthreads();
#pragma unroll
                    for (int q = 0; q < NW; ++q)
                        cand = sh.idx[2][q] < cand ? sh.idx[2][q] : cand;
                    __syncthreads();  // (read before a later failure writes them)
                }
                if (cand == INT_MAX) break;
                j = __builtin_amdgcn_readfirstlane(cand);
                load_pt(soa, n, d, (int64_t)clo + j, p);
                continue;
            }
            // ---- u_r = column / pivot ----
#pragma unroll
            for (int k = 0; k < K; ++k) {
                a[k] = a[k] / piv;
                if (rok[k]) U[(int64_t)r * m + ir[k]] = a[k];
                a[k] = rok[k] ? a[k] : (T)0;
                if (r < nl) UL[r * P + k * NT + tid] = a[k];
            }
            {
                const int kq = K == 1 ? 0 : ip / NT;
                if (tid == ip - kq * NT) rused |= 1u << kq;
            }
            // ---- v_r = the residual row ----
            T v[K];
            phi_rows<T, K>(Kf, y, p, v);
            update(v, VL, V, nc, ic, UL, U, m, ip, r);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (cok[k]) V[(int64_t)r * nc + ic[k]] = v[k];
                v[k] = cok[k] ? v[k] : (T)0;
                if (r < nl) VL[r * P + k * NT + tid] = v[k];
                const T aa = v[k] < (T)0 ? -v[k] : v[k];
                best[k] = cok[k] && !((cused >> k) & 1u) && aa > (T)-1 ? aa : (T)-1;
            }
            // ---- the products of term r with terms l <= r, FP64 ----
            double ds = 0.0;
            if (!fixed) {
                const int c8 = wave_col8(lane);
                for (int l0 = 0; l0 <= r; l0 += 8) {
                    const double su = products(a, UL, U, m, ir, l0, r);
                    const double sv = products(v, VL, V, nc, ic, l0, r);
                    if constexpr (NW == 1) {
                        const int l = l0 + c8;
                        const double g = su * sv;
                        ds += l < r ? 2.0 * g : (l == r ? g : 0.0);
                        if (r < l0 + 8) last_p = lane_read(g, wave_lane8(r - l0));
                    } else if ((lane & 7) == 0) {
                        sh.pu[w][l0 + c8] = su;
                        sh.pv[w][l0 + c8] = sv;
                    }
                }
            }
            // ---- the next column pivot; the norm recursion ----
            int jn = INT_MAX;
            int kn = 0, ln = 0;
            top = (T)-1;
            if (wave_pivot(best, top, kn, ln)) {
                jn = kn * NT + w * kWave + ln;
                point(y, kn, ln);
            }
            if constexpr (NW > 1) {
                if (lane == 0) {
                    sh.best[1][w] = top;
                    sh.idx[1][w] = jn;
#pragma unroll
                    for (int c = 0; c < 3; ++c) sh.pt[1][w][c] = p[c];
                }
                __syncthreads();
                Arg<T> cmx{sh.best[1][0], sh.idx[1][0], (T)0};
                int wq = 0;
#pragma unroll
                for (int q = 1; q < NW; ++q) {
                    const Arg<T> other{sh.best[1][q], sh.idx[1][q], (T)0};
                    wq = other.best > cmx.best || (other.best == cmx.best && other.idx < cmx.idx)
                             ? q
                             : wq;
                    arg_combine(cmx, other);
                }
                jn = __builtin_amdgcn_readfirstlane(cmx.idx);
#pragma unroll
                for (int c = 0; c < 3; ++c) p[c] = sh.pt[1][wq][c];
                if (!fixed) {
                    // lane l (and l + 64) sums the waves' products of column l
                    double g = 0.0;
                    for (int l = lane; l <= r; l += kWave) {
                        double su = sh.pu[0][l], sv = sh.pv[0][l];
#pragma unroll
                        for (int q = 1; q < NW; ++q) {
                            su += sh.pu[q][l];
                            sv += sh.pv[q][l];
                        }
                        g = su * sv;
                        ds += l < r ? 2.0 * g : g;
                    }
                    last_p = lane_read(g, r & 63);
                    S2 += wave_total(ds);
                }
            } else if (!fixed) {
                S2 += lane_read(wave_cols_total(ds), 0);
            }
            ++r;
            // ---- the stopping test, squared ----
            if (!fixed && !one_shot && last_p <= tol2 * S2) break;
            if (jn == INT_MAX) break;
            j = jn;
        }
        if (tid == 0) {
            rank_out[b] = refused ? -1 : r;
            if (steps_out) steps_out[b] = steps;
        }
        __syncthreads();
    }
}

// arguments of a class's launch from its first entry of the order
template <typename T, int NT, int KR>
void launch_class(const AcaArgs& a, int64_t o0, int64_t nb, int lds_words, hipStream_t st) {
    KernelEval<T> K(a.kern);
    constexpr int64_t kGrid = 0x7fffffff;  // a workgroup per block
    for (; nb > 0; nb -= kGrid, o0 += kGrid)
        hipLaunchKernelGGL((aca_kernel<T, NT, KR>), dim3((unsigned)std::min(nb, kGrid)), dim3(NT),
                           (size_t)lds_words * sizeof(uint32_t), st, (const T*)a.soa, a.soa64,
                           a.n, a.d, K, a.blocks, a.order + o0, std::min(nb, kGrid), a.uoff,
                           a.voff, a.ubase, a.vbase, a.kmax, a.eps, a.aca_eta, (T)a.eps0, a.fixed,
                           a.rtarget, a.one_shot, a.cap_only,
                           Overflow{a.ovf_used, a.ovf_cap, a.ovf_u0, a.ovf_v0, a.ovf_moved},
                           lds_words, (T*)a.U, (T*)a.V, a.rank, a.steps);
}

template <typename T, int NW, int K, int NL>
void launch_lds_class(const AcaArgs& a, int64_t o0, int64_t nb, hipStream_t st) {
    static_assert(NL % 8 == 0 && aca_lds_bytes<T, NW * kWave * K>(NL) + sizeof(LdsShared<T, NW>) <=
                                     kLdsBytes,
                  "whole batches of eight columns, within a compute unit's LDS");
    constexpr int nl = NL;
    if (nb <= 0) return;
    const unsigned grid = (unsigned)(nb < 0x7fffffff ? nb : 0x7fffffff);
    KernelEval<T> Kf(a.kern);
    hipLaunchKernelGGL((aca_lds_kernel<T, NW, K>), dim3(grid), dim3(NW * kWave),
                       (aca_lds_bytes<T, NW * kWave * K>(nl)), st,
                       (const T*)a.soa, a.soa64, a.n, a.d, Kf, a.blocks, a.order + o0, nb, a.uoff,
                       a.voff, a.ubase, a.vbase, a.kmax, a.eps, a.aca_eta, (T)a.eps0, a.fixed,
                       a.rtarget, a.one_shot, a.cap_only,
                       Overflow{a.ovf_used, a.ovf_cap, a.ovf_u0, a.ovf_v0, a.ovf_moved}, nl,
                       (T*)a.U, (T*)a.V, a.rank, a.steps);
}

// the size class of a block whose larger side has s points (see kAcaClassRows)
__device__ __forceinline__ int size_class(int s) {
    int c = 0;
#pragma unroll
    for (int q = 1; q < kAcaClasses; ++q) c = s <= kAcaClassRows[q] ? q : c;
    return c;
}

// sort keys of the ACA's classes: 0 for the blocks of the many-workgroup path
// (below level lvl0, a prefix of the level-sorted list), 1 + size class else
__global__ void class_keys_kernel(const int4* __restrict__ blocks,
                                  const int32_t* __restrict__ level, int64_t nb, int lvl0,
                                  uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b >= nb) return;
    const int4 bl = blocks[b];
    const int m = bl.y - bl.x, nc = bl.w - bl.z;
    keys[b] = level[b] < lvl0 ? 0ull : (uint64_t)(1 + size_class(m > nc ? m : nc));
    vals[b] = (uint32_t)b;
}

// out[c] = the first entry of the sorted keys that is > c (c = 0 ..
// kAcaClasses): the first entry of size class c, and at the end their number
__global__ void class_bounds_kernel(const uint64_t* __restrict__ keys, int64_t nb,
                                    int64_t* __restrict__ out) {
    const int c = threadIdx.x;
    if (blockIdx.x != 0 || c > kAcaClasses) return;
    int64_t lo = 0, hi = nb;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (keys[mid] <= (uint64_t)c)
            lo = mid + 1;
        else
            hi = mid;
    }
    out[c] = lo;
}

// blocks that continued in overflow storage: their storage offsets move there
__global__ void apply_moved_kernel(const int64_t* __restrict__ moved, int64_t nb, int64_t u0,
                                   int64_t v0, int64_t* __restrict__ uoff,
                                   int64_t* __restrict__ voff) {
    const int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (b < nb && moved[b] >= 0) {
        uoff[b] = u0 + moved[b];
        voff[b] = v0 + moved[b];
    }
}

}  // namespace

hipError_t launch_class_keys(const int4* blocks, const int32_t* level, int64_t nb, int lvl0,
                             uint64_t* keys, uint32_t* vals, hipStream_t st) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(class_keys_kernel, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st,
                       blocks, level, nb, lvl0, keys, vals);
    return hipGetLastError();
}

hipError_t launch_class_bounds(const uint64_t* keys, int64_t nb, int64_t* out, hipStream_t st) {
    hipLaunchKernelGGL(class_bounds_kernel, dim3(1), dim3(64), 0, st, keys, nb, out);
    return hipGetLastError();
}

hipError_t launch_apply_moved(const int64_t* moved, int64_t nb, int64_t u0, int64_t v0,
                              int64_t* uoff, int64_t* voff, hipStream_t st) {
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(apply_moved_kernel, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st,
                       moved, nb, u0, v0, uoff, voff);
    return hipGetLastError();
}

// The size classes (kAcaClassRows), each in its own launch over its range of
// the order.  Which kernel and shape, with the class's time alone on the
// N = 2^20 2-d FP32 / N = 100003 3-d FP32 / N = 2^19 2-d FP64 builds:
//   above 4096 points: 1024 threads (FP64 512): 18.0 ms against 25.3 ms with
//     512 threads, the largest blocks' steps being the class's tail (FP64 at
//     1024 threads and two rows a thread: 16.5 ms, as with 512 and four);
//   to 4096: 512 threads 3.9 ms (1024 threads 6.8);
//   to 2048: 256 threads 4.2 / 2.7 / 3.8 ms (columns in LDS at eight waves
//     4.6 / 2.1 ms, one workgroup a compute unit);
//   to 1024: columns in LDS, four waves of four rows 3.0 / 3.7 ms against 4.2 /
//     3.1; FP64 256 threads 4.6 (LDS 5.2);
//   to 512: two waves of four rows 3.6 / 6.6 (eight waves of one row 12.2 /
//     15.5); FP64 four waves of two 2.9 (two of four 3.5);
//   to 256: one wave of four rows 2.05 / 3.7 (four waves of one 4.5 / 6.3);
//     FP64 two waves of two 3.4 (one of four 3.7);
//   to 128: one wave of two rows 5.6 (two waves of one 8.5); to 64: one wave.
// Eight columns in LDS and not sixteen: the LDS of a block bounds the waves in
// flight (to 512 points 3.6 against 5.5 ms, to 256 2.1 against 4.0).
// The first class reserves the LDS mask words of the list's largest block.  (Blocks
// [0, nsplit) take the multi-workgroup path of k_aca_split.hip.)
// aca_classes_begin queues the classes on the streams aux[0..2] (or on st
// where null) after the work already queued on st; aca_classes_join makes
// st wait for them.  Running the classes concurrently keeps the few large
// blocks of the upper levels from holding back the many small ones.
template <typename T>
static void launch_classes(const AcaArgs& a, hipStream_t s0, hipStream_t s1, hipStream_t s2) {
    const int64_t* c = a.cls;
    constexpr bool D = sizeof(T) == 8;
    launch_class<T, D ? 512 : 1024, 4>(a, c[0], c[1] - c[0], a.big_words, s0);
    launch_class<T, 512, 4>(a, c[1], c[2] - c[1], 2 * 4096 / 32, s0);
    launch_class<T, 256, 4>(a, c[2], c[3] - c[2], 2 * 2048 / 32, s1);
    if constexpr (D)
        launch_class<T, 256, 4>(a, c[3], c[4] - c[3], 2 * 1024 / 32, s1);
    else
        launch_lds_class<T, 4, 4, 8>(a, c[3], c[4] - c[3], s1);
    launch_lds_class<T, D ? 4 : 2, D ? 2 : 4, 8>(a, c[4], c[5] - c[4], s2);
    launch_lds_class<T, D ? 2 : 1, D ? 2 : 4, 8>(a, c[5], c[6] - c[5], s1);
    launch_lds_class<T, 1, 2, 8>(a, c[6], c[7] - c[6], s2);
    launch_lds_class<T, 1, 1, 8>(a, c[7], c[8] - c[7], s2);
}

hipError_t aca_classes_begin(const AcaArgs& a, int f64, hipStream_t st, const hipStream_t* aux) {
    hipStream_t s0 = aux && aux[0] ? aux[0] : st;
    hipStream_t s1 = aux && aux[1] ? aux[1] : s0;
    hipStream_t s2 = aux && aux[2] ? aux[2] : s1;
    hipError_t e = hipSuccess;
    if (aux) {
        hipEvent_t go = nullptr;
        e = hipEventCreateWithFlags(&go, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventRecord(go, st);
        for (int k = 0; k < 3 && e == hipSuccess; ++k)
            if (aux[k]) e = hipStreamWaitEvent(aux[k], go, 0);
        if (go) (void)hipEventDestroy(go);
    }
    if (e != hipSuccess) return e;
    if (f64)
        launch_classes<double>(a, s0, s1, s2);
    else
        launch_classes<float>(a, s0, s1, s2);
    return hipGetLastError();
}

hipError_t aca_classes_join(hipStream_t st, const hipStream_t* aux) {
    if (!aux) return hipSuccess;
    hipError_t e = hipSuccess;
    for (int k = 0; k < 3 && e == hipSuccess; ++k) {
        if (!aux[k]) continue;
        hipEvent_t done = nullptr;
        e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventRecord(done, aux[k]);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, done, 0);
        if (done) (void)hipEventDestroy(done);
    }
    return e;
}

namespace {
// out[0] += steps_b m_b + rank_b n_b (kernel evaluations: a column per step,
// a row per accepted step), out[1] += 2 rank_b (rank_b - 1) (m_b + n_b)
// (multiply-adds of the residual updates and of the norm recursion's inner
// products); integer atomics, order-free
__global__ void aca_work_kernel(const int4* __restrict__ blocks, const int32_t* __restrict__ rank,
                                const int32_t* __restrict__ steps, int64_t nb,
                                unsigned long long* __restrict__ out) {
    unsigned long long ev = 0, fl = 0;
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < nb;
         b += (int64_t)gridDim.x * blockDim.x) {
        const int4 bl = blocks[b];
        const unsigned long long m = bl.y - bl.x, nc = bl.w - bl.z;
        const unsigned long long r = rank[b] > 0 ? rank[b] : 0, s = steps[b] > 0 ? steps[b] : 0;
        ev += s * m + r * nc;
        fl += r > 0 ? 2ull * r * (r - 1) * (m + nc) : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        ev += __shfl_xor(ev, o, 64);
        fl += __shfl_xor(fl, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&out[0], ev);
        atomicAdd(&out[1], fl);
    }
}
}  // namespace

hipError_t launch_aca_work(const int4* blocks, const int32_t* rank, const int32_t* steps,
                           int64_t nb, unsigned long long* out, hipStream_t st) {
    hipError_t e = hipMemsetAsync(out, 0, 2 * sizeof(unsigned long long), st);
    if (e != hipSuccess || nb == 0) return e;
    const unsigned grid = (unsigned)std::min<int64_t>((nb + 255) / 256, kStatBlocks);
    hipLaunchKernelGGL(aca_work_kernel, dim3(grid), dim3(256), 0, st, blocks, rank, steps, nb, out);
    return hipGetLastError();
}


}  // namespace hmx
