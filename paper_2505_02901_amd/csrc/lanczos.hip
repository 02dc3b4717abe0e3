// Lanczos iteration on the GPU (eigval0 / eigvals_lanczos, Sec. 3.7.1; the
// recurrence of Lanczos 1950):
//   w = H v_j;  alpha_j = Re<v_j, w>;  w -= alpha_j v_j + beta_j v_{j-1};
//   [optional: classical Gram-Schmidt against all v_i, twice];
//   beta_{j+1} = |w|;  v_{j+1} = w / beta_{j+1}.
// Vectors are stored in FP64 or FP32 (complex if the block is); every dot
// product, norm, coefficient and the three-term update are computed in FP64
// and rounded once on store.  Reductions use fixed-order block partials, so
// the scalars are bitwise reproducible.  The scalars live on the device
// (no host round trip per step); the host reads them back to test
// convergence and solves the tridiagonal problem with the implicit QL
// method (Bowdler, Martin, Reinsch and Wilkinson, 1968).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>
#include <vector>

#include "xdg_internal.hpp"

namespace xdg {

namespace {
constexpr int RB = 256;    // threads per block of the vector kernels
constexpr int MAXC = 16;   // scalar columns per row (nvec <= 8, complex)

// Sum over threads that share a column (t = column mod cols, cols a power of
// two dividing RB); sh[0 .. cols) holds the block totals afterwards.
__device__ inline void block_col_reduce(double *sh, int cols) {
    for (int s = RB / 2; s >= cols; s >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    }
    __syncthreads();
}

// The vector operations of one workgroup: number lb of the nb that share the
// vector's n scalars.  They are used by kernels on one vector block (lb =
// blockIdx.x) and by kernels on many vector blocks at once (below), and give
// the same bits in both.
//
// dot_part: partials[lb][c] = sum over the workgroup's scalars of column c of
// a*b.  The flat scalar index q has column q % cols because the grid stride
// is a multiple of cols.
template <class T>
__device__ __forceinline__ void dot_part(const T *a, const T *b, uint64_t n, int cols,
                                         double *partials, uint32_t lb, uint32_t nb, double *sh) {
    double acc = 0.0;
    const uint64_t stride = (uint64_t)nb * RB;
    for (uint64_t q = (uint64_t)lb * RB + threadIdx.x; q < n; q += stride)
        acc += (double)a[q] * (double)b[q];
    sh[threadIdx.x] = acc;
    block_col_reduce(sh, cols);
    if ((int)threadIdx.x < cols) partials[(size_t)lb * cols + threadIdx.x] = sh[threadIdx.x];
}

// Fixed-order total of the partials, pairs of columns combined for complex
// vectors (Re<a,b> = sum re*re + im*im).  mode 0: out = s; 1: out = sqrt(s).
// hist (may be null) receives the values too; they stay in sh[v * C].
__device__ __forceinline__ void total_part(const double *partials, int n_blocks, int cols, int C,
                                           int mode, double *out, double *hist, double *sh) {
    const int c = threadIdx.x % cols;
    double acc = 0.0;
    for (int blk = threadIdx.x / cols; blk < n_blocks; blk += RB / cols)
        acc += partials[(size_t)blk * cols + c];
    sh[threadIdx.x] = acc;
    block_col_reduce(sh, cols);
    if ((int)threadIdx.x < cols / C) {
        const int v = threadIdx.x;
        double s = sh[v * C];
        if (C == 2) s += sh[v * C + 1];
        const double r = mode == 1 ? sqrt(s) : s;
        if (out) out[v] = r;
        if (hist) hist[v] = r;
        sh[v * C] = r;
    }
}

// one scalar of w - alpha v - beta vprev in FP64, rounded once
template <class T>
__device__ __forceinline__ T updated(T w, T v, T vprev, bool has_prev, double a, double b) {
    double x = (double)w - a * (double)v;
    if (has_prev) x -= b * (double)vprev;
    return (T)x;
}
// one scalar divided by beta (zero where beta vanished: invariant subspace)
template <class T>
__device__ __forceinline__ T scaled(T x, double bt) {
    return bt > 0.0 ? (T)((double)x / bt) : T(0);
}

// w = w - alpha v - beta vprev (FP64, one rounding), partial |w|^2
template <class T>
__device__ __forceinline__ void update_part(T *w, const T *v, const T *vprev, uint64_t n, int cols,
                                            int C, const double *alpha, const double *beta,
                                            double *partials, uint32_t lb, uint32_t nb,
                                            double *sh) {
    double acc = 0.0;
    const uint64_t stride = (uint64_t)nb * RB;
    // cols divides RB, so every scalar of this thread is in column threadIdx.x % cols
    const int vec = (int)(threadIdx.x % cols) / C;
    const double a = alpha[vec], b = vprev ? beta[vec] : 0.0;
    for (uint64_t q = (uint64_t)lb * RB + threadIdx.x; q < n; q += stride) {
        const T r = updated<T>(w[q], v[q], vprev ? vprev[q] : T(0), vprev != nullptr, a, b);
        w[q] = r;
        acc += (double)r * (double)r;
    }
    sh[threadIdx.x] = acc;
    block_col_reduce(sh, cols);
    if ((int)threadIdx.x < cols) partials[(size_t)lb * cols + threadIdx.x] = sh[threadIdx.x];
}

// dst = src / beta
template <class T>
__device__ __forceinline__ void scale_part(const T *src, T *dst, uint64_t n, int cols, int C,
                                           const double *beta, uint32_t lb, uint32_t nb) {
    const uint64_t stride = (uint64_t)nb * RB;
    // cols divides RB, so every scalar of this thread is in column threadIdx.x % cols
    const double bt = beta[(int)(threadIdx.x % cols) / C];
    for (uint64_t q = (uint64_t)lb * RB + threadIdx.x; q < n; q += stride)
        dst[q] = scaled<T>(src[q], bt);
}

// One column (a single real vector): four consecutive scalars per thread
// through one vector load each, the same arithmetic per scalar as above.
// Scalars past the last full group of four go to workgroup 0.
template <class T>
using Vec4 = T __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ void dot1_part(const T *a, const T *b, uint64_t n, double *partials,
                                          uint32_t lb, uint32_t nb, double *sh) {
    double acc = 0.0;
    const uint64_t n4 = n / 4, stride = (uint64_t)nb * RB;
    for (uint64_t q = (uint64_t)lb * RB + threadIdx.x; q < n4; q += stride) {
        const Vec4<T> x = reinterpret_cast<const Vec4<T> *>(a)[q];
        const Vec4<T> y = reinterpret_cast<const Vec4<T> *>(b)[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += (double)x[e] * (double)y[e];
    }
    if (lb == 0)
        for (uint64_t q = 4 * n4 + threadIdx.x; q < n; q += RB) acc += (double)a[q] * (double)b[q];
    sh[threadIdx.x] = acc;
    block_col_reduce(sh, 1);
    if (threadIdx.x == 0) partials[lb] = sh[0];
}

template <class T>
__device__ __forceinline__ void update1_part(T *w, const T *v, const T *vprev, uint64_t n,
                                             const double *alpha, const double *beta,
                                             double *partials, uint32_t lb, uint32_t nb,
                                             double *sh) {
    double acc = 0.0;
    const double a = alpha[0], b = vprev ? beta[0] : 0.0;
    const uint64_t n4 = n / 4, stride = (uint64_t)nb * RB;
    for (uint64_t q = (uint64_t)lb * RB + threadIdx.x; q < n4; q += stride) {
        Vec4<T> x = reinterpret_cast<const Vec4<T> *>(w)[q];
        const Vec4<T> y = reinterpret_cast<const Vec4<T> *>(v)[q];
        Vec4<T> z = {};
        if (vprev) z = reinterpret_cast<const Vec4<T> *>(vprev)[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const T r = updated<T>(x[e], y[e], z[e], vprev != nullptr, a, b);
            x[e] = r;
            acc += (double)r * (double)r;
        }
        reinterpret_cast<Vec4<T> *>(w)[q] = x;
    }
    if (lb == 0)
        for (uint64_t q = 4 * n4 + threadIdx.x; q < n; q += RB) {
            const T r = updated<T>(w[q], v[q], vprev ? vprev[q] : T(0), vprev != nullptr, a, b);
            w[q] = r;
            acc += (double)r * (double)r;
        }
    sh[threadIdx.x] = acc;
    block_col_reduce(sh, 1);
    if (threadIdx.x == 0) partials[lb] = sh[0];
}

template <class T>
__device__ __forceinline__ void scale1_part(const T *src, T *dst, uint64_t n, const double *beta,
                                            uint32_t lb, uint32_t nb) {
    const double bt = beta[0];
    const uint64_t n4 = n / 4, stride = (uint64_t)nb * RB;
    for (uint64_t q = (uint64_t)lb * RB + threadIdx.x; q < n4; q += stride) {
        Vec4<T> x = reinterpret_cast<const Vec4<T> *>(src)[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = scaled<T>(x[e], bt);
        reinterpret_cast<Vec4<T> *>(dst)[q] = x;
    }
    if (lb == 0)
        for (uint64_t q = 4 * n4 + threadIdx.x; q < n; q += RB)
            dst[q] = scaled<T>(src[q], bt);
}

// ---- one vector block ----
template <class T>
__global__ __launch_bounds__(RB) void k_dot(const T *a, const T *b, uint64_t n, int cols,
                                            double *partials) {
    __shared__ double sh[RB];
    dot_part(a, b, n, cols, partials, blockIdx.x, gridDim.x, sh);
}

__global__ __launch_bounds__(RB) void k_finalize(const double *partials, int n_blocks, int cols,
                                                 int C, int mode, double *out, double *hist) {
    __shared__ double sh[RB];
    total_part(partials, n_blocks, cols, C, mode, out, hist, sh);
}

template <class T>
__global__ __launch_bounds__(RB) void k_update(T *w, const T *v, const T *vprev, uint64_t n,
                                               int cols, int C, const double *alpha,
                                               const double *beta, double *partials) {
    __shared__ double sh[RB];
    update_part(w, v, vprev, n, cols, C, alpha, beta, partials, blockIdx.x, gridDim.x, sh);
}

template <class T>
__global__ __launch_bounds__(RB) void k_scale(const T *src, T *dst, uint64_t n, int cols, int C,
                                              const double *beta) {
    scale_part(src, dst, n, cols, C, beta, blockIdx.x, gridDim.x);
}

template <class T>
__global__ __launch_bounds__(RB) void k_dot1(const T *a, const T *b, uint64_t n,
                                             double *partials) {
    __shared__ double sh[RB];
    dot1_part(a, b, n, partials, blockIdx.x, gridDim.x, sh);
}

template <class T>
__global__ __launch_bounds__(RB) void k_update1(T *w, const T *v, const T *vprev, uint64_t n,
                                                const double *alpha, const double *beta,
                                                double *partials) {
    __shared__ double sh[RB];
    update1_part(w, v, vprev, n, alpha, beta, partials, blockIdx.x, gridDim.x, sh);
}

template <class T>
__global__ __launch_bounds__(RB) void k_scale1(const T *src, T *dst, uint64_t n,
                                               const double *beta) {
    scale1_part(src, dst, n, beta, blockIdx.x, gridDim.x);
}

// Short vectors (at most FUSE_WGS workgroups): the total of the previous
// kernel's partials is taken by every workgroup itself, in the order of
// k_finalize, which saves a launch between two kernels of 2-3 us.  Longer
// ones would read the partials of up to 2048 workgroups 2048 times.
constexpr int FUSE_WGS = 256;

template <class T, bool ONE>
__global__ __launch_bounds__(RB) void k_total_update(T *w, const T *v, const T *vprev, uint64_t n,
                                                     int cols, int C, const double *dots,
                                                     double *alpha, double *host_alpha,
                                                     const double *beta, double *partials) {
    __shared__ double sh[RB];
    const bool first = blockIdx.x == 0;
    total_part(dots, gridDim.x, cols, C, 0, first ? alpha : nullptr, first ? host_alpha : nullptr,
               sh);
    __syncthreads();
    const double a = sh[0];   // one vector
    __syncthreads();
    if constexpr (ONE)
        update1_part(w, v, vprev, n, &a, beta, partials, blockIdx.x, gridDim.x, sh);
    else
        update_part(w, v, vprev, n, cols, C, &a, beta, partials, blockIdx.x, gridDim.x, sh);
}

template <class T, bool ONE>
__global__ __launch_bounds__(RB) void k_total_scale(const T *src, T *dst, uint64_t n, int cols,
                                                    int C, const double *norms, double *beta,
                                                    double *host_beta) {
    __shared__ double sh[RB];
    const bool first = blockIdx.x == 0;
    total_part(norms, gridDim.x, cols, C, 1, first ? beta : nullptr, first ? host_beta : nullptr,
               sh);
    __syncthreads();
    const double b = sh[0];
    if constexpr (ONE)
        scale1_part(src, dst, n, &b, blockIdx.x, gridDim.x);
    else
        scale_part(src, dst, n, cols, C, &b, blockIdx.x, gridDim.x);
}

// A step of the second pass on known alpha and beta: next = (w - alpha v -
// beta_prev vprev) / beta with the two roundings of the first pass, and
// acc += c next in FP64, in one pass over the vectors (before: update, scale
// and the accumulation apart, nine vector passes instead of six).
template <class T>
__global__ __launch_bounds__(RB) void k_ritz_step(const T *w, const T *v, const T *vprev, T *next,
                                                  double *acc, uint64_t n, const double *alpha,
                                                  const double *beta_prev, const double *beta,
                                                  double c) {
    const uint64_t stride = (uint64_t)gridDim.x * RB;
    const double a = *alpha, b = vprev ? *beta_prev : 0.0, bt = *beta;
    for (uint64_t q = (uint64_t)blockIdx.x * RB + threadIdx.x; q < n; q += stride) {
        const T r = scaled<T>(
            updated<T>(w[q], v[q], vprev ? vprev[q] : T(0), vprev != nullptr, a, b), bt);
        next[q] = r;
        acc[q] = __builtin_fma(c, (double)r, acc[q]);
    }
}

// ---- many vector blocks at once ----
// One launch for an operation on all blocks of a batch.  With a launch per
// block a step of 20 small blocks was 123 graph nodes of 2-4 us (ring N = 20,
// all momenta, four vectors each: 540 us per step); the workgroups of all
// blocks are numbered through, each block keeping the workgroups, and so the
// order of every sum, that it has alone.
struct ManyBlock {
    char *buf;             // vector slots, `slot` bytes apart
    uint64_t slot, n;      // n: scalars of a vector
    double *partials;      // [workgroups][cols]
    double *s;             // its scalars (the same places in every block)
    uint32_t first, wgs;   // its workgroups: [first, first + wgs)
};
struct ManyArgs {
    const ManyBlock *blk;
    int n_blk, cols, C;
};

__device__ __forceinline__ ManyBlock many_block(const ManyArgs &A, uint32_t wg) {
    int lo = 0, hi = A.n_blk - 1;   // last block with first <= wg
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (A.blk[mid].first <= wg) lo = mid; else hi = mid - 1;
    }
    return A.blk[lo];
}
template <class T>
__device__ __forceinline__ T *slot_of(const ManyBlock &b, int slot) {
    return reinterpret_cast<T *>(b.buf + b.slot * (uint64_t)slot);
}

// partials of slot va . slot vb
template <class T, bool ONE>
__global__ __launch_bounds__(RB) void k_many_dot(ManyArgs A, int va, int vb) {
    __shared__ double sh[RB];
    const ManyBlock b = many_block(A, blockIdx.x);
    const uint32_t lb = blockIdx.x - b.first;
    if constexpr (ONE)
        dot1_part(slot_of<T>(b, va), slot_of<T>(b, vb), b.n, b.partials, lb, b.wgs, sh);
    else
        dot_part(slot_of<T>(b, va), slot_of<T>(b, vb), b.n, A.cols, b.partials, lb, b.wgs, sh);
}

// totals into the scalars at `out` (and the history at `hist` >= 0, row *jdev)
__global__ __launch_bounds__(RB) void k_many_total(ManyArgs A, int mode, int out, int hist,
                                                   const int *jdev) {
    __shared__ double sh[RB];
    const ManyBlock b = A.blk[blockIdx.x];
    total_part(b.partials, (int)b.wgs, A.cols, A.C, mode, b.s + out,
               hist >= 0 ? b.s + hist + (size_t)(*jdev) * (A.cols / A.C) : nullptr, sh);
}

// slot w -= alpha slot v + beta slot vp (vp < 0: none), partial |w|^2
template <class T, bool ONE>
__global__ __launch_bounds__(RB) void k_many_update(ManyArgs A, int w, int v, int vp, int alpha,
                                                    int beta) {
    __shared__ double sh[RB];
    const ManyBlock b = many_block(A, blockIdx.x);
    const uint32_t lb = blockIdx.x - b.first;
    const T *p = vp < 0 ? nullptr : slot_of<T>(b, vp);
    if constexpr (ONE)
        update1_part(slot_of<T>(b, w), slot_of<T>(b, v), p, b.n, b.s + alpha, b.s + beta,
                     b.partials, lb, b.wgs, sh);
    else
        update_part(slot_of<T>(b, w), slot_of<T>(b, v), p, b.n, A.cols, A.C, b.s + alpha,
                    b.s + beta, b.partials, lb, b.wgs, sh);
}

// slot dst = slot src / beta; the end of a step (keep >= 0): the scalars at
// `beta` are copied to `keep` and the step counter advances (nothing in this
// launch reads either)
template <class T, bool ONE>
__global__ __launch_bounds__(RB) void k_many_scale(ManyArgs A, int src, int dst, int beta,
                                                   int keep, int *jdev) {
    const ManyBlock b = many_block(A, blockIdx.x);
    const uint32_t lb = blockIdx.x - b.first;
    if constexpr (ONE)
        scale1_part(slot_of<T>(b, src), slot_of<T>(b, dst), b.n, b.s + beta, lb, b.wgs);
    else
        scale_part(slot_of<T>(b, src), slot_of<T>(b, dst), b.n, A.cols, A.C, b.s + beta, lb,
                   b.wgs);
    if (keep >= 0 && lb == 0 && (int)threadIdx.x < A.cols / A.C)
        b.s[keep + threadIdx.x] = b.s[beta + threadIdx.x];
    if (jdev && blockIdx.x == 0 && threadIdx.x == 0) *jdev += 1;
}

__global__ void k_set_scalars(int *jdev, double *prev_beta, int nv) {
    for (int v = threadIdx.x; v < nv; v += blockDim.x) prev_beta[v] = 0.0;
    if (threadIdx.x == 0) *jdev = 0;
}

// Reorthogonalisation of one vector against the stored Krylov vectors V_i,
// i < k (classical Gram-Schmidt: the coefficients c_i = <V_i, w> first, then
// w -= sum_i c_i V_i; complex when C = 2, conj(V_i) in the product).  Both
// kernels stream row tiles: each thread owns ru 16-byte chunks of a tile
// (L = 16 / sizeof(T) scalars each, consecutive threads on consecutive
// chunks), so a block covers RB * ru * L scalars and a column is read with
// ru independent 16-byte loads per thread; RG columns are in flight at once.
// Sums are FP64 in a fixed order (bitwise reproducible).
// 16-byte chunks per thread and column: eight scalars per thread for both
// types (FP32 with four chunks held too many registers for enough waves)
template <class T>
constexpr int ru() { return sizeof(T) == 4 ? 2 : 4; }
constexpr int RG = 4;   // columns per step

template <class T> struct Chunk16;
template <> struct Chunk16<float> {
    typedef float type __attribute__((ext_vector_type(4)));
};
template <> struct Chunk16<double> {
    typedef double type __attribute__((ext_vector_type(2)));
};

template <class T>
constexpr int tile_scalars() { return RB * ru<T>() * (16 / (int)sizeof(T)); }

// scalars [q, q + L) of column `col` (zero beyond n): one 16-byte load when
// the chunk is whole, scalar loads at the ragged end
template <class T>
__device__ __forceinline__ void load_chunk(const T *col, uint64_t q, uint64_t n, T *out) {
    constexpr int L = 16 / (int)sizeof(T);
    if (q + L <= n) {
        typedef typename Chunk16<T>::type V16;
        const V16 v = *(const __attribute__((address_space(1))) V16 *)(col + q);
#pragma unroll
        for (int e = 0; e < L; ++e) out[e] = v[e];
    } else {
#pragma unroll
        for (int e = 0; e < L; ++e) out[e] = q + e < n ? col[q + e] : T(0);
    }
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// N values per lane summed over the wave together: each exchange step first
// halves the values a lane keeps (the lanes of one half of the exchange keep
// the lower values, the others the upper ones), then the last value is
// summed over the remaining lane groups.  Lane l returns the wave total of
// value l / (64 / N): N - 1 + 6 - log2(N) exchanges of a double instead of 6 N.
template <int N>
__device__ __forceinline__ double wave_sum_n(double (&v)[N], int lane) {
    static_assert(N == 1 || N == 2 || N == 4 || N == 8, "N in {1, 2, 4, 8}");
    int o = 32;
#pragma unroll
    for (int n = N; n > 1; n >>= 1, o >>= 1) {
        const bool up = (lane & o) != 0;
#pragma unroll
        for (int i = 0; i < n / 2; ++i) {
            const double keep = up ? v[i + n / 2] : v[i];
            const double send = up ? v[i] : v[i + n / 2];
            v[i] = keep + __shfl_xor(send, o, 64);
        }
    }
    double r = v[0];
#pragma unroll
    for (; o >= 1; o >>= 1) r += __shfl_xor(r, o, 64);
    return r;
}

// partials[(i C + c) nb + block] = the block's share of Re / Im <V_i, w>.
// skip (may be null): a device flag; when set the pass does nothing.
template <class T, int C>
__global__ __launch_bounds__(RB) void k_reorth_dots(const T *V, uint64_t ld, int k, const T *w,
                                                    uint64_t nsc, double *partials,
                                                    const int *skip) {
    if (skip && *skip) return;
    constexpr int RU = ru<T>(), L = 16 / (int)sizeof(T), S = RU * L;
    __shared__ double sh[RB / 64][RG * C];
    const int nb = gridDim.x, t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const uint64_t tile0 = (uint64_t)blockIdx.x * tile_scalars<T>();
    T wr[S];
#pragma unroll
    for (int u = 0; u < RU; ++u)
        load_chunk<T>(w, tile0 + ((uint64_t)u * RB + t) * L, nsc, wr + u * L);
    for (int i0 = 0; i0 < k; i0 += RG) {
        T vr[RG][S];
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            const int i = i0 + g < k ? i0 + g : k - 1;   // a repeated column is discarded
#pragma unroll
            for (int u = 0; u < RU; ++u)
                load_chunk<T>(V + (size_t)i * ld, tile0 + ((uint64_t)u * RB + t) * L, nsc,
                              vr[g] + u * L);
        }
        double part[RG * C];   // value g C + c: Re (c = 0) / Im of <V_{i0+g}, w>
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int e = 0; e < S; e += C) {
                if (C == 1) {
                    re = fma((double)vr[g][e], (double)wr[e], re);
                } else {
                    const double a = vr[g][e], b = vr[g][e + 1], x = wr[e], y = wr[e + 1];
                    re = fma(a, x, fma(b, y, re));       // conj(V) w
                    im = fma(a, y, fma(-b, x, im));
                }
            }
            part[g * C] = re;
            if (C == 2) part[g * C + 1] = im;
        }
        {
            constexpr int Q = 64 / (RG * C);   // lanes per value after the exchanges
            const double r = wave_sum_n<RG * C>(part, lane);
            if ((lane & (Q - 1)) == 0) sh[wave][lane / Q] = r;
        }
        __syncthreads();
        if (t < RG * C && i0 + t / C < k) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < RB / 64; ++q) s += sh[q][t];
            partials[((size_t)(i0 + t / C) * C + t % C) * nb + blockIdx.x] = s;
        }
        __syncthreads();
    }
}

// coef[2 i + c] = sum over blocks (fixed order) of the partials; one block
// per (i, c); coef[2 i + 1] = 0 for real vectors
template <int C>
__global__ __launch_bounds__(RB) void k_reorth_finalize(const double *partials, int n_blocks,
                                                        double *coef, const int *skip) {
    if (skip && *skip) return;
    __shared__ double sh[RB];
    const int e = blockIdx.x;   // i C + c
    double s = 0.0;
    for (int b = threadIdx.x; b < n_blocks; b += RB) s += partials[(size_t)e * n_blocks + b];
    sh[threadIdx.x] = s;
    block_col_reduce(sh, 1);
    if (threadIdx.x == 0) {
        const int i = e / C, c = e % C;
        coef[2 * i + c] = sh[0];
        if (C == 1) coef[2 * i + 1] = 0.0;
    }
}

// w -= sum_i c_i V_i, accumulated in FP64 and rounded once on store
template <class T, int C>
__global__ __launch_bounds__(RB) void k_reorth_sub(const T *V, uint64_t ld, int k,
                                                   const double *coef, T *w, uint64_t nsc,
                                                   const int *skip) {
    if (skip && *skip) return;
    constexpr int RU = ru<T>(), L = 16 / (int)sizeof(T), S = RU * L;
    const int t = threadIdx.x;
    const uint64_t tile0 = (uint64_t)blockIdx.x * tile_scalars<T>();
    double acc[S];
    {
        T w0[S];
#pragma unroll
        for (int u = 0; u < RU; ++u)
            load_chunk<T>(w, tile0 + ((uint64_t)u * RB + t) * L, nsc, w0 + u * L);
#pragma unroll
        for (int e = 0; e < S; ++e) acc[e] = (double)w0[e];
    }
    for (int i0 = 0; i0 < k; i0 += RG) {
        T vr[RG][S];
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            const int i = i0 + g < k ? i0 + g : k - 1;
#pragma unroll
            for (int u = 0; u < RU; ++u)
                load_chunk<T>(V + (size_t)i * ld, tile0 + ((uint64_t)u * RB + t) * L, nsc,
                              vr[g] + u * L);
        }
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            if (i0 + g >= k) break;
            const double cr = coef[2 * (i0 + g)], ci = coef[2 * (i0 + g) + 1];
#pragma unroll
            for (int e = 0; e < S; e += C) {
                if (C == 1) {
                    acc[e] = fma(-cr, (double)vr[g][e], acc[e]);
                } else {
                    const double a = vr[g][e], b = vr[g][e + 1];
                    acc[e] = fma(-cr, a, fma(ci, b, acc[e]));
                    acc[e + 1] = fma(-cr, b, fma(-ci, a, acc[e + 1]));
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < RU; ++u) {
        const uint64_t q = tile0 + ((uint64_t)u * RB + t) * L;
        if (q + L <= nsc) {
            typedef typename Chunk16<T>::type V16;
            V16 v;
#pragma unroll
            for (int e = 0; e < L; ++e) v[e] = (T)acc[u * L + e];
            *(__attribute__((address_space(1))) V16 *)(w + q) = v;
        } else {
#pragma unroll
            for (int e = 0; e < L; ++e)
                if (q + e < nsc) w[q + e] = (T)acc[u * L + e];
        }
    }
}

// Second Gram-Schmidt pass only where the first removed more than half of
// |w|^2 (Daniel, Gragg, Kaufman and Stewart 1976, eta = 1/sqrt 2): skip = 1
// when |w'|^2 >= |w|^2 / 2 (no cancellation, w' orthogonal to working
// precision).
__global__ void k_dgks(const double *n0, const double *n1, int *skip) {
    if (threadIdx.x == 0) *skip = (*n1 >= 0.5 * *n0) ? 1 : 0;
}

int vec_grid(uint64_t n) {
    const uint64_t want = (n + RB - 1) / RB;
    return (int)std::max<uint64_t>(1, std::min<uint64_t>(want, (uint64_t)device_cu_count() * 8));
}

// One family of vector kernels for a dtype.
struct VecOps {
    bool single;
    int cols, C;
    uint64_t n;        // scalars per vector block
    int grid;
    double *partials;  // [grid][cols]
    hipStream_t st;

    // one column and vector-aligned buffers: the four-wide kernels
    bool vec4(const void *p) const {
        return cols == 1 && ((uintptr_t)p % (single ? 16 : 32)) == 0;
    }
    int dot(const void *a, const void *b) const {
        if (vec4(a) && vec4(b)) {
            if (single)
                hipLaunchKernelGGL(k_dot1<float>, dim3(grid), dim3(RB), 0, st, (const float *)a,
                                   (const float *)b, n, partials);
            else
                hipLaunchKernelGGL(k_dot1<double>, dim3(grid), dim3(RB), 0, st, (const double *)a,
                                   (const double *)b, n, partials);
            XDG_TRY_HIP(hipGetLastError());
            return XDG_OK;
        }
        if (single)
            hipLaunchKernelGGL(k_dot<float>, dim3(grid), dim3(RB), 0, st, (const float *)a,
                               (const float *)b, n, cols, partials);
        else
            hipLaunchKernelGGL(k_dot<double>, dim3(grid), dim3(RB), 0, st, (const double *)a,
                               (const double *)b, n, cols, partials);
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }
    // hist (may be null): a second place for the total, device or page-locked host memory
    int finalize(int mode, double *out, double *hist) const {
        hipLaunchKernelGGL(k_finalize, dim3(1), dim3(RB), 0, st, partials, grid, cols, C, mode,
                           out, hist);
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }
    int update(void *w, const void *v, const void *vprev, const double *alpha,
               const double *beta) const {
        if (vec4(w) && vec4(v) && (!vprev || vec4(vprev))) {
            if (single)
                hipLaunchKernelGGL(k_update1<float>, dim3(grid), dim3(RB), 0, st, (float *)w,
                                   (const float *)v, (const float *)vprev, n, alpha, beta,
                                   partials);
            else
                hipLaunchKernelGGL(k_update1<double>, dim3(grid), dim3(RB), 0, st, (double *)w,
                                   (const double *)v, (const double *)vprev, n, alpha, beta,
                                   partials);
            XDG_TRY_HIP(hipGetLastError());
            return XDG_OK;
        }
        if (single)
            hipLaunchKernelGGL(k_update<float>, dim3(grid), dim3(RB), 0, st, (float *)w,
                               (const float *)v, (const float *)vprev, n, cols, C, alpha, beta,
                               partials);
        else
            hipLaunchKernelGGL(k_update<double>, dim3(grid), dim3(RB), 0, st, (double *)w,
                               (const double *)v, (const double *)vprev, n, cols, C, alpha, beta,
                               partials);
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }
    int scale(const void *src, void *dst, const double *beta) const {
        if (vec4(src) && vec4(dst)) {
            if (single)
                hipLaunchKernelGGL(k_scale1<float>, dim3(grid), dim3(RB), 0, st,
                                   (const float *)src, (float *)dst, n, beta);
            else
                hipLaunchKernelGGL(k_scale1<double>, dim3(grid), dim3(RB), 0, st,
                                   (const double *)src, (double *)dst, n, beta);
            XDG_TRY_HIP(hipGetLastError());
            return XDG_OK;
        }
        if (single)
            hipLaunchKernelGGL(k_scale<float>, dim3(grid), dim3(RB), 0, st, (const float *)src,
                               (float *)dst, n, cols, C, beta);
        else
            hipLaunchKernelGGL(k_scale<double>, dim3(grid), dim3(RB), 0, st, (const double *)src,
                               (double *)dst, n, cols, C, beta);
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }

    // the total of the dot product's partials, then the update with it (one
    // vector, at most FUSE_WGS workgroups); its norm partials go to `norms`
    bool fusable() const { return cols == C && grid <= FUSE_WGS; }
    template <class F>
    int typed(bool one, F &&f) const {
        if (single) {
            if (one) f(float(), std::true_type()); else f(float(), std::false_type());
        } else {
            if (one) f(double(), std::true_type()); else f(double(), std::false_type());
        }
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }
    int total_update(void *w, const void *v, const void *vprev, double *alpha, double *host_alpha,
                     const double *beta, double *norms) const {
        return typed(vec4(w) && vec4(v) && (!vprev || vec4(vprev)), [&](auto t, auto one) {
            using T = decltype(t);
            hipLaunchKernelGGL((k_total_update<T, decltype(one)::value>), dim3(grid), dim3(RB), 0,
                               st, (T *)w, (const T *)v, (const T *)vprev, n, cols, C, partials,
                               alpha, host_alpha, beta, norms);
        });
    }
    int total_scale(const void *src, void *dst, const double *norms, double *beta,
                    double *host_beta) const {
        return typed(vec4(src) && vec4(dst), [&](auto t, auto one) {
            using T = decltype(t);
            hipLaunchKernelGGL((k_total_scale<T, decltype(one)::value>), dim3(grid), dim3(RB), 0,
                               st, (const T *)src, (T *)dst, n, cols, C, norms, beta, host_beta);
        });
    }
};

// The vector operations of a batch: n blocks of `slots` vector slots each (a
// block's slots 256-byte aligned, as many blocks in an allocation as fit
// ARENA bytes, larger ones alone), with `n_scal` scalars per block and a step
// counter.
struct ManyOps {
    bool single;
    ManyArgs A;
    uint32_t wgs;          // workgroups of all blocks
    hipStream_t st;
    std::vector<ManyBlock> blk;
    // (one allocation for 32 blocks of 4.8 GB took 4.4 s on every call after
    // the first, one per block 0.2 to 4.6 s: N = 32 ring, every momentum, 20
    // steps of 8 complex FP32 vectors 7.7 against 3.5 s)
    static constexpr uint64_t ARENA = (uint64_t)256 << 20;
    std::vector<DevBuf> bufs;
    DevBuf parts, scal, desc;
    int *jdev;
    size_t n_scal;

    int setup(int n, const int64_t *dims, int cols, int C, bool single_, int slots, size_t n_scal_,
              hipStream_t st_) {
        single = single_;
        st = st_;
        n_scal = n_scal_;
        blk.resize(n);
        wgs = 0;
        for (int i = 0; i < n; ++i) {
            ManyBlock &b = blk[i];
            b.n = (uint64_t)dims[i] * cols;
            b.slot = ((single ? 4 : 8) * b.n + 255) & ~(uint64_t)255;
            b.first = wgs;
            b.wgs = (uint32_t)vec_grid(b.n);
            wgs += b.wgs;
        }
        XDG_RETURN_IF(parts.alloc(sizeof(double) * (size_t)wgs * cols));
        XDG_RETURN_IF(scal.alloc(sizeof(double) * n_scal * n + 16));
        bufs = std::vector<DevBuf>(n);
        char *p = nullptr;
        for (int i = 0, last = 0; i < n; ++i) {
            ManyBlock &b = blk[i];
            if (i >= last) {   // the blocks from i on that share an allocation
                uint64_t bytes = b.slot * slots;
                for (last = i + 1; last < n && bytes + blk[last].slot * slots <= ARENA; ++last)
                    bytes += blk[last].slot * slots;
                XDG_RETURN_IF(bufs[i].alloc(bytes));
                p = bufs[i].as<char>();
            }
            b.buf = p;
            p += b.slot * slots;
            b.partials = parts.as<double>() + (size_t)b.first * cols;
            b.s = scal.as<double>() + n_scal * i;
        }
        jdev = reinterpret_cast<int *>(scal.as<double>() + n_scal * n);
        XDG_RETURN_IF(desc.upload(blk.data(), sizeof(ManyBlock) * n));
        A = ManyArgs{desc.as<ManyBlock>(), n, cols, C};
        return XDG_OK;
    }
    char *vec(int i, int slot) const { return blk[i].buf + blk[i].slot * slot; }

    template <class F>
    int launch(F &&f) const {
        // one real vector: the four-wide forms, as for a block alone
        if (single) {
            if (A.cols == 1) f(float(), std::true_type()); else f(float(), std::false_type());
        } else {
            if (A.cols == 1) f(double(), std::true_type()); else f(double(), std::false_type());
        }
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }
    int dot(int va, int vb) const {
        return launch([&](auto t, auto one) {
            hipLaunchKernelGGL((k_many_dot<decltype(t), decltype(one)::value>), dim3(wgs),
                               dim3(RB), 0, st, A, va, vb);
        });
    }
    int total(int mode, int out, int hist) const {
        hipLaunchKernelGGL(k_many_total, dim3(A.n_blk), dim3(RB), 0, st, A, mode, out, hist, jdev);
        XDG_TRY_HIP(hipGetLastError());
        return XDG_OK;
    }
    int update(int w, int v, int vp, int alpha, int beta) const {
        return launch([&](auto t, auto one) {
            hipLaunchKernelGGL((k_many_update<decltype(t), decltype(one)::value>), dim3(wgs),
                               dim3(RB), 0, st, A, w, v, vp, alpha, beta);
        });
    }
    int scale(int src, int dst, int beta, int keep, int *counter) const {
        return launch([&](auto t, auto one) {
            hipLaunchKernelGGL((k_many_scale<decltype(t), decltype(one)::value>), dim3(wgs),
                               dim3(RB), 0, st, A, src, dst, beta, keep, counter);
        });
    }
};

// acc += c v (FP64 accumulation of the Ritz vector)
template <class T>
__global__ __launch_bounds__(RB) void k_acc_axpy(double *acc, const T *v, uint64_t n, double c) {
    const uint64_t stride = (uint64_t)gridDim.x * RB;
    for (uint64_t q = (uint64_t)blockIdx.x * RB + threadIdx.x; q < n; q += stride)
        acc[q] = __builtin_fma(c, (double)v[q], acc[q]);
}

// out = acc / nrm[0], one rounding to T
template <class T>
__global__ __launch_bounds__(RB) void k_acc_out(const double *acc, T *out, uint64_t n,
                                                const double *nrm) {
    const double s = nrm[0] > 0.0 ? 1.0 / nrm[0] : 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * RB;
    for (uint64_t q = (uint64_t)blockIdx.x * RB + threadIdx.x; q < n; q += stride)
        out[q] = (T)(acc[q] * s);
}

thread_local double g_t_total = 0.0, g_t_apply = 0.0;

// XDG_LANCZOS_PROGRESS=n: print a line to stderr every n iterations (0 = off)
int progress_every() {
    static int every = -1;
    if (every < 0) {
        const char *e = getenv("XDG_LANCZOS_PROGRESS");
        every = e ? std::max(0, atoi(e)) : 0;
    }
    return every;
}

}  // namespace

// Implicit QL with shifts taken from the leading 2x2 block (Bowdler, Martin,
// Reinsch, Wilkinson 1968) on the symmetric tridiagonal matrix with alpha on
// the diagonal and beta[i] coupling i and i+1.  d receives the eigenvalues
// (unsorted); z0, if given, the first components of the eigenvectors (the
// rotations applied to the first row of the identity).
static void tridiag_ql(int m, const double *alpha, const double *beta, std::vector<double> &d,
                       std::vector<double> *z0) {
    d.assign(alpha, alpha + m);
    std::vector<double> e(m, 0.0);
    for (int i = 0; i + 1 < m; ++i) e[i] = beta[i];
    if (z0) {
        z0->assign(m, 0.0);
        (*z0)[0] = 1.0;
    }
    for (int l = 0; l < m; ++l) {
        for (int sweep = 0; sweep < 200; ++sweep) {
            int q = l;
            while (q < m - 1) {
                const double scale = std::fabs(d[q]) + std::fabs(d[q + 1]);
                if (std::fabs(e[q]) <= 1e-16 * scale) break;
                ++q;
            }
            if (q == l) break;
            double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
            double r = std::hypot(g, 1.0);
            g = d[q] - d[l] + e[l] / (g + (g >= 0 ? r : -r));
            double s = 1.0, c = 1.0, p = 0.0;
            bool split = false;
            for (int i = q - 1; i >= l; --i) {
                const double f = s * e[i], bb = c * e[i];
                r = std::hypot(f, g);
                e[i + 1] = r;
                if (r == 0.0) {
                    d[i + 1] -= p;
                    e[q] = 0.0;
                    split = true;
                    break;
                }
                s = f / r;
                c = g / r;
                g = d[i + 1] - p;
                r = (d[i] - g) * s + 2.0 * c * bb;
                p = s * r;
                d[i + 1] = g + p;
                g = c * r - bb;
                if (z0) {
                    double &zi = (*z0)[i], &zj = (*z0)[i + 1];
                    const double t = zj;
                    zj = s * zi + c * t;
                    zi = c * zi - s * t;
                }
            }
            if (split) continue;
            d[l] -= p;
            e[l] = g;
            e[q] = 0.0;
        }
    }
}

// Eigenvalues of the symmetric tridiagonal matrix, ascending.
void tridiag_eigenvalues(int m, const double *alpha, const double *beta, std::vector<double> &out) {
    std::vector<double> d;
    tridiag_ql(m, alpha, beta, d, nullptr);
    std::sort(d.begin(), d.end());
    out = d;
}

// Eigenvalue number k (ascending) of the symmetric tridiagonal matrix by
// multisection on Sturm counts (the number of negative pivots of T - x is the
// number of eigenvalues below x; Givens 1954): seven points a round, whose
// pivots are independent, so a round costs little more than one count and
// yields three bits.  A full QL run costs O(m^2) square roots for all
// eigenvalues (m = 32: 57 us, m = 200: 2.0 ms on one core; this: 4 and 30 us).
// lo, hi (may be NaN): a guess of an enclosing interval, checked.
static double tridiag_kth(int m, const double *alpha, const double *beta, int k, double lo,
                          double hi) {
    double g0 = HUGE_VAL, g1 = -HUGE_VAL, b2max = 0.0, sum = 0.0;
    static thread_local std::vector<double> b2;
    b2.assign(m, 0.0);
    for (int i = 0; i < m; ++i) {
        const double l = i ? std::fabs(beta[i - 1]) : 0.0, r = i + 1 < m ? std::fabs(beta[i]) : 0.0;
        g0 = std::min(g0, alpha[i] - l - r);
        g1 = std::max(g1, alpha[i] + l + r);
        if (i + 1 < m) b2[i + 1] = beta[i] * beta[i];
        b2max = std::max(b2max, b2[i]);
        sum += alpha[i] + l;
    }
    if (!std::isfinite(sum) || !std::isfinite(g0) || !std::isfinite(g1)) return NAN;
    constexpr int P = 7;
    constexpr double eps = 2.220446049250313e-16;
    const double tiny = 2.3e-308 * std::max(1.0, b2max);
    const double norm = std::max(std::fabs(g0), std::fabs(g1));
    auto counts = [&](const double *x, int *n) {
        double q[P];
        int c[P] = {};
        for (int p = 0; p < P; ++p) q[p] = 1.0;
        for (int i = 0; i < m; ++i) {
            const double a = alpha[i], bb = b2[i];
            for (int p = 0; p < P; ++p) {
                double v = (a - x[p]) - bb / q[p];
                v = std::fabs(v) < tiny ? -tiny : v;
                c[p] += v < 0.0;
                q[p] = v;
            }
        }
        for (int p = 0; p < P; ++p) n[p] = c[p];
    };
    double x[P];
    int n[P];
    const double slack = 4.0 * eps * norm + tiny;
    if (lo <= hi) {
        for (int p = 0; p < P; ++p) x[p] = p ? hi : lo;
        counts(x, n);
        if (!(n[0] <= k)) lo = g0 - slack;
        if (!(n[1] > k)) hi = g1 + slack;
    } else {
        lo = g0 - slack;
        hi = g1 + slack;
    }
    for (int round = 0; round < 100; ++round) {
        const double w = hi - lo;
        if (w <= 2.0 * eps * std::max(std::fabs(lo), std::fabs(hi)) || w <= 0.25 * eps * norm)
            break;
        for (int p = 0; p < P; ++p) x[p] = lo + w * ((p + 1) / 8.0);
        counts(x, n);
        double nl = lo, nh = hi;
        for (int p = 0; p < P; ++p) {
            if (n[p] <= k) nl = std::max(nl, x[p]);
            if (n[P - 1 - p] > k) nh = std::min(nh, x[P - 1 - p]);
        }
        if (!(nl < nh) || (nl == lo && nh == hi)) break;
        lo = nl;
        hi = nh;
    }
    return 0.5 * (lo + hi);
}

// Eigenvalue number k of the matrix: the lowest ones alone, further ones with all.
constexpr int KTH_ALONE = 8;
static double tridiag_eigenvalue(int m, const double *alpha, const double *beta, int k,
                                 std::vector<double> &all) {
    if (k < KTH_ALONE) return tridiag_kth(m, alpha, beta, k, NAN, NAN);
    if ((int)all.size() != m) tridiag_eigenvalues(m, alpha, beta, all);
    return all[k];
}

// Eigenvalues (ascending) and the squared first components of their
// eigenvectors: the nodes and weights of the Gauss quadrature that the
// Lanczos recurrence defines for the start vector.
void tridiag_spectral_weights(int m, const double *alpha, const double *beta,
                              std::vector<double> &evals, std::vector<double> &weights) {
    std::vector<double> d, z;
    tridiag_ql(m, alpha, beta, d, &z);
    std::vector<int> order(m);
    for (int i = 0; i < m; ++i) order[i] = i;
    std::sort(order.begin(), order.end(), [&](int a, int b) { return d[a] < d[b]; });
    evals.resize(m);
    weights.resize(m);
    for (int i = 0; i < m; ++i) {
        evals[i] = d[order[i]];
        weights[i] = z[order[i]] * z[order[i]];
    }
}

int lanczos_single(xdg_ham_s *h, const void *v0, int k, double tol, int max_iter, uint64_t seed,
                   int prec, double *evals, int *n_iter, double *alpha, double *beta,
                   hipStream_t st, double *t_total, double *t_apply) {
    const xdg_basis_s *b = h->basis;
    if (k < 1 || max_iter < 1 || !evals || !n_iter || !(tol >= 0.0)) {
        set_error("lanczos: need k >= 1, max_iter >= 1, tol >= 0 and output pointers");
        return XDG_EINVAL;
    }
    if (prec < XDG_PREC_F64 || prec > XDG_PREC_F64_REORTH) {
        set_error("unknown precision form %d", prec);
        return XDG_EINVAL;
    }
    const int64_t D = b->dim;
    if (D < 1) {
        set_error("lanczos on an empty block");
        return XDG_EINVAL;
    }
    const bool single = prec == XDG_PREC_F32VEC || prec == XDG_PREC_F32VEC_REORTH;
    const bool reorth = prec == XDG_PREC_F32VEC_REORTH || prec == XDG_PREC_F64_REORTH;
    const int C = b->is_complex ? 2 : 1;
    const int dtype = C == 2 ? (single ? XDG_C64 : XDG_C128) : (single ? XDG_F32 : XDG_F64);
    const size_t esz = (single ? 4 : 8) * C;
    const uint64_t nsc = (uint64_t)D * C;
    const size_t vbytes = (size_t)D * esz;
    // slots 256-byte aligned (the vector kernels load four scalars at a time)
    const size_t vstride = (vbytes + 255) & ~(size_t)255;
    const uint64_t ld = vstride / (single ? 4 : 8);   // slot stride in scalars

    DevBuf bufs, wbuf, scal, parts, rparts;
    // vectors: reorth keeps every v_j (column j of V); otherwise three rotate
    const int nstore = reorth ? max_iter + 1 : 3;
    XDG_RETURN_IF(bufs.alloc(vstride * nstore));
    XDG_RETURN_IF(wbuf.alloc(vbytes));
    // scalars: the start norm, |w|^2 before and after a first
    // reorthogonalisation pass, hist_alpha[max_iter], hist_beta[max_iter],
    // coef[2 (max_iter + 1)], then the skip flag of the second pass
    XDG_RETURN_IF(scal.alloc(sizeof(double) * (3 + 2 * (size_t)max_iter + 2 * (size_t)(max_iter + 1)) + 16));
    double *start_nrm = scal.as<double>(), *nrm0 = start_nrm + 1, *nrm1 = start_nrm + 2;
    double *hist_a = start_nrm + 3, *hist_b = hist_a + max_iter;
    double *coef = hist_b + max_iter;
    int *skip2 = reinterpret_cast<int *>(coef + 2 * (size_t)(max_iter + 1));
    // the kernels write every alpha and beta here too, so that the host reads
    // them without a copy once their step has passed
    double *ha = nullptr;
    XDG_RETURN_IF(host_scalars(2 * (size_t)max_iter, &ha));
    double *hb = ha + max_iter;
    VecOps ops{single, C, C, nsc, vec_grid(nsc), nullptr, st};
    XDG_RETURN_IF(parts.alloc(sizeof(double) * (size_t)ops.grid * MAXC));
    ops.partials = parts.as<double>();
    // reorthogonalisation: one block per row tile; partial sums per (column, block)
    const int rtile = single ? tile_scalars<float>() : tile_scalars<double>();
    const int rgrid = (int)((nsc + rtile - 1) / rtile);
    if (reorth)
        XDG_RETURN_IF(rparts.alloc(sizeof(double) * (size_t)C * rgrid * (max_iter + 1)));

    auto vec = [&](int i) -> char * { return bufs.as<char>() + vstride * i; };
    char *w = wbuf.as<char>();
    if (v0)
        XDG_TRY_HIP(hipMemcpyAsync(vec(0), v0, vbytes, hipMemcpyDeviceToDevice, st));
    else
        XDG_RETURN_IF(random_fill((int64_t)nsc, seed, 1, single, vec(0), st));
    XDG_RETURN_IF(ops.dot(vec(0), vec(0)));
    XDG_RETURN_IF(ops.finalize(1, start_nrm, nullptr));
    XDG_RETURN_IF(ops.scale(vec(0), vec(0), start_nrm));
    DevBuf norms;   // fused form: |w|^2 partials beside those of the dot product
    const bool fused = !reorth && ops.fusable();
    if (fused) XDG_RETURN_IF(norms.alloc(sizeof(double) * (size_t)ops.grid * MAXC));
    if (relabelled(h, nullptr)) h->lanczos_relabelled = true;

    // one event pair per iteration around the apply; summed at the end
    struct Events {
        std::vector<hipEvent_t> e;
        int at(size_t i, hipEvent_t *out) {
            while (e.size() <= i) {
                hipEvent_t x = nullptr;
                XDG_TRY_HIP(hipEventCreate(&x));
                e.push_back(x);
            }
            *out = e[i];
            return XDG_OK;
        }
        ~Events() {
            for (hipEvent_t x : e) (void)hipEventDestroy(x);
        }
    } evs;
    struct CheckEvent {
        hipEvent_t e = nullptr;
        ~CheckEvent() {
            if (e) (void)hipEventDestroy(e);
        }
    } checked;
    XDG_TRY_HIP(hipEventCreateWithFlags(&checked.e, hipEventDisableTiming));
    double prev_k = NAN, last_move = NAN;
    int m = 0, status = XDG_ENOCONV;
    bool stop = false;
    double apply_s = 0.0;
    // The test of iteration j: breakdown anywhere since the last test
    // truncates the run there; the k-th lowest Ritz value within tol stops it.
    auto test = [&](int mm) -> int {
        XDG_TRY_HIP(hipEventSynchronize(checked.e));
        m = mm;
        for (int t = std::max(0, mm - 16); t < mm; ++t)
            if (hb[t] <= 1e-13 * std::max(1.0, std::fabs(ha[t])) || !std::isfinite(hb[t])) {
                m = t + 1;
                stop = true;
                status = XDG_OK;
                return XDG_OK;
            }
        if (tol > 0.0 && mm >= k) {
            // the k-th value only falls as the matrix grows: look just below the last one
            const double span = 4.0 * last_move + 1e-13 * std::fabs(prev_k);
            const double th = tridiag_kth(mm, ha, hb, k - 1, prev_k - span,
                                          prev_k + 1e-13 * std::fabs(prev_k));
            if (std::isfinite(prev_k) && std::fabs(th - prev_k) <= tol * std::fabs(th)) {
                stop = true;
                status = XDG_OK;
            }
            last_move = std::fabs(th - prev_k);
            prev_k = th;
        }
        return XDG_OK;
    };
    // Where an iteration is short beside a round trip to the host (about 20
    // us), the next one is enqueued before the test of the last: at most one
    // iteration too many runs, and its numbers are not used.
    const bool ahead = nsc <= (uint64_t)1 << 22;
    int pending = 0;
    XDG_TRY_HIP(hipStreamSynchronize(st));
    const auto t0 = std::chrono::steady_clock::now();
    int iv = 0, ip = -1, in = 1;   // rotating indices (v, vprev, next) when not reorth
    for (int j = 0; j < max_iter && !stop; ++j) {
        char *v = reorth ? vec(j) : vec(iv);
        char *vp = reorth ? (j ? vec(j - 1) : nullptr) : (ip >= 0 ? vec(ip) : nullptr);
        char *next = reorth ? vec(j + 1) : vec(in);
        hipEvent_t e0, e1;
        XDG_RETURN_IF(evs.at(2 * (size_t)j, &e0));
        XDG_RETURN_IF(evs.at(2 * (size_t)j + 1, &e1));
        XDG_TRY_HIP(hipEventRecord(e0, st));
        XDG_RETURN_IF(apply_tuned(h, v, w, 1, dtype, st));
        XDG_TRY_HIP(hipEventRecord(e1, st));
        XDG_RETURN_IF(ops.dot(v, w));
        const double *beta_prev = j ? hist_b + (j - 1) : nullptr;
        if (fused) {
            XDG_RETURN_IF(ops.total_update(w, v, vp, hist_a + j, ha + j, beta_prev,
                                           norms.as<double>()));
            XDG_RETURN_IF(ops.total_scale(w, next, norms.as<double>(), hist_b + j, hb + j));
        } else {
            XDG_RETURN_IF(ops.finalize(0, hist_a + j, ha + j));
            XDG_RETURN_IF(ops.update(w, v, vp, hist_a + j, beta_prev));
        }
        if (reorth) {
            // classical Gram-Schmidt against v_0 .. v_j, FP64 coefficients; the
            // second pass runs only where the first removed more than half of |w|^2
            const int kk = j + 1;
            double *rp = rparts.as<double>();
            auto pass = [&](const int *skip) -> int {
                if (single) {
                    const float *Vf = (const float *)vec(0);
                    float *wf = (float *)w;
                    if (C == 1) {
                        hipLaunchKernelGGL((k_reorth_dots<float, 1>), dim3(rgrid), dim3(RB), 0, st,
                                           Vf, ld, kk, wf, nsc, rp, skip);
                        hipLaunchKernelGGL(k_reorth_finalize<1>, dim3(kk), dim3(RB), 0, st, rp,
                                           rgrid, coef, skip);
                        hipLaunchKernelGGL((k_reorth_sub<float, 1>), dim3(rgrid), dim3(RB), 0, st,
                                           Vf, ld, kk, coef, wf, nsc, skip);
                    } else {
                        hipLaunchKernelGGL((k_reorth_dots<float, 2>), dim3(rgrid), dim3(RB), 0, st,
                                           Vf, ld, kk, wf, nsc, rp, skip);
                        hipLaunchKernelGGL(k_reorth_finalize<2>, dim3(2 * kk), dim3(RB), 0, st,
                                           rp, rgrid, coef, skip);
                        hipLaunchKernelGGL((k_reorth_sub<float, 2>), dim3(rgrid), dim3(RB), 0, st,
                                           Vf, ld, kk, coef, wf, nsc, skip);
                    }
                } else {
                    const double *Vd = (const double *)vec(0);
                    double *wd = (double *)w;
                    if (C == 1) {
                        hipLaunchKernelGGL((k_reorth_dots<double, 1>), dim3(rgrid), dim3(RB), 0,
                                           st, Vd, ld, kk, wd, nsc, rp, skip);
                        hipLaunchKernelGGL(k_reorth_finalize<1>, dim3(kk), dim3(RB), 0, st, rp,
                                           rgrid, coef, skip);
                        hipLaunchKernelGGL((k_reorth_sub<double, 1>), dim3(rgrid), dim3(RB), 0,
                                           st, Vd, ld, kk, coef, wd, nsc, skip);
                    } else {
                        hipLaunchKernelGGL((k_reorth_dots<double, 2>), dim3(rgrid), dim3(RB), 0,
                                           st, Vd, ld, kk, wd, nsc, rp, skip);
                        hipLaunchKernelGGL(k_reorth_finalize<2>, dim3(2 * kk), dim3(RB), 0, st,
                                           rp, rgrid, coef, skip);
                        hipLaunchKernelGGL((k_reorth_sub<double, 2>), dim3(rgrid), dim3(RB), 0,
                                           st, Vd, ld, kk, coef, wd, nsc, skip);
                    }
                }
                XDG_TRY_HIP(hipGetLastError());
                return XDG_OK;
            };
            XDG_RETURN_IF(ops.finalize(0, nrm0, nullptr));   // |w|^2 from the update
            XDG_RETURN_IF(pass(nullptr));
            XDG_RETURN_IF(ops.dot(w, w));
            XDG_RETURN_IF(ops.finalize(0, nrm1, nullptr));
            hipLaunchKernelGGL(k_dgks, dim3(1), dim3(64), 0, st, nrm0, nrm1, skip2);
            XDG_TRY_HIP(hipGetLastError());
            XDG_RETURN_IF(pass(skip2));
            XDG_RETURN_IF(ops.dot(w, w));
        }
        if (!fused) XDG_RETURN_IF(ops.finalize(1, hist_b + j, hb + j));
        if (pending) {   // the iteration before this one
            XDG_RETURN_IF(test(pending));
            pending = 0;
            if (stop) break;
        }
        m = j + 1;
        if (progress_every() && m % progress_every() == 0) {
            XDG_TRY_HIP(hipStreamSynchronize(st));
            fprintf(stderr, "[xdg] lanczos iteration %d / %d\n", m, max_iter);
        }
        if (tol > 0.0 || m == max_iter || (m % 16) == 0) {
            XDG_TRY_HIP(hipEventRecord(checked.e, st));
            if (ahead && m < max_iter)
                pending = m;
            else
                XDG_RETURN_IF(test(m));
        }
        if (stop) break;
        if (!fused) XDG_RETURN_IF(ops.scale(w, next, hist_b + j));
        if (!reorth) {
            ip = iv;
            iv = in;
            in = (in + 1) % 3;
            if (in == ip) in = (in + 1) % 3;
        }
    }
    XDG_TRY_HIP(hipStreamSynchronize(st));
    const double total =
        std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    for (int j = 0; j < m; ++j) {
        float ms = 0;
        hipEvent_t e0, e1;
        XDG_RETURN_IF(evs.at(2 * (size_t)j, &e0));
        XDG_RETURN_IF(evs.at(2 * (size_t)j + 1, &e1));
        if (hipEventElapsedTime(&ms, e0, e1) == hipSuccess) apply_s += 1e-3 * ms;
    }
    if (tol == 0.0 && !stop) status = XDG_OK;
    std::vector<double> all;
    for (int e = 0; e < k; ++e) evals[e] = e < m ? tridiag_eigenvalue(m, ha, hb, e, all) : NAN;
    *n_iter = m;
    if (alpha) std::copy(ha, ha + m, alpha);
    if (beta) std::copy(hb, hb + m, beta);
    g_t_total = total;
    g_t_apply = apply_s;
    if (t_total) *t_total = total;
    if (t_apply) *t_apply = apply_s;
    return status;
}

// n blocks x nvec recurrences in lockstep; each step (batched apply, then
// per-block dot / update / norm / scale) is captured once per buffer
// rotation phase into a HIP graph and replayed.
// Eigenvector of the symmetric tridiagonal matrix for its eigenvalue number
// `which` (ascending), by inverse iteration: (T - theta) x = x_prev solved by
// Gaussian elimination with partial pivoting on the tridiagonal band, three
// sweeps.  Normalised, first nonzero component made positive.
void tridiag_eigvec(int m, const double *alpha, const double *beta, int which,
                    std::vector<double> &x, double &theta) {
    std::vector<double> ev;
    theta = tridiag_eigenvalue(m, alpha, beta, which, ev);
    double tnorm = 0.0;
    for (int i = 0; i < m; ++i)
        tnorm = std::max(tnorm, std::fabs(alpha[i]) + (i ? std::fabs(beta[i - 1]) : 0.0) +
                                    (i + 1 < m ? std::fabs(beta[i]) : 0.0));
    const double tiny = std::max(tnorm, 1e-300) * 1e-15;
    // factor P (T - theta) = L U; U has diagonals d, u1, u2; L multipliers f
    std::vector<double> d(m), u1(m, 0.0), u2(m, 0.0), f(m, 0.0);
    std::vector<char> swp(m, 0);
    for (int i = 0; i < m; ++i) {
        d[i] = alpha[i] - theta;
        if (i + 1 < m) u1[i] = beta[i];
    }
    for (int i = 0; i + 1 < m; ++i) {
        const double sub = beta[i];   // row i+1, column i
        if (std::fabs(d[i]) >= std::fabs(sub)) {
            if (d[i] == 0.0) d[i] = tiny;
            f[i] = sub / d[i];
            d[i + 1] -= f[i] * u1[i];
        } else {
            // rows i and i+1 exchanged
            swp[i] = 1;
            f[i] = d[i] / sub;
            d[i] = sub;
            const double r1 = u1[i];       // old row i, column i+1
            u1[i] = d[i + 1];              // old row i+1, column i+1
            d[i + 1] = r1 - f[i] * u1[i];
            if (i + 2 < m) {
                u2[i] = u1[i + 1];         // old row i+1, column i+2
                u1[i + 1] = -f[i] * u2[i];
            }
        }
    }
    if (d[m - 1] == 0.0) d[m - 1] = tiny;
    x.assign(m, 1.0);
    for (int sweep = 0; sweep < 3; ++sweep) {
        // forward: apply P and L^-1
        for (int i = 0; i + 1 < m; ++i) {
            if (swp[i]) std::swap(x[i], x[i + 1]);
            x[i + 1] -= f[i] * x[i];
        }
        // back substitution with U
        for (int i = m - 1; i >= 0; --i) {
            double r = x[i];
            if (i + 1 < m) r -= u1[i] * x[i + 1];
            if (i + 2 < m) r -= u2[i] * x[i + 2];
            x[i] = r / (d[i] != 0.0 ? d[i] : tiny);
        }
        double nrm = 0.0;
        for (double v : x) nrm += v * v;
        nrm = std::sqrt(nrm);
        for (double &v : x) v /= nrm;
    }
    for (int i = 0; i < m; ++i)
        if (x[i] != 0.0) {
            if (x[i] < 0.0)
                for (double &v : x) v = -v;
            break;
        }
}

int lanczos_eigvec(xdg_ham_s *h, const void *v0, uint64_t seed, int prec, int m,
                   const double *alpha, const double *beta, int which, void *psi, double *ritz,
                   hipStream_t st) {
    const xdg_basis_s *b = h->basis;
    if (prec != XDG_PREC_F64 && prec != XDG_PREC_F32VEC) {
        set_error("second Lanczos pass: precision form %d not supported (no reorthogonalisation)",
                  prec);
        return XDG_EINVAL;
    }
    if (m < 1 || which < 0 || which >= m || !alpha || !beta || !psi || psi == v0) {
        set_error("second Lanczos pass: need n_iter >= 1, 0 <= which < n_iter, alpha, beta and a "
                  "psi distinct from v0");
        return XDG_EINVAL;
    }
    const int64_t D = b->dim;
    if (D < 1) {
        set_error("lanczos on an empty block");
        return XDG_EINVAL;
    }
    for (int j = 0; j + 1 < m; ++j)
        if (!(beta[j] > 0.0)) {
            set_error("second Lanczos pass: beta[%d] = %g ends the recurrence before n_iter", j,
                      beta[j]);
            return XDG_EINVAL;
        }
    // The vectors equal those of the first pass only in the labelling it ran in: if
    // that has been given up since, the matrix of this one takes its place (with the
    // other's, rounding errors grew to 2.7 times the residual on a 6x6 block).
    std::vector<double> own_a, own_b;
    if (h->lanczos_relabelled && !relabelled(h, nullptr)) {
        own_a.resize(m);
        own_b.resize(m);
        double lowest = 0.0;
        int steps = 0;
        const double total = g_t_total, apply = g_t_apply;   // (of the caller's first pass)
        XDG_RETURN_IF(lanczos_single(h, v0, 1, 0.0, m, seed, prec, &lowest, &steps, own_a.data(),
                                     own_b.data(), st, nullptr, nullptr));
        g_t_total = total;
        g_t_apply = apply;
        if (steps == m) {
            alpha = own_a.data();
            beta = own_b.data();
        }
    }
    std::vector<double> c;
    double theta = 0.0;
    tridiag_eigvec(m, alpha, beta, which, c, theta);
    if (ritz) *ritz = theta;

    const bool single = prec == XDG_PREC_F32VEC;
    const int C = b->is_complex ? 2 : 1;
    const int dtype = C == 2 ? (single ? XDG_C64 : XDG_C128) : (single ? XDG_F32 : XDG_F64);
    const size_t esz = (single ? 4 : 8) * C;
    const uint64_t nsc = (uint64_t)D * C;
    const size_t vbytes = (size_t)D * esz;
    const size_t vstride = (vbytes + 255) & ~(size_t)255;   // 256-byte aligned slots
    DevBuf bufs, wbuf, acc, scal, parts;
    XDG_RETURN_IF(bufs.alloc(vstride * 3));
    XDG_RETURN_IF(wbuf.alloc(vbytes));
    XDG_RETURN_IF(acc.alloc(sizeof(double) * nsc));
    // scalars: nrm, alpha[m], beta[m]
    XDG_RETURN_IF(scal.alloc(sizeof(double) * (1 + 2 * (size_t)m)));
    double *nrm = scal.as<double>(), *al_d = nrm + 1, *be_d = al_d + m;
    std::vector<double> ab(alpha, alpha + m);
    ab.insert(ab.end(), beta, beta + m);
    XDG_RETURN_IF(copy_h2d(al_d, ab.data(), sizeof(double) * ab.size(), st));
    XDG_TRY_HIP(hipMemsetAsync(acc.p, 0, acc.bytes, st));
    VecOps ops{single, C, C, nsc, vec_grid(nsc), nullptr, st};
    XDG_RETURN_IF(parts.alloc(sizeof(double) * (size_t)ops.grid * MAXC));
    ops.partials = parts.as<double>();
    auto vec = [&](int i) -> char * { return bufs.as<char>() + vstride * i; };
    char *w = wbuf.as<char>();
    // start vector exactly as in the first pass
    if (v0)
        XDG_TRY_HIP(hipMemcpyAsync(vec(0), v0, vbytes, hipMemcpyDeviceToDevice, st));
    else
        XDG_RETURN_IF(random_fill((int64_t)nsc, seed, 1, single, vec(0), st));
    XDG_RETURN_IF(ops.dot(vec(0), vec(0)));
    XDG_RETURN_IF(ops.finalize(1, nrm, nullptr));
    XDG_RETURN_IF(ops.scale(vec(0), vec(0), nrm));
    const int g = vec_grid(nsc);
    if (single)
        hipLaunchKernelGGL(k_acc_axpy<float>, dim3(g), dim3(RB), 0, st, acc.as<double>(),
                           (const float *)vec(0), nsc, c[0]);
    else
        hipLaunchKernelGGL(k_acc_axpy<double>, dim3(g), dim3(RB), 0, st, acc.as<double>(),
                           (const double *)vec(0), nsc, c[0]);
    XDG_TRY_HIP(hipGetLastError());
    int iv = 0, ip = -1, in = 1;
    for (int j = 0; j + 1 < m; ++j) {
        char *v = vec(iv), *vp = ip >= 0 ? vec(ip) : nullptr;
        XDG_RETURN_IF(apply_tuned(h, v, w, 1, dtype, st));
        const double *bp = j ? be_d + j - 1 : nullptr;
        if (single)
            hipLaunchKernelGGL(k_ritz_step<float>, dim3(g), dim3(RB), 0, st, (const float *)w,
                               (const float *)v, (const float *)vp, (float *)vec(in),
                               acc.as<double>(), nsc, al_d + j, bp, be_d + j, c[j + 1]);
        else
            hipLaunchKernelGGL(k_ritz_step<double>, dim3(g), dim3(RB), 0, st, (const double *)w,
                               (const double *)v, (const double *)vp, (double *)vec(in),
                               acc.as<double>(), nsc, al_d + j, bp, be_d + j, c[j + 1]);
        XDG_TRY_HIP(hipGetLastError());
        ip = iv;
        iv = in;
        in = (in + 1) % 3;
        if (in == ip) in = (in + 1) % 3;
        if (progress_every() && (j + 1) % progress_every() == 0) {
            XDG_TRY_HIP(hipStreamSynchronize(st));
            fprintf(stderr, "[xdg] second lanczos pass %d / %d\n", j + 1, m);
        }
    }
    // psi = acc / |acc|
    VecOps dops{false, 1, 1, nsc, vec_grid(nsc), parts.as<double>(), st};
    XDG_RETURN_IF(dops.dot(acc.p, acc.p));
    XDG_RETURN_IF(dops.finalize(1, nrm, nullptr));
    if (single)
        hipLaunchKernelGGL(k_acc_out<float>, dim3(g), dim3(RB), 0, st, acc.as<double>(),
                           (float *)psi, nsc, nrm);
    else
        hipLaunchKernelGGL(k_acc_out<double>, dim3(g), dim3(RB), 0, st, acc.as<double>(),
                           (double *)psi, nsc, nrm);
    XDG_TRY_HIP(hipGetLastError());
    XDG_TRY_HIP(hipStreamSynchronize(st));
    return XDG_OK;
}

int lanczos_batched(int n, xdg_ham_s *const *hams, const void *const *v0s, int64_t nvec,
                    int n_iter, uint64_t seed, int prec, double *evals, double *alpha,
                    double *beta, hipStream_t user_st, double *t_total, double *t_apply) {
    if (n < 1 || n_iter < 1 || !evals) {
        set_error("batched lanczos: need n >= 1, n_iter >= 1 and evals");
        return XDG_EINVAL;
    }
    if (nvec != 1 && nvec != 2 && nvec != 4 && nvec != 8) {
        set_error("batched lanczos: nvec must be 1, 2, 4 or 8");
        return XDG_EINVAL;
    }
    if (prec != XDG_PREC_F64 && prec != XDG_PREC_F32VEC) {
        set_error("batched lanczos supports XDG_PREC_F64 and XDG_PREC_F32VEC");
        return XDG_EINVAL;
    }
    bool any_c = false;
    for (int i = 0; i < n; ++i) {
        if (!hams[i] || hams[i]->basis->dim < 1) {
            set_error("batched lanczos: block %d is null or empty", i);
            return XDG_EINVAL;
        }
        any_c |= hams[i]->basis->is_complex;
    }
    const bool single = prec == XDG_PREC_F32VEC;
    const int C = any_c ? 2 : 1;
    const int dtype = any_c ? (single ? XDG_C64 : XDG_C128) : (single ? XDG_F32 : XDG_F64);
    const size_t ssz = single ? 4 : 8;
    const int cols = (int)nvec * C;

    hipStream_t st = user_st;
    hipStream_t own = nullptr;
    if (!st) {
        XDG_TRY_HIP(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
        st = own;
    }
    // slots: v0, v1, v2 (rotating) and w.  Scalars per block: current alpha
    // and beta, previous beta, then both histories.
    const int W = 3, nv = (int)nvec;
    const int cur_a = 0, cur_b = nv, prev_b = 2 * nv, hist_a = 3 * nv,
              hist_b = hist_a + n_iter * nv;
    std::vector<int64_t> dims(n);
    for (int i = 0; i < n; ++i) dims[i] = hams[i]->basis->dim;
    ManyOps ops;
    XDG_RETURN_IF(ops.setup(n, dims.data(), cols, C, single, 4,
                            (size_t)3 * nv + 2 * (size_t)n_iter * nv, st));
    for (int i = 0; i < n; ++i) {
        char *v = ops.vec(i, 0);
        const uint64_t nsc = ops.blk[i].n;
        if (v0s && v0s[i])
            XDG_TRY_HIP(hipMemcpyAsync(v, v0s[i], ssz * nsc, hipMemcpyDeviceToDevice, st));
        else
            XDG_RETURN_IF(random_fill((int64_t)nsc, seed + (uint64_t)i, 1, single, v, st));
        hipLaunchKernelGGL(k_set_scalars, dim3(1), dim3(64), 0, st, ops.jdev,
                           ops.blk[i].s + prev_b, nv);
    }
    XDG_TRY_HIP(hipGetLastError());
    XDG_RETURN_IF(ops.dot(0, 0));
    XDG_RETURN_IF(ops.total(1, cur_b, -1));
    XDG_RETURN_IF(ops.scale(0, 0, cur_b, -1, nullptr));
    auto vecp = [&](int i, int slot) -> char * { return ops.vec(i, slot); };
    // phase p: v = slot p, vprev = slot (p+2)%3 (none at j = 0), next = slot (p+1)%3, w = slot 3
    std::vector<xdg_ham_s *> hv(hams, hams + n);
    const std::vector<RelabelledRef> in = relabelled(n, hv.data(), nullptr);   // to the end of the run
    auto prepare = [&](int p, BatchPlan *P, uint32_t tile) -> int {
        std::vector<const void *> xs(n);
        std::vector<void *> ys(n);
        for (int i = 0; i < n; ++i) {
            xs[i] = vecp(i, p);
            ys[i] = vecp(i, 3);
        }
        return batch_prepare(n, hv.data(), in.data(), xs.data(), ys.data(), nvec, dtype, P, tile);
    };
    // launch shape of the batched apply (tuned once per set of blocks)
    BatchShape best_shape;
    {
        std::vector<const void *> xs(n);
        std::vector<void *> ys(n);
        for (int i = 0; i < n; ++i) {
            xs[i] = vecp(i, 0);
            ys[i] = vecp(i, 3);
        }
        XDG_RETURN_IF(batch_shape_tuned(n, hv.data(), in.data(), xs.data(), ys.data(), nvec,
                                        dtype, st, &best_shape));
    }
    BatchPlan plans[3];
    for (int p = 0; p < 3; ++p) XDG_RETURN_IF(prepare(p, &plans[p], best_shape.tile));
    const int best_grid = best_shape.grid;
    auto enqueue_step = [&](int p, bool first) -> int {
        XDG_RETURN_IF(batch_launch(plans[p], best_grid, best_shape.nv, st));
        XDG_RETURN_IF(ops.dot(p, W));
        XDG_RETURN_IF(ops.total(0, cur_a, hist_a));
        XDG_RETURN_IF(ops.update(W, p, first ? -1 : (p + 2) % 3, cur_a, prev_b));
        XDG_RETURN_IF(ops.total(1, cur_b, hist_b));
        return ops.scale(W, (p + 1) % 3, cur_b, prev_b, ops.jdev);
    };
    XDG_TRY_HIP(hipStreamSynchronize(st));
    const auto t0 = std::chrono::steady_clock::now();
    // step 0 runs eagerly (it has no v_{j-1}); later steps replay graphs
    XDG_RETURN_IF(enqueue_step(0, true));
    hipGraphExec_t exec[3] = {nullptr, nullptr, nullptr};
    hipGraph_t graphs[3] = {nullptr, nullptr, nullptr};
    int rc = XDG_OK;
    for (int p = 0; p < 3 && rc == XDG_OK && n_iter > 1; ++p) {
        XDG_TRY_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
        rc = enqueue_step(p, false);
        hipError_t e = hipStreamEndCapture(st, &graphs[p]);
        if (rc == XDG_OK && e != hipSuccess) {
            set_error("graph capture failed: %s", hipGetErrorString(e));
            rc = XDG_EHIP;
        }
        if (rc == XDG_OK) {
            e = hipGraphInstantiate(&exec[p], graphs[p], nullptr, nullptr, 0);
            if (e != hipSuccess) {
                set_error("graph instantiation failed: %s", hipGetErrorString(e));
                rc = XDG_EHIP;
            }
        }
    }
    for (int j = 1; j < n_iter && rc == XDG_OK; ++j) {
        hipError_t e = hipGraphLaunch(exec[j % 3], st);
        if (e != hipSuccess) {
            set_error("graph launch failed: %s", hipGetErrorString(e));
            rc = XDG_EHIP;
        }
        if (rc == XDG_OK && progress_every() && (j + 1) % progress_every() == 0) {
            (void)hipStreamSynchronize(st);
            fprintf(stderr, "[xdg] batched lanczos iteration %d / %d\n", j + 1, n_iter);
        }
    }
    if (rc == XDG_OK) {
        hipError_t e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            set_error("batched lanczos: %s", hipGetErrorString(e));
            rc = XDG_EHIP;
        }
    }
    const double total =
        std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    for (int p = 0; p < 3; ++p) {
        if (exec[p]) (void)hipGraphExecDestroy(exec[p]);
        if (graphs[p]) (void)hipGraphDestroy(graphs[p]);
    }
    if (rc == XDG_OK) {
        std::vector<double> all(ops.n_scal * n), a1(n_iter), b1(n_iter), ritz;
        rc = copy_d2h(all.data(), ops.scal.p, sizeof(double) * all.size(), st);
        for (int i = 0; i < n && rc == XDG_OK; ++i) {
            const double *ha = all.data() + ops.n_scal * i + hist_a, *hb = ha + (hist_b - hist_a);
            for (int v = 0; v < nvec; ++v) {
                int m = n_iter;
                for (int j = 0; j < n_iter; ++j) {
                    a1[j] = ha[(size_t)j * nvec + v];
                    b1[j] = hb[(size_t)j * nvec + v];
                    if (alpha) alpha[((size_t)i * nvec + v) * n_iter + j] = a1[j];
                    if (beta) beta[((size_t)i * nvec + v) * n_iter + j] = b1[j];
                }
                for (int j = 0; j < n_iter; ++j)
                    if (b1[j] <= 1e-13 * std::max(1.0, std::fabs(a1[j])) || !std::isfinite(b1[j])) {
                        m = j + 1;
                        break;
                    }
                evals[(size_t)i * nvec + v] =
                    tridiag_eigenvalue(m, a1.data(), b1.data(), 0, ritz);
            }
        }
    }
    if (own) (void)hipStreamDestroy(own);
    g_t_total = total;
    g_t_apply = 0.0;
    if (t_total) *t_total = total;
    if (t_apply) *t_apply = 0.0;
    return rc;
}

// Microcanonical TPQ sequence (Sec. 4.6, after Sugiura and Shimizu 2012):
// |k+1> = (l - H/N)|k> / norm from a unit start vector; per step one H x,
// the FP64 products <k|H|k> and <H k|H k> into device histories, then the
// next vector H|k> - l N |k> (the sign drops out of every expectation value)
// normalised in place.  The histories reach the host once, at the end.
int tpq_micro(xdg_ham_s *h, const void *v0, uint64_t seed, int prec, double l, int n_steps,
              double *u, double *u2, hipStream_t st) {
    const xdg_basis_s *b = h->basis;
    if (n_steps < 1 || !u || !u2 || !std::isfinite(l)) {
        set_error("tpq: need n_steps >= 1, output arrays and a finite l");
        return XDG_EINVAL;
    }
    if (prec != XDG_PREC_F64 && prec != XDG_PREC_F32VEC) {
        set_error("tpq: precision form %d (XDG_PREC_F64 or XDG_PREC_F32VEC)", prec);
        return XDG_EINVAL;
    }
    const int64_t D = b->dim;
    if (D < 1) {
        set_error("tpq on an empty block");
        return XDG_EINVAL;
    }
    const bool single = prec == XDG_PREC_F32VEC;
    const int C = b->is_complex ? 2 : 1;
    const int dtype = C == 2 ? (single ? XDG_C64 : XDG_C128) : (single ? XDG_F32 : XDG_F64);
    const size_t esz = (single ? 4 : 8) * C;
    const uint64_t nsc = (uint64_t)D * C;
    const size_t vbytes = (size_t)D * esz;
    const size_t vstride = (vbytes + 255) & ~(size_t)255;
    const double N = (double)b->n_sites;

    DevBuf vbuf, scal, parts;
    XDG_RETURN_IF(vbuf.alloc(2 * vstride));
    // scalars: norm, l N, histories of <v,Hv> and <Hv,Hv>
    XDG_RETURN_IF(scal.alloc(sizeof(double) * (2 + 2 * (size_t)n_steps)));
    double *s_nrm = scal.as<double>(), *s_ln = s_nrm + 1, *h_vw = s_nrm + 2, *h_ww = h_vw + n_steps;
    VecOps ops{single, C, C, nsc, vec_grid(nsc), nullptr, st};
    XDG_RETURN_IF(parts.alloc(sizeof(double) * (size_t)ops.grid * MAXC));
    ops.partials = parts.as<double>();
    char *v = vbuf.as<char>(), *w = v + vstride;
    if (v0)
        XDG_TRY_HIP(hipMemcpyAsync(v, v0, vbytes, hipMemcpyDeviceToDevice, st));
    else
        XDG_RETURN_IF(random_fill((int64_t)nsc, seed, 1, single, v, st));
    const double ln = l * N;
    XDG_TRY_HIP(hipMemcpyAsync(s_ln, &ln, sizeof(double), hipMemcpyHostToDevice, st));
    XDG_RETURN_IF(ops.dot(v, v));
    XDG_RETURN_IF(ops.finalize(1, s_nrm, nullptr));
    XDG_RETURN_IF(ops.scale(v, v, s_nrm));
    for (int k = 0; k < n_steps; ++k) {
        XDG_RETURN_IF(apply_tuned(h, v, w, 1, dtype, st));
        XDG_RETURN_IF(ops.dot(v, w));
        XDG_RETURN_IF(ops.finalize(0, h_vw + k, nullptr));
        XDG_RETURN_IF(ops.dot(w, w));
        XDG_RETURN_IF(ops.finalize(0, h_ww + k, nullptr));
        if (k + 1 < n_steps) {
            XDG_RETURN_IF(ops.update(w, v, nullptr, s_ln, nullptr));   // w = H v - l N v
            XDG_RETURN_IF(ops.finalize(1, s_nrm, nullptr));
            XDG_RETURN_IF(ops.scale(w, v, s_nrm));
        }
    }
    std::vector<double> hv(n_steps), hw(n_steps);
    XDG_RETURN_IF(copy_d2h(hv.data(), h_vw, sizeof(double) * n_steps, st));
    XDG_RETURN_IF(copy_d2h(hw.data(), h_ww, sizeof(double) * n_steps, st));
    for (int k = 0; k < n_steps; ++k) {
        u[k] = hv[k] / N;
        u2[k] = hw[k] / (N * N);
    }
    return XDG_OK;
}

// The same sequence for n blocks x nvec start vectors in lockstep: one
// batched H x per step over every block (the persistent launch), per-column
// FP64 products and updates; one captured step replayed n_steps times.
int tpq_micro_batched(int n, xdg_ham_s *const *hams, const void *const *v0s, int64_t nvec,
                      uint64_t seed, int prec, double l, int n_steps, double *u, double *u2,
                      hipStream_t user_st) {
    if (n < 1 || n_steps < 1 || !u || !u2 || !std::isfinite(l)) {
        set_error("batched tpq: need n >= 1, n_steps >= 1, output arrays and a finite l");
        return XDG_EINVAL;
    }
    if (nvec != 1 && nvec != 2 && nvec != 4 && nvec != 8) {
        set_error("batched tpq: nvec must be 1, 2, 4 or 8");
        return XDG_EINVAL;
    }
    if (prec != XDG_PREC_F64 && prec != XDG_PREC_F32VEC) {
        set_error("batched tpq: precision form %d (XDG_PREC_F64 or XDG_PREC_F32VEC)", prec);
        return XDG_EINVAL;
    }
    bool any_c = false;
    for (int i = 0; i < n; ++i) {
        if (!hams[i] || hams[i]->basis->dim < 1) {
            set_error("batched tpq: block %d is null or empty", i);
            return XDG_EINVAL;
        }
        any_c |= hams[i]->basis->is_complex;
    }
    const bool single = prec == XDG_PREC_F32VEC;
    const int C = any_c ? 2 : 1;
    const int dtype = any_c ? (single ? XDG_C64 : XDG_C128) : (single ? XDG_F32 : XDG_F64);
    const size_t ssz = single ? 4 : 8;
    const int cols = (int)nvec * C;

    hipStream_t st = user_st;
    hipStream_t own = nullptr;
    if (!st) {
        XDG_TRY_HIP(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
        st = own;
    }
    struct OwnStream {
        hipStream_t s;
        ~OwnStream() {
            if (s) (void)hipStreamDestroy(s);
        }
    } own_guard{own};
    // slots: v and w.  Scalars per block and vector: l N, norm, <v, Hv>,
    // <Hv, Hv>; then the two histories.
    const int nv = (int)nvec;
    const int ln = 0, nrm = nv, vw = 2 * nv, ww = 3 * nv, h_vw = 4 * nv, h_ww = h_vw + n_steps * nv;
    std::vector<int64_t> dims(n);
    for (int i = 0; i < n; ++i) dims[i] = hams[i]->basis->dim;
    ManyOps ops;
    XDG_RETURN_IF(ops.setup(n, dims.data(), cols, C, single, 2,
                            (size_t)4 * nv + 2 * (size_t)n_steps * nv, st));
    std::vector<double> lnv(nvec);
    for (int i = 0; i < n; ++i) {
        std::fill(lnv.begin(), lnv.end(), l * (double)hams[i]->basis->n_sites);
        XDG_RETURN_IF(copy_h2d(ops.blk[i].s + ln, lnv.data(), sizeof(double) * nvec, st));
        char *v = ops.vec(i, 0);
        const uint64_t nsc = ops.blk[i].n;
        if (v0s && v0s[i])
            XDG_TRY_HIP(hipMemcpyAsync(v, v0s[i], ssz * nsc, hipMemcpyDeviceToDevice, st));
        else
            XDG_RETURN_IF(random_fill((int64_t)nsc, seed + (uint64_t)i, 1, single, v, st));
    }
    XDG_RETURN_IF(ops.dot(0, 0));
    XDG_RETURN_IF(ops.total(1, nrm, -1));
    XDG_RETURN_IF(ops.scale(0, 0, nrm, -1, nullptr));
    hipLaunchKernelGGL(k_set_scalars, dim3(1), dim3(64), 0, st, ops.jdev, ops.blk[0].s + nrm, 0);
    XDG_TRY_HIP(hipGetLastError());
    std::vector<xdg_ham_s *> hv(hams, hams + n);
    std::vector<const void *> xs(n);
    std::vector<void *> ys(n);
    for (int i = 0; i < n; ++i) {
        xs[i] = ops.vec(i, 0);
        ys[i] = ops.vec(i, 1);
    }
    BatchShape shape;
    const std::vector<RelabelledRef> in = relabelled(n, hv.data(), nullptr);   // to the end of the run
    XDG_RETURN_IF(batch_shape_tuned(n, hv.data(), in.data(), xs.data(), ys.data(), nvec, dtype, st,
                                    &shape));
    BatchPlan plan;
    XDG_RETURN_IF(batch_prepare(n, hv.data(), in.data(), xs.data(), ys.data(), nvec, dtype, &plan,
                                shape.tile));
    auto step = [&]() -> int {
        XDG_RETURN_IF(batch_launch(plan, shape.grid, shape.nv, st));
        XDG_RETURN_IF(ops.dot(0, 1));
        XDG_RETURN_IF(ops.total(0, vw, h_vw));
        XDG_RETURN_IF(ops.dot(1, 1));
        XDG_RETURN_IF(ops.total(0, ww, h_ww));
        XDG_RETURN_IF(ops.update(1, 0, -1, ln, ln));   // H v - l N v
        XDG_RETURN_IF(ops.total(1, nrm, -1));
        return ops.scale(1, 0, nrm, -1, ops.jdev);
    };
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int rc = XDG_OK;
    XDG_TRY_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    rc = step();
    hipError_t e = hipStreamEndCapture(st, &graph);
    if (rc == XDG_OK && e != hipSuccess) {
        set_error("graph capture failed: %s", hipGetErrorString(e));
        rc = XDG_EHIP;
    }
    if (rc == XDG_OK && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
        set_error("graph instantiation failed");
        rc = XDG_EHIP;
    }
    for (int k = 0; k < n_steps && rc == XDG_OK; ++k) {
        if (hipGraphLaunch(exec, st) != hipSuccess) {
            set_error("graph launch failed");
            rc = XDG_EHIP;
        }
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (rc == XDG_OK) {
        std::vector<double> all(ops.n_scal * n);
        rc = copy_d2h(all.data(), ops.scal.p, sizeof(double) * all.size(), st);
        for (int i = 0; i < n && rc == XDG_OK; ++i) {
            const double *hv_ = all.data() + ops.n_scal * i + h_vw, *hw_ = hv_ + (h_ww - h_vw);
            const double N = (double)hams[i]->basis->n_sites;
            for (int v = 0; v < nvec; ++v)
                for (int k = 0; k < n_steps; ++k) {
                    u[((size_t)i * nvec + v) * n_steps + k] = hv_[(size_t)k * nvec + v] / N;
                    u2[((size_t)i * nvec + v) * n_steps + k] = hw_[(size_t)k * nvec + v] / (N * N);
                }
        }
    }
    return rc;
}

int last_timing(double *total, double *apply) {
    if (total) *total = g_t_total;
    if (apply) *apply = g_t_apply;
    return XDG_OK;
}

}  // namespace xdg
