// Expectation values of symmetrised Ising correlations on a block
// (measurements, Sec. 3.8; symmetrisation of an operator over the group,
// Sec. 3.13).  O_ab = (1/|G|) sum_g S^z_{g(a)} S^z_{g(b)} is diagonal on the
// symmetric basis, with value o_ab(s) = (1/|G|) sum_g sz_s(g(a)) sz_s(g(b)) on
// representative s, so <psi|O_ab|psi> = sum_s |psi_s|^2 o_ab(s).  The group
// meets every pair of the orbit of {a, b} equally often, so with S pairs in
// the orbit and n(s) of them holding unequal spins o_ab = (S - 2 n(s)) / (4 S):
// a lane counts n in integers, and the products with |psi_s|^2 are summed in
// a fixed order.
#include <algorithm>
#include <complex>
#include <vector>

#include "device_common.hpp"

namespace xdg {

namespace {

constexpr int MB = 256;       // threads per block of the correlations
constexpr int PB_RING = 16;   // pairs per pass: distances of a ring
constexpr int PB_SITE = 7;    // pairs per pass: partner masks (3.5 KB of kernel arguments)

// Pairs of one pass.  Ring: the orbit is {i, i + d} for all sites i (n(s) =
// set bits of s ^ rotr(s, d), each pair counted once per i).  Otherwise the
// partners of a site in the orbit, each pair at its lower site: sites[k] has the
// sites with any, mask[k] their partners one after the other.
template <bool RING> struct SzPairs;
template <> struct SzPairs<true> {
    int n, N;
    int d[PB_RING];
    double scale[PB_RING];         // 1 / (4 S)
};
template <> struct SzPairs<false> {
    int n, N;
    int S[PB_SITE];
    double scale[PB_SITE];
    uint64_t sites[PB_SITE];
    uint64_t mask[PB_SITE][64];
};
template <bool RING>
constexpr int sz_pairs() { return RING ? PB_RING : PB_SITE; }
static_assert(sizeof(SzPairs<false>) <= 4000, "kernel arguments");

template <class W>
__device__ __forceinline__ int popc(W v) {
    if constexpr (sizeof(W) == 4)
        return __popc(v);
    else
        return __popcll(v);
}

// Streams reps and psi once per pass.  Before, each pair of sites was a
// compare and an FP64 add per state (ring N = 30, 15 distances, complex FP64:
// 688 us in two passes); an orbit now costs three instructions per state on
// a ring and three to six per site otherwise, so that memory bounds the ring
// pass (103 MB) and the integer units the others.  The ring N = 30 example
// with a transfer after it, whole calls: 1293 -> 177 us.
template <class W, class T, int C, bool RING>
__global__ __launch_bounds__(MB) void k_szsz(const W *reps, int64_t dim, const T *psi,
                                             SzPairs<RING> A, double *partials) {
    constexpr int PB = sz_pairs<RING>();
    __shared__ double sh[MB / 64][PB];
    double acc[PB];
#pragma unroll
    for (int k = 0; k < PB; ++k) acc[k] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * MB;
    for (int64_t i = (int64_t)blockIdx.x * MB + threadIdx.x; i < dim; i += stride) {
        const W s = gld(reps + i);
        double p = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const double v = (double)gld(psi + i * C + c);
            p = __builtin_fma(v, v, p);
        }
#pragma unroll
        for (int k = 0; k < PB; ++k) {
            if (k >= A.n) break;
            int o;
            if constexpr (RING) {
                o = A.N - 2 * popc<W>(s ^ rotr_n<W>(s, A.d[k], A.N));
            } else {
                // The first site's mask stays in registers over the rows: the orbits
                // of blocks without a group, and most of mirrors, end there.  Without a
                // group, N = 26, 10.4 M rows, 23 pairs, FP64: 1234 us over all sites of
                // every pair, 799 pair by pair as before that, 215 so; two elements
                // (mirror, N = 24) 291, 267 and 116 us; 6x6 lattice, 35 pairs 1.60,
                // 4.58 and 1.23 ms.
                int n = 0;
                auto count = [&](int a, W m) {
                    const W up = W(0) - ((s >> a) & W(1));   // all ones where site a is up
                    n += popc<W>((s ^ up) & m);
                };
                uint64_t left = A.sites[k];
                if (left) {
                    count(__builtin_ctzll(left), (W)A.mask[k][0]);
                    left &= left - 1;
                    for (int e = 1; left; ++e, left &= left - 1)
                        count(__builtin_ctzll(left), (W)A.mask[k][e]);
                }
                o = A.S[k] - 2 * n;
            }
            acc[k] = __builtin_fma(p, (double)o, acc[k]);
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < PB; ++k) {
        if (k >= A.n) break;
        double v = acc[k];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) sh[wave][k] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < A.n) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < MB / 64; ++w) v += sh[w][threadIdx.x];
        partials[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = v;
    }
}

// out[k] = scale[k] times the fixed-order total of pair k's partials
template <bool RING>
__global__ __launch_bounds__(MB) void k_szsz_total(const double *partials, int n_blocks,
                                                   SzPairs<RING> A, double *out) {
    __shared__ double sh[MB];
    double v = 0.0;
    for (int b = threadIdx.x; b < n_blocks; b += MB)
        v += partials[(size_t)blockIdx.x * n_blocks + b];
    sh[threadIdx.x] = v;
    for (int h = MB / 2; h > 0; h >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    }
    if (threadIdx.x == 0) out[blockIdx.x] = sh[0] * A.scale[blockIdx.x];
}

// The site pairs {g(a), g(c)} of one orbit: partners of each site at the
// pair's lower site, their number, and the ring distance when the orbit is
// {i, i + d} for all i (-1 otherwise).
struct Orbit {
    uint64_t mask[64] = {};
    int S = 0, ring = -1;
};

Orbit pair_orbit(const xdg_basis_s *b, int a, int c) {
    const int N = b->n_sites;
    Orbit o;
    auto add = [&](uint64_t *m, int i, int j) { m[std::min(i, j)] |= 1ull << std::max(i, j); };
    if (b->n_sym) {
        for (int g = 0; g < b->n_sym; ++g) {
            const int32_t *p = b->perm.data() + (size_t)g * N;
            add(o.mask, p[a], p[c]);
        }
    } else {
        add(o.mask, a, c);
    }
    uint64_t ring[64] = {};
    const int d = ((c - a) % N + N) % N;
    for (int i = 0; i < N; ++i) add(ring, i, (i + d) % N);
    if (std::equal(o.mask, o.mask + N, ring)) o.ring = d;
    for (int i = 0; i < N; ++i) o.S += __builtin_popcountll(o.mask[i]);
    if (a == c) std::fill(o.mask, o.mask + 64, 0ull);   // S^z_i S^z_i = 1/4: no unequal pair
    return o;
}

// One pass: np pairs into out (host).  ws: partials [PB][grid], then totals [PB].
template <bool RING>
int szsz_pass(const xdg_basis_s *b, const void *psi, int dtype, const SzPairs<RING> &A, int grid,
              double *ws, double *out, hipStream_t st) {
    double *tot = ws + (size_t)sz_pairs<RING>() * grid;
    const bool single = dtype_single(dtype), cplx = dtype_complex(dtype);
    auto go = [&](auto w, auto t) {
        using W = decltype(w);
        using T = decltype(t);
        if (cplx)
            hipLaunchKernelGGL((k_szsz<W, T, 2, RING>), dim3(grid), dim3(MB), 0, st,
                               b->reps.as<W>(), b->dim, (const T *)psi, A, ws);
        else
            hipLaunchKernelGGL((k_szsz<W, T, 1, RING>), dim3(grid), dim3(MB), 0, st,
                               b->reps.as<W>(), b->dim, (const T *)psi, A, ws);
    };
    if (b->wide) {
        if (single) go(uint64_t(), float()); else go(uint64_t(), double());
    } else {
        if (single) go(uint32_t(), float()); else go(uint32_t(), double());
    }
    XDG_TRY_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_szsz_total<RING>, dim3(A.n), dim3(MB), 0, st, ws, grid, A, tot);
    XDG_TRY_HIP(hipGetLastError());
    return copy_d2h(out, tot, sizeof(double) * A.n, st);
}

}  // namespace

int expect_szsz(xdg_basis_s *b, const void *psi, int dtype, int n_pairs, const int32_t *pairs,
                double *out, hipStream_t st) {
    if (n_pairs < 0 || (n_pairs > 0 && (!pairs || !out)) || (b->dim > 0 && n_pairs > 0 && !psi)) {
        set_error("expect_szsz: bad arguments");
        return XDG_EINVAL;
    }
    if (dtype < XDG_F64 || dtype > XDG_C64) {
        set_error("unknown dtype %d", dtype);
        return XDG_EINVAL;
    }
    if (b->is_complex && !dtype_complex(dtype)) {
        set_error("the block has complex characters: vectors must be XDG_C128 or XDG_C64");
        return XDG_EINVAL;
    }
    for (int k = 0; k < n_pairs; ++k)
        if (pairs[2 * k] < 0 || pairs[2 * k] >= b->n_sites || pairs[2 * k + 1] < 0 ||
            pairs[2 * k + 1] >= b->n_sites) {
            set_error("pair %d = (%d, %d) outside [0, %d)", k, pairs[2 * k], pairs[2 * k + 1],
                      b->n_sites);
            return XDG_EINVAL;
        }
    if (n_pairs == 0) return XDG_OK;
    if (b->dim == 0) {
        std::fill(out, out + n_pairs, 0.0);
        return XDG_OK;
    }
    const int N = b->n_sites;
    const int grid = (int)std::min<int64_t>((b->dim + MB - 1) / MB, (int64_t)device_cu_count() * 4);
    // partials and totals live with the basis (at most 132 KB); one call at a time uses them
    std::lock_guard<std::mutex> lock(b->measure_mu);
    const size_t ws_bytes = sizeof(double) * PB_RING * ((size_t)grid + 1);
    if (b->measure_ws.bytes < ws_bytes) XDG_RETURN_IF(b->measure_ws.alloc(ws_bytes));
    double *ws = b->measure_ws.as<double>();
    SzPairs<true> R{};
    SzPairs<false> M{};
    R.N = M.N = N;
    int ring_at[PB_RING], mask_at[PB_SITE];   // output positions of the pass's pairs
    double got[PB_RING];
    for (int k = 0; k <= n_pairs; ++k) {
        const bool last = k == n_pairs;
        if (R.n == PB_RING || (last && R.n)) {
            XDG_RETURN_IF(szsz_pass<true>(b, psi, dtype, R, grid, ws, got, st));
            for (int e = 0; e < R.n; ++e) out[ring_at[e]] = got[e];
            R.n = 0;
        }
        if (M.n == PB_SITE || (last && M.n)) {
            XDG_RETURN_IF(szsz_pass<false>(b, psi, dtype, M, grid, ws, got, st));
            for (int e = 0; e < M.n; ++e) out[mask_at[e]] = got[e];
            M.n = 0;
        }
        if (last) break;
        const Orbit o = pair_orbit(b, pairs[2 * k], pairs[2 * k + 1]);
        if (o.ring >= 0) {
            ring_at[R.n] = k;
            R.d[R.n] = o.ring;
            R.scale[R.n++] = 0.25 / N;
        } else {
            mask_at[M.n] = k;
            M.S[M.n] = o.S;
            M.scale[M.n] = 0.25 / o.S;
            M.sites[M.n] = 0;
            for (int a = 0, e = 0; a < N; ++a)
                if (o.mask[a]) {
                    M.sites[M.n] |= 1ull << a;
                    M.mask[M.n][e++] = o.mask[a];
                }
            ++M.n;
        }
    }
    return XDG_OK;
}

}  // namespace xdg

// ---------------------------------------------------------------------------
// Diagonal one-site operators between blocks (the operator at a momentum of
// Sec. 3.13, used for dynamical structure factors, Sec. 4.4):
//   O = sum_j c_j S^z_j.  If c is covariant, c_{g^-1(i)} = mu(g) c_i with
//   mu(g) = chi_in(g) / chi_out(g), then O maps the symmetric state of
//   representative s in the input block to o(s) times the symmetric state of
//   s in the output block, o(s) = sum_j c_j sz_s(j) (zero when s has no state
//   in the output block).  y[r] = o(s_r) x[idx_in(s_r)] over the output rows.
namespace xdg {
namespace {

constexpr int TB = 512;          // threads per block of the transfer
constexpr int TCB = 8;           // sites per chunk of the o(s) tables

struct TransferArgs {
    double2 c[64];
    int N, n_up, u1;
    const uint2 *rwords;         // index of the input block (see k_lookup)
    uint64_t n_rwords;
    const void *rtab;
    uint32_t rtab_words;         // 4-byte words of rtab
    RankLayout L;
    const void *hash;
    uint64_t n_lines, empty;
};

// One lane per output row: o(s) from tables of c over 8-site chunks, the
// row's position in the input block, one product.  The tables (and the rank
// tables of the index) sit in LDS, built once per block; rows ascend in both
// blocks, so x is read almost in order and the pass streams reps, index
// words, x and y.  Before, the states were widened to 8 bytes, looked up
// into an array of positions and multiplied in three passes with their own
// allocations and waits (ring N = 30, complex FP64, 5.2 M rows: 85 us of
// kernels in a call of about 400 us).
template <class W, class T, bool CPLX>
__global__ __launch_bounds__(TB) void k_diag_transfer(const W *reps_out, int64_t dim_out,
                                                      TransferArgs A, const T *x, T *y) {
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *tab = reinterpret_cast<double2 *>(smem);
    const int nc = (A.N + TCB - 1) / TCB;
    for (int e = threadIdx.x; e < nc << TCB; e += TB) {
        const int k = e >> TCB, v = e & ((1 << TCB) - 1);
        double2 o = make_double2(0.0, 0.0);
        for (int q = 0; q < TCB && k * TCB + q < A.N; ++q) {
            const double sz = ((v >> q) & 1) ? 0.5 : -0.5;
            o.x = __builtin_fma(A.c[k * TCB + q].x, sz, o.x);
            o.y = __builtin_fma(A.c[k * TCB + q].y, sz, o.y);
        }
        tab[e] = o;
    }
    uint32_t *rt = reinterpret_cast<uint32_t *>(tab + ((size_t)nc << TCB));
    for (uint32_t e = threadIdx.x; e < A.rtab_words; e += TB)
        rt[e] = gld(static_cast<const uint32_t *>(A.rtab) + e);
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * TB;
    for (int64_t r = (int64_t)blockIdx.x * TB + threadIdx.x; r < dim_out; r += stride) {
        const W s = gld(reps_out + r);
        int64_t q = r;   // no group: the two blocks are the same list
        if (!A.u1) {
            if (A.n_rwords)
                q = rank_find(A.rwords, A.n_rwords, colex_rank<W>(rt, A.L, s));
            else
                q = A.n_lines ? hash_find<W>(A.hash, A.n_lines, (W)A.empty, s) : -1;
        }
        double orr = 0.0, oi = 0.0;
        for (int k = 0; k < nc; ++k) {
            const double2 t = tab[(k << TCB) | ((uint32_t)(s >> (k * TCB)) & 255u)];
            orr += t.x;
            oi += t.y;
        }
        if constexpr (CPLX) {
            double yr = 0.0, yi = 0.0;
            if (q >= 0) {
                const double xr = (double)gld(x + 2 * q), xi = (double)gld(x + 2 * q + 1);
                yr = orr * xr - oi * xi;
                yi = orr * xi + oi * xr;
            }
            gst(y + 2 * r, (T)yr);
            gst(y + 2 * r + 1, (T)yi);
        } else {
            gst(y + r, q >= 0 ? (T)(orr * (double)gld(x + q)) : T(0));
        }
    }
}

}  // namespace

int apply_diag_transfer(xdg_basis_s *bin, xdg_basis_s *bout, const double *coef, const void *x,
                        void *y, int dtype, hipStream_t st) {
    if (!coef || (bout->dim > 0 && (!y || (!x && bin->dim > 0))) || x == y) {
        set_error("diag transfer: bad arguments");
        return XDG_EINVAL;
    }
    if (dtype < XDG_F64 || dtype > XDG_C64) {
        set_error("unknown dtype %d", dtype);
        return XDG_EINVAL;
    }
    const int N = bin->n_sites;
    if (bout->n_sites != N || bout->n_up != bin->n_up || bout->n_sym != bin->n_sym ||
        bout->perm != bin->perm) {
        set_error("diag transfer: the blocks need the same sites, n_up and group");
        return XDG_EINVAL;
    }
    bool coef_cplx = false;
    for (int j = 0; j < N; ++j) coef_cplx |= std::fabs(coef[2 * j + 1]) > 0.0;
    const bool cplx = dtype_complex(dtype);
    if (!cplx && (coef_cplx || bin->is_complex || bout->is_complex)) {
        set_error("diag transfer: complex coefficients or blocks need XDG_C128 / XDG_C64");
        return XDG_EINVAL;
    }
    // covariance: c_{g^-1(i)} = mu(g) c_i with mu(g) = chi_in(g) / chi_out(g)
    if (bin->n_sym) {
        double cmax = 0.0;
        for (int j = 0; j < N; ++j) cmax = std::max(cmax, std::hypot(coef[2 * j], coef[2 * j + 1]));
        const double inv_scale = 1.0 / std::max(1.0, cmax);
        std::vector<int> inv(N);
        for (int g = 0; g < bin->n_sym; ++g) {
            const std::complex<double> ci(bin->chi[2 * g], bin->chi[2 * g + 1]);
            const std::complex<double> co(bout->chi[2 * g], bout->chi[2 * g + 1]);
            const std::complex<double> mu = ci / co;
            for (int i = 0; i < N; ++i) inv[bin->perm[(size_t)g * N + i]] = i;
            for (int i = 0; i < N; ++i) {
                const std::complex<double> a(coef[2 * inv[i]], coef[2 * inv[i] + 1]);
                const std::complex<double> b(coef[2 * i], coef[2 * i + 1]);
                if (std::norm((a - mu * b) * inv_scale) > 1e-24) {
                    set_error("diag transfer: coefficients do not carry the character ratio of "
                              "the two blocks (element %d, site %d)", g, i);
                    return XDG_ENOTSYM;
                }
            }
        }
    }
    const int64_t Dout = bout->dim;
    if (Dout == 0) return XDG_OK;
    TransferArgs A{};
    for (int j = 0; j < N; ++j) A.c[j] = make_double2(coef[2 * j], coef[2 * j + 1]);
    A.N = N;
    A.u1 = bout->plan.kind == K_U1;
    if (!A.u1 && bin->dim > 0) {
        A.rwords = bin->rwords.as<uint2>();
        A.n_rwords = bin->n_rwords;
        A.rtab = bin->rtab.p;
        A.rtab_words = bin->n_rwords ? (uint32_t)(bin->rtab.bytes / 4) : 0;
        A.L = bin->rank;
        A.hash = bin->hash.p;
        A.n_lines = bin->hidx.n_lines;
        A.empty = bin->n_up == N ? 0ull : ~0ull;
    }
    const size_t lds = ((size_t)((N + TCB - 1) / TCB) << TCB) * sizeof(double2) + 4 * (size_t)A.rtab_words;
    const int grid = (int)std::min<int64_t>((Dout + TB - 1) / TB, (int64_t)device_cu_count() * 2);
    auto go = [&](auto w) -> int {
        using W = decltype(w);
        const W *reps = bout->reps.as<W>();
        auto launch = [&](auto f, auto t) -> int {
            using T = decltype(t);
            if (lds > 65536)
                XDG_TRY_HIP(hipFuncSetAttribute((const void *)f,
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)lds));
            hipLaunchKernelGGL(f, dim3(grid), dim3(TB), lds, st, reps, Dout, A, (const T *)x,
                               (T *)y);
            XDG_TRY_HIP(hipGetLastError());
            return XDG_OK;
        };
        switch (dtype) {
            case XDG_F64: return launch(k_diag_transfer<W, double, false>, double());
            case XDG_F32: return launch(k_diag_transfer<W, float, false>, float());
            case XDG_C128: return launch(k_diag_transfer<W, double, true>, double());
            default: return launch(k_diag_transfer<W, float, true>, float());
        }
    };
    XDG_RETURN_IF(bout->wide ? go(uint64_t()) : go(uint32_t()));
    XDG_TRY_HIP(hipStreamSynchronize(st));
    return XDG_OK;
}

}  // namespace xdg
