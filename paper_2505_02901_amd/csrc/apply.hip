// Host side of the matrix-free application: sector descriptors, launch
// shapes, the autotuner, the batched persistent launch and nnz counting.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "apply_impl.hpp"

namespace xdg {

size_t lds_limit();

// dynamic LDS available to the apply kernels: the device limit minus the
// static shared data (sector descriptor, tile counter)
static size_t lds_budget() {
    const size_t stat = sizeof(SectorDesc) + 64;
    return lds_limit() > stat ? lds_limit() - stat : 0;
}

// two workgroups of the apply kernel fit in one CU's LDS: run the variant
// limited to 64 VGPRs (8 waves per SIMD)
static int occ_for(size_t lds) {
    const size_t stat = sizeof(SectorDesc) + 64;
    return 2 * (lds + stat) <= lds_limit() ? 1 : 0;
}

size_t dtype_size(int dtype) {
    switch (dtype) {
        case XDG_F64: return 8;
        case XDG_F32: return 4;
        case XDG_C128: return 16;
        case XDG_C64: return 8;
    }
    return 0;
}
bool dtype_complex(int dtype) { return dtype == XDG_C128 || dtype == XDG_C64; }
bool dtype_single(int dtype) { return dtype == XDG_F32 || dtype == XDG_C64; }

// persistent apply grid of `mult` 1024-lane equivalents per compute unit
int apply_grid_for(int mult) { return device_cu_count() * mult * BLOCKS_PER_1024; }

namespace {

int launch_dispatch(int kind, bool wide, bool single, bool acc64, bool cplx, int nv,
                    const ApplyArgs &A, unsigned grid, unsigned block, size_t lds, hipStream_t st) {
    switch (kind) {
        case K_U1:
            return launch_kind<K_U1>(wide, single, acc64, cplx, nv, A, grid, block, lds, st);
        case K_AFF:
            return launch_kind<K_AFF>(wide, single, acc64, cplx, nv, A, grid, block, lds, st);
        case K_SUB:
            return launch_kind<K_SUB>(wide, single, acc64, cplx, nv, A, grid, block, lds, st);
        case K_TAB:
            return launch_kind<K_TAB>(wide, single, acc64, cplx, nv, A, grid, block, lds, st);
    }
    set_error("unknown search kind %d", kind);
    return XDG_EINVAL;
}

// The sector the products run in.
const xdg_basis_s *product_basis(const xdg_ham_s *h, const Relabelled *in) {
    return in ? in->basis.get() : h->basis;
}

SectorDesc make_desc(const xdg_ham_s *h, const Relabelled *in, bool single, const void *x,
                     void *y) {
    const xdg_basis_s *b = product_basis(h, in);
    const BondSet &bonds = in ? h->inner_bonds : h->bonds;
    SectorDesc d{};
    d.umap = in ? in->umap.as<uint32_t>() : nullptr;
    d.reps = b->reps.p;
    d.stab = b->stab.as<uint16_t>();
    d.dim = b->dim;
    d.hash = b->hash.p;
    d.n_lines = b->hidx.n_lines;
    d.empty = b->wide ? (b->n_up == b->n_sites ? 0ull : ~0ull)
                      : (b->n_up == b->n_sites ? 0ull : 0xFFFFFFFFull);
    d.lin = b->lin.as<uint32_t>();
    d.nlo = b->lin_nlo;
    d.rwords = b->n_rwords ? b->rwords.as<uint2>() : nullptr;
    d.n_rwords = b->n_rwords;
    d.rtab = b->rtab.p;
    d.rl = b->rank;
    d.n_up = b->n_up;
    d.n_sites = b->n_sites;
    d.n_sym = b->n_sym;
    d.n_bonds = h->n_bonds;
    d.aff = b->t_aff.as<AffineElem>();
    d.ring = b->plan.ring;
    d.ring_gidx = b->t_ring.as<int16_t>();
    d.bytetab = b->t_bytes.as<uint64_t>();
    d.n_bchunks = b->plan.bytes.n_chunks;
    d.mintop = b->t_mintop.as<uint16_t>();
    d.cand_off = b->t_candoff.as<uint32_t>();
    d.cand_list = b->t_candlist.as<uint16_t>();
    d.sp = b->t_pid.as<uint32_t>();
    d.tperm = b->t_tperm.as<uint16_t>();
    d.n_s = b->plan.sub.n_s;
    d.m = b->plan.sub.m;
    d.pb = b->plan.sub.pb;
    d.n_perm = b->plan.sub.n_perm;
    d.n_cand = (uint32_t)b->plan.sub.cand_list.size();
    d.subf = b->plan.kind == K_SUB && b->plan.sub.packed() && bonds.x.p;
    d.pk_tab = b->t_pktab.as<uint32_t>();
    d.pk_cand = b->t_pkcand.as<uint16_t>();
    d.n_pk = (uint32_t)b->plan.sub.pk_cand.size();
    d.pk_nb = b->plan.sub.pk_nb;
    d.bx = d.subf ? bonds.x.as<BondX>() : nullptr;
    d.bonds = single ? bonds.f.p : bonds.d.p;
    d.chi = single ? b->chi_f.p : b->chi_d.p;
    d.sqrtt = single ? b->sqrt_f.p : b->sqrt_d.p;
    double jq = 0.0;
    for (double j : h->jz) jq += 0.25 * j;
    d.jz_quarter = jq;
    d.ring_bonds = bonds.ring;
    d.ring_eq = bonds.ring_eq;
    d.chi_one = b->chi_trivial;
    d.u1_adj = b->u1_adj.as<uint32_t>();
    if (h->u1_rtab.p) {
        d.u1 = U1_RANK;
        d.rtab = h->u1_rtab.p;
        d.rl = h->u1_rank;
    }
    d.x = x;
    d.y = y;
    return d;
}

// Real-valued kernels serve complex vectors on a real block: the real and
// imaginary parts are independent columns of a [dim][2 nvec] real block.
struct Form {
    bool single, cplx_kernel;
    bool acc64;     // FP64 amplitudes and row accumulation
    bool tsingle;   // FP32 amplitude tables (single && !acc64)
    int64_t cols;   // columns seen by the kernel
};

int form_of(const xdg_basis_s *b, int dtype, int64_t nvec, Form *f) {
    if (dtype < XDG_F64 || dtype > XDG_C64) {
        set_error("unknown dtype %d", dtype);
        return XDG_EINVAL;
    }
    if (nvec < 1) {
        set_error("nvec = %lld must be >= 1", (long long)nvec);
        return XDG_EINVAL;
    }
    if (b->is_complex && !dtype_complex(dtype)) {
        set_error("the block (dimension %lld, %d group elements) has complex characters: "
                  "vectors must be XDG_C128 or XDG_C64 (got dtype %d)",
                  (long long)b->dim, b->n_sym, dtype);
        return XDG_EINVAL;
    }
    f->single = dtype_single(dtype);
    f->cplx_kernel = b->is_complex;
    f->acc64 = !f->single || !(b->plan.flags & XDG_FLAG_F32_ACCUMULATE);
    f->tsingle = f->single && !f->acc64;
    f->cols = (dtype_complex(dtype) && !b->is_complex) ? 2 * nvec : nvec;
    return XDG_OK;
}

// Rank-addressed x: row i of x (spr scalars) goes to the slot of reps[i]
// (block_slot in the packed form, top_rank otherwise) of xr (`slot` scalars
// apart); the other slots hold zeros.
template <class W, class T>
__global__ __launch_bounds__(256) void k_xr_scatter(const W *reps, int64_t dim, int spr, int slot,
                                                   const T *x, T *xr, const uint32_t *rtab,
                                                   RankLayout L, int B, const uint64_t *top,
                                                   uint64_t slots, const uint32_t *umap,
                                                   const uint32_t *xb_ent, const uint32_t *xb_off,
                                                   const uint2 *xb_top) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < dim; i += stride) {
        const W s = reps[i];
        const uint64_t r = xb_ent ? block_slot(xb_ent, xb_off, xb_top, B / 3, (uint32_t)(s >> B),
                                               (uint32_t)s & ((1u << B) - 1u))
                                  : top_rank<W>(rtab, L, B, top, s);
        if (r >= slots) continue;   // never for a basis state
        if (umap) {                 // relabelled sector: the caller's position and sign
            const uint32_t u = gld(umap + i);
            const int64_t p = (int64_t)(u & 0x7FFFFFFFu);
            for (int c = 0; c < spr; ++c) {
                const T v = x[p * spr + c];
                xr[r * slot + c] = u >> 31 ? -v : v;
            }
            continue;
        }
        for (int c = 0; c < spr; ++c) xr[r * slot + c] = x[i * spr + c];
    }
}

__global__ __launch_bounds__(256) void k_zero32(uint32_t *p, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) p[i] = 0u;
}

// Columns of a slot of the rank-addressed x: up to eight are padded to a power
// of two, so that a slot lies in one cache line (the padding is never used).
int xr_columns(int64_t cols) {
    int n = 1;
    while (n < cols) n *= 2;
    return cols <= 8 ? n : (int)cols;
}

// Fill the rank-addressed copy of x for this call (caller holds h->xr_mu):
// wait for the last launch that read it, (re)allocate and zero it when the
// layout changes (not under graph capture), then scatter x.
// columns: those of a slot (f.cols itself where a padded copy finds no room).
int xr_prepare(xdg_ham_s *h, const Relabelled *in, const void *x, const Form &f, hipStream_t st,
               bool *capturing, int *columns) {
    const xdg_basis_s *b = product_basis(h, in);
    const uint32_t *umap = in ? in->umap.as<uint32_t>() : nullptr;
    const int spr = (int)f.cols * (f.cplx_kernel ? 2 : 1);
    const size_t tsz = f.single ? 4 : 8;
    int slot = xr_columns(f.cols) * (f.cplx_kernel ? 2 : 1);   // scalars
    size_t slot_bytes = (size_t)slot * tsz, need = (size_t)b->xr_slots * slot_bytes;
    auto unpadded = [&] {
        slot = spr;
        slot_bytes = (size_t)slot * tsz;
        need = (size_t)b->xr_slots * slot_bytes;
    };
    if (h->xr_of == b && h->xr_slot_bytes == (size_t)spr * tsz) unpadded();   // as before
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    XDG_TRY_HIP(hipStreamIsCapturing(st, &cs));
    *capturing = cs != hipStreamCaptureStatusNone;
    if (!h->xr_ev) XDG_TRY_HIP(hipEventCreateWithFlags(&h->xr_ev, hipEventDisableTiming));
    if (!*capturing) XDG_TRY_HIP(hipStreamWaitEvent(st, h->xr_ev, 0));
    const int gcap = device_cu_count() * 32;
    if (h->xr_buf.bytes < need || h->xr_slot_bytes != slot_bytes || h->xr_of != b) {
        if (*capturing) {
            set_error("the rank-addressed copy of x is set up by a first call outside graph capture");
            return XDG_EINVAL;
        }
        if (h->xr_buf.bytes < need) {
            h->xr_slot_bytes = 0;
            h->xr_buf.release();   // waits for the device
            const std::string before = get_error();
            int rc = h->xr_buf.alloc(need);
            if (rc == XDG_ENOMEM && slot != spr) {
                unpadded();
                rc = h->xr_buf.alloc(need);
                if (rc == XDG_OK) set_error("%s", before.c_str());
            }
            XDG_RETURN_IF(rc);
        }
        const uint64_t nw = need / 4;
        const unsigned g = (unsigned)std::min<uint64_t>((nw + 255) / 256, (uint64_t)gcap);
        hipLaunchKernelGGL(k_zero32, dim3(std::max(1u, g)), dim3(256), 0, st,
                           h->xr_buf.as<uint32_t>(), nw);
        XDG_TRY_HIP(hipGetLastError());
        h->xr_slot_bytes = slot_bytes;
        h->xr_of = b;
    }
    *columns = slot / (f.cplx_kernel ? 2 : 1);
    const unsigned g =
        (unsigned)std::min<int64_t>((b->dim + 255) / 256, (int64_t)gcap);
    const uint64_t *top = b->xr_top.as<uint64_t>();
    if (b->wide) {
        if (f.single)
            hipLaunchKernelGGL((k_xr_scatter<uint64_t, float>), dim3(g), dim3(256), 0, st,
                               b->reps.as<uint64_t>(), b->dim, spr, slot, (const float *)x,
                               h->xr_buf.as<float>(), b->xr_rtab.as<uint32_t>(), b->rank,
                               b->xr_bits, top,
                               b->xr_slots, umap, b->xb_ent.as<uint32_t>(),
                               b->xb_off.as<uint32_t>(), b->xb_top.as<uint2>());
        else
            hipLaunchKernelGGL((k_xr_scatter<uint64_t, double>), dim3(g), dim3(256), 0, st,
                               b->reps.as<uint64_t>(), b->dim, spr, slot, (const double *)x,
                               h->xr_buf.as<double>(), b->xr_rtab.as<uint32_t>(), b->rank,
                               b->xr_bits, top,
                               b->xr_slots, umap, b->xb_ent.as<uint32_t>(),
                               b->xb_off.as<uint32_t>(), b->xb_top.as<uint2>());
    } else {
        if (f.single)
            hipLaunchKernelGGL((k_xr_scatter<uint32_t, float>), dim3(g), dim3(256), 0, st,
                               b->reps.as<uint32_t>(), b->dim, spr, slot, (const float *)x,
                               h->xr_buf.as<float>(), b->xr_rtab.as<uint32_t>(), b->rank,
                               b->xr_bits, top,
                               b->xr_slots, umap, b->xb_ent.as<uint32_t>(),
                               b->xb_off.as<uint32_t>(), b->xb_top.as<uint2>());
        else
            hipLaunchKernelGGL((k_xr_scatter<uint32_t, double>), dim3(g), dim3(256), 0, st,
                               b->reps.as<uint32_t>(), b->dim, spr, slot, (const double *)x,
                               h->xr_buf.as<double>(), b->xr_rtab.as<uint32_t>(), b->rank,
                               b->xr_bits, top,
                               b->xr_slots, umap, b->xb_ent.as<uint32_t>(),
                               b->xb_off.as<uint32_t>(), b->xb_top.as<uint2>());
    }
    XDG_TRY_HIP(hipGetLastError());
    return XDG_OK;
}

// Vectors of the next pass: a kernel exists for every number up to 8, so that
// three vectors share one search (two passes of 2 and 1 took 10.7 ms on the
// 6x6 triangular lattice, 12 of 36 up, FP64).
int pick_nv(int64_t remaining, int cap) { return (int)std::min<int64_t>(remaining, cap); }

}  // namespace

// The few-rows loop serves blocks (or batches) below a line.  Its time grows
// with the rows from the first on; the row loop takes the time of one lane's
// chain, which the terms of a row make long: those touch at most the
// min(n_up, n_down) sites of the rarer spin.  So the line is in rows times
// n_sites / min(n_up, n_down) (twice the rows at half filling), and higher
// where a search is longer (a second scan for reflections; the packed and the
// byte-table searches by the group's size) and, since the row loop searches
// once per eight vectors, where there are more of those; it is lower where a
// wave holds the terms of a single row (more than 64 bonds).  Measured, FP64,
// one vector, row loop against few-rows loop (us), the line's number behind:
//   rings: N = 22, 11 up 21.9 and 19.4 (64 K), N = 23, 11 up 23.7 and 24.7 (123 K);
//     N = 28, 6 and 7 up 15.1 and 11.8 (63 K), 17.6 and 25.9 (169 K); N = 48, 5 up
//     23.7 and 69.9 (342 K); next neighbours too: N = 22, 11 up 52.5 and 45.0 (64 K),
//     N = 32, 6 up 31.6 and 55.1 (151 K), N = 36, 5 up 49.8 and 55.3 (75 K);
//     with eight vectors N = 23, 11 up 31.3 and 25.1 (123 K), N = 28, 7 up 24.1 and
//     25.8 (169 K), complex N = 25, 9 up 76.9 and 46.7 (227 K), N = 36, 6 up 61 and
//     73 (324 K);
//   rings with reflections: N = 24, 12 up 36.6 and 30.8 (114 K), N = 25, 12 up 40.7
//     and 54.8 (209 K), N = 40, 6 up 38.3 and 63.0 (324 K);
//   4x6 square, 48 elements: 48 bonds 151 and 117 (114 K), 96 bonds 208 and 166
//     (74 K), 224 and 253 (100 K); 24 elements, 96 bonds 169 and 284 (145 K);
//   6x6 square, 36 elements: 210 and 69 (75 K), 192 and 276 (325 K); 288 elements:
//     897 and 782 (483 K); 40 sites, 160 elements: 469 and 821 (667 K);
//   6x6 triangular, three blocks (packed inside): 916 and 403 (199 K), 877 and 1292
//     (633 K); 27 sites by blocks: 824 and 296 (87 K), 586 and 790 (258 K).
// Without a group a term is too cheap to share out (184756 rows: 41 against
// 13 us).
static int64_t few_line(const xdg_basis_s *b, int n_bonds, int64_t cols, bool cplx) {
    if (b->plan.kind == K_U1) return 0;
    const int64_t passes = std::min<int64_t>(8, (cols + 7) / 8);
    if (b->plan.kind == K_AFF) {
        // (its searches are short enough for the gathers of many vectors to count)
        const bool twice = b->plan.ring == 2;
        const int64_t gathers = cols < 8 || twice ? 100 : cplx ? 250 : 160;
        return std::max(100 * passes, gathers) * (n_bonds > 64 ? 400 : 750) * (twice ? 2 : 1);
    }
    const bool by_group = b->plan.kind == K_TAB || b->plan.sub.packed();
    return passes * std::min<int64_t>(500000, (n_bonds > 64 && !b->wide ? 90000 : 150000) *
                                                  (int64_t)(by_group ? std::max(1, b->n_sym / 32) : 1));
}
static int64_t few_weight(const xdg_basis_s *b) {
    return b->dim * b->n_sites / std::max(1, std::min(b->n_up, b->n_sites - b->n_up));
}
// Rows so short that the row loop's chain ends before the few-rows loop has staged
// its tables (one wave a workgroup does that there): thin fillings of rings and of
// groups of shifts and mirrors.  `terms`: what a row has at most; both loops' times
// are about linear in it, in the sites and in the length of a search, and the line
// below is where the fits cross.  Measured, FP64, row loop against few-rows loop (us):
//   rings, one vector: 2 up 5.9 and 7.8 (N = 16), 5.8 and 11.2 (32), 8.7 and 15.0
//     (40); 3 up 7.4 and 8.2 (12), 7.3 and 12.6 (32); 4 up 9.3 and 9.2 (16), 9.9 and
//     11.6 (24), 10.8 and 11.4 (32); N = 28, 6 up 15.1 and 11.8; next neighbours
//     too: 2 up 11.7 and 14.4 (32); eight vectors: 3 up 8.4 and 12.6 (32, 155 rows),
//     4 up 14.9 and 13.6 (28, 735 rows), 17.6 and 10.5 (32, 1128 rows);
//   with reflections: 3 up 9.3 and 10.9 (20), 4 up 11.9 and 12.5 (24);
//   mirror: 2 up 5.7 and 6.4 (8), 3 up 6.9 and 6.4 (8), 7.5 and 8.7 (16), 8.7 and 11.6
//     (32), 15.4 and 11.4 (40), 4 up 10.4 and 9.0 (20);
//   8 shifts: 2 up 8.6 and 9.5 (16), 3 up 11.2 and 10.1 (16), 12.1 and 14.1 (32).
static bool short_rows(const xdg_basis_s *b, const BondSet &bonds, int n_bonds, int64_t cols,
                       bool cplx) {
    if (b->plan.kind != K_AFF) return false;
    const int N = b->n_sites, ring = b->plan.ring;
    const int64_t terms = 2 * (int64_t)n_bonds * std::min(b->n_up, N - b->n_up) / N;
    const int64_t most = (ring ? 8 : 6) - (b->wide ? 2 : 0);
    if (terms > most || b->dim * (cols * (cplx ? 2 : 1) - 1) > 3000) return false;
    const int search = ring == 2 ? 10 : ring ? 8 : 6 + b->n_sym;   // a term's, in tenths of us
    const int64_t row = terms * ((b->wide ? search * 3 / 2 : search) - 4) +
                        (bonds.ring ? 0 : n_bonds / 3);
    const int64_t few = ring ? 8 + 8 * N / 5 : 2 + 8 * N / 5 + 2 * b->n_sym;
    return row < few;
}
bool below_few_line(const xdg_basis_s *b) { return few_weight(b) < few_line(b, 0, 1, false); }

// Blocks without a group: is an exchange of sites that are not neighbouring
// numbers rare (at most one bond in eight)?
static bool u1_near(const xdg_ham_s *h) { return 8 * h->bonds.far <= h->n_bonds; }

// Far exchanges of blocks without a group go through rank tables in LDS where
// staging them pays and the state has 32 bits; otherwise through Lin's tables.
// Measured, FP64, one vector, Lin against rank tables: 4x6 square, 12 up, 2.7 M
// rows 127 and 121 us; 5x6, 10 up, 30 M rows 1.74 and 1.48 ms; 4x6, 7 up, 0.35 M
// rows 21 and 23 us; 4x4, 8 up 10.7 and 15.1 us; 6x6, 8 up (64-bit states) 2.14
// and 2.75 ms.
bool u1_wants_rank(const xdg_ham_s *h) {
    const xdg_basis_s *b = h->basis;
    return !u1_near(h) && !b->wide && b->dim >= 1 << 19;
}

static size_t bond_bytes(const xdg_ham_s *h) { return a16(sizeof(BondD) * (size_t)h->n_bonds); }

// Which loop a product without a group takes: all lanes on one bond
// (process_row_u1), or each lane on its own (process_row_own).  The first reads
// x in order and holds several gathers in flight, but takes every bond, also
// those whose spins are equal in most rows; so it needs a filling where a bond's
// spins differ often enough.  `unequal`: percent of the rows in which they do.
// Measured against the loop over own bonds (times it needs over the other's):
//   rings, FP64, 1 vector: 1.80 at 52 % (N = 24), 1.34 at 35 % (32, 7 up), 1.01 at
//     29 % (36, 6 up), 0.93 at 22 % (40, 5 up); 4 vectors 1.52, 1.20, 1.00, 0.83;
//     8 vectors 1.22 at 52 % (28, 14 up), 1.10 at 44 % (32, 10 up), 0.79 at 35 %;
//   FP32, 1 vector: 1.08 at 35 %, 0.99 at 32 % (36, 7 up); 8 vectors: 1.23 at 52 %
//     (24), 1.06 at 39 % (36, 9 up), 0.90 at 35 %;
//   square lattices, rank tables, FP64, 1 vector: 1.19 at 40 % (5x6, 8 up), 1.07 at
//     37 % (5x6, 7 up), 0.92 at 31 % (4x8, 6 up); 4 vectors 1.12, 1.06, 0.89; 8
//     vectors 0.89 at 53 % (4x6); FP32, 1 vector: 1.08 at 48 % (5x5, 9 up), 0.98 at
//     40 %; 8 vectors 1.11 at 52 %, 0.95 at 44 % (4x8, 10 up);
//   64-bit states, Lin's tables (6x6): FP64, 1 vector 1.08 at 36 % (8 up), 0.97 at
//     32 %; 4 vectors 0.90 at 39 % (9 up); FP32 1.07 at 39 %, 0.97 at 36 %;
//   fewer than 2^19 rows with far bonds: 0.94 (4x6, 7 up) and less;
//   every pair of 24 sites coupled, 10 up: 0.88.
static bool u1_own(const xdg_ham_s *h, bool single, int64_t cols) {
    const xdg_basis_s *b = h->basis;
    if (b->plan.kind != K_U1 || b->n_sites < 2) return false;
    const int N = b->n_sites, n = b->n_up;
    const int unequal = 200 * n * (N - n) / (N * (N - 1));
    constexpr int never = 101;
    int least;
    if (u1_near(h))
        least = cols <= 4 ? (single ? 33 : 29) : (single ? 39 : 44);
    else if (b->dim < 1 << 19 || 6 * h->bonds.far > 5 * h->n_bonds)
        least = never;
    else if (b->wide)
        least = cols <= 2 ? (single ? 38 : 36) : never;
    else if (single)
        least = cols <= 4 ? 41 : 48;
    else
        least = cols <= 2 ? 36 : cols <= 4 ? 38 : never;
    // the own bonds are picked lane by lane from LDS
    return unequal < least && bond_bytes(h) <= lds_budget();
}

// Its shape: rows per wave (about 128 (row, bond) pairs, two for every lane),
// the workgroup, and its LDS behind `tables` bytes of staged tables.  False
// where the terms of even one wave do not fit.
static bool few_shape(int64_t rows, int n_bonds, bool cplx, bool single_acc, size_t tables,
                      int *few, int *block, size_t *lds) {
    const int nb = std::max(n_bonds, 1);
    *few = std::max(1, std::min(16, 128 / nb));
    const size_t per_wave = single_acc ? few_bytes<float>(cplx, *few * nb)
                                       : few_bytes<double>(cplx, *few * nb);
    const int64_t waves = (rows + *few - 1) / *few;
    // a workgroup per compute unit at least, as large as that leaves it; one wave
    // that is alone has the others of its workgroup stage the tables (4x6 square,
    // translations, 1 up: 57 us with none, 16 with fifteen; row loop 24)
    int w = waves > 1 ? 1 : 16;
    while (w < 16 && (int64_t)w * device_cu_count() < waves) w *= 2;
    while (w > 1 && a16(tables) + w * per_wave > lds_budget()) w /= 2;
    *block = 64 * w;
    *lds = a16(tables) + w * per_wave;
    return *lds <= lds_budget();
}

// LDS bytes the apply kernel stages for this form, whether the sublattice
// tables fit with them, and whether two workgroups fit one compute unit
void apply_lds(const xdg_ham_s *h, int dtype, size_t *lds, int *stage_sub, int *occ_ok) {
    const RelabelledRef in = relabelled(h, nullptr);
    const xdg_basis_s *b = product_basis(h, in.get());
    const bool tsingle = dtype_single(dtype) && (b->plan.flags & XDG_FLAG_F32_ACCUMULATE);
    const SectorDesc d = make_desc(h, in.get(), tsingle, nullptr, nullptr);
    size_t n = tsingle ? stage_bytes<float>(d, b->plan.kind, 1)
                       : stage_bytes<double>(d, b->plan.kind, 1);
    int st = 1;
    if (n > lds_budget()) {
        st = 0;
        n = tsingle ? stage_bytes<float>(d, b->plan.kind, 0) : stage_bytes<double>(d, b->plan.kind, 0);
    }
    *lds = n;
    *stage_sub = st;
    *occ_ok = st ? occ_for(n) : 0;
}

bool tables_fit(const xdg_ham_s *h, const Relabelled *in) {
    return stage_bytes<double>(make_desc(h, in, false, nullptr, nullptr),
                               product_basis(h, in)->plan.kind, 0) <= lds_budget();
}

int apply_launch(xdg_ham_s *h, const void *x, void *y, int64_t nvec, int dtype, hipStream_t st,
                 const LaunchCfg *cfg) {
    const RelabelledRef in = relabelled(h, st);
    const xdg_basis_s *b = product_basis(h, in.get());
    Form f;
    XDG_RETURN_IF(form_of(b, dtype, nvec, &f));
    if (b->dim == 0) return XDG_OK;
    if (!x || !y || x == y) {
        set_error("x and y must be distinct non-null device pointers");
        return XDG_EINVAL;
    }
    LaunchCfg c = cfg ? *cfg : LaunchCfg{};
    const unsigned block = APPLY_BLOCK;
    const int64_t need = (b->dim + block - 1) / block;
    const int64_t gmax = c.grid > 0 ? c.grid : (int64_t)apply_grid_for(2);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(need, gmax));
    ApplyArgs A{};
    A.one = make_desc(h, in.get(), f.tsingle, x, y);
    A.own = u1_own(h, f.single, f.cols);
    if (A.own) A.one.u1 = U1_OWN;
    if (c.sub_form == 2) {
        A.one.subf = 0;
        A.one.bx = nullptr;
    }
    // rank-addressed x: when its tables fit in LDS with the others
    bool xr_on = c.xr && b->xr_slots && b->plan.kind == K_SUB, capturing = false;
    if (xr_on) {
        A.one.xr = b->reps.p;     // the copy is set below; non-null for the LDS size
        A.one.xb_ent = b->xb_ent.as<uint32_t>();
        A.one.xb_off = b->xb_off.as<uint32_t>();
        A.one.xb_top = b->xb_top.as<uint2>();
        A.one.xb_w32 = b->xr_slots <= 0xFFFFFFFFull;
        A.one.xr_top = b->xr_top.as<uint64_t>();
        A.one.xr_top32 = b->xr_top32.as<uint32_t>();
        A.one.xr_slots = b->xr_slots;
        A.one.xr_cols = xr_columns(f.cols);
        A.one.xr_bits = b->xr_bits;
        A.one.xr_rows = b->xr_rows;
        A.one.xr_rtab = b->xr_rtab.as<uint32_t>();
        const size_t lx = f.tsingle ? stage_bytes<float>(A.one, b->plan.kind, 1)
                                    : stage_bytes<double>(A.one, b->plan.kind, 1);
        if (lx > lds_budget()) {
            xr_on = false;
            A.one.xr = nullptr;
            A.one.xr_top = nullptr;
            A.one.xr_top32 = nullptr;
            A.one.xb_ent = nullptr;
        }
    }
    std::unique_lock<std::mutex> xr_lock;
    if (xr_on) {
        xr_lock = std::unique_lock<std::mutex>(h->xr_mu);
        XDG_RETURN_IF(xr_prepare(h, in.get(), x, f, st, &capturing, &A.one.xr_cols));
        A.one.xr = h->xr_buf.p;
    }
    A.nvec = f.cols;
    size_t lds = f.tsingle ? stage_bytes<float>(A.one, b->plan.kind, 1)
                           : stage_bytes<double>(A.one, b->plan.kind, 1);
    A.ring = ring_loop_ok(A.one, b->plan.kind, b->wide);
    A.stage_sub = 1;
    if (lds > lds_budget()) {
        A.stage_sub = 0;
        lds = f.tsingle ? stage_bytes<float>(A.one, b->plan.kind, 0)
                        : stage_bytes<double>(A.one, b->plan.kind, 0);
    }
    A.occ = A.stage_sub ? (c.occ >= 0 ? (c.occ && occ_for(lds)) : occ_for(lds)) : 0;
    A.compact = c.compact > 0 && !xr_on ? 1 : 0;   // the compacted loop reads x itself
    // few rows: terms shared out over the lanes (never with an explicit shape)
    int few = 0, few_block = 0;
    size_t few_lds = 0;
    if (c.few && !xr_on && A.stage_sub && f.cols < (int64_t)1 << 24 &&
        few_shape(b->dim, h->n_bonds, f.cplx_kernel, f.tsingle, lds, &few, &few_block, &few_lds)) {
        A.few = few;
        A.few_off = (uint32_t)a16(lds);
        A.occ = A.compact = 0;
        const int64_t per = (int64_t)few * (few_block / 64);
        const int64_t g = std::min<int64_t>((b->dim + per - 1) / per, 2 * (int64_t)device_cu_count());
        return launch_dispatch(b->plan.kind, b->wide, f.single, f.acc64, f.cplx_kernel, 1, A,
                               (unsigned)g, (unsigned)few_block, few_lds, st);
    }
    // fewer rows than fill the chip.  No group: nothing to stage, so workgroups
    // small enough for two on every compute unit.  Sublattice coding: one on every
    // compute unit, of at least 256 lanes, which stage the tables together (4x6
    // square, 112800 rows, FP64: 120 -> 105 us; 5x5, 104384 rows: 470 -> 418 us).
    unsigned lanes = block, groups = grid;
    if (c.small && b->plan.kind == K_U1) {
        while (lanes > 64 && b->dim < (int64_t)2 * lanes * device_cu_count()) lanes /= 2;
        groups = (unsigned)((b->dim + lanes - 1) / lanes);
    } else if (c.small && b->plan.kind == K_SUB && !xr_on) {
        while (lanes > 256 && 2 * b->dim <= (int64_t)lanes * device_cu_count()) lanes /= 2;
        groups = (unsigned)((b->dim + lanes - 1) / lanes);
    }
    const int cap = std::min(c.nv > 0 ? c.nv : 8,
                             xr_on                          ? xr_max_nv(f.cplx_kernel)
                             : A.compact && f.cols <= 3 ? 2   // the compacted loop takes two
                                                        : 8);
    for (int64_t v0 = 0; v0 < f.cols;) {
        const int nv = pick_nv(f.cols - v0, cap);
        A.v0 = (int)v0;
        if (xr_on && b->chi_trivial && !f.cplx_kernel)
            XDG_RETURN_IF(launch_sub_xr_trivial(b->wide, f.single, f.acc64, nv, A, grid, block,
                                                lds, st));
        else if (xr_on)
            XDG_RETURN_IF(launch_sub_xr(b->wide, f.single, f.acc64, f.cplx_kernel, nv, A, grid,
                                        block, lds, st));
        else
            XDG_RETURN_IF(launch_dispatch(b->plan.kind, b->wide, f.single, f.acc64,
                                          f.cplx_kernel, nv, A, groups, lanes, lds, st));
        v0 += nv;
    }
    if (xr_on && !capturing) XDG_TRY_HIP(hipEventRecord(h->xr_ev, st));
    return XDG_OK;
}

// Launch-shape autotuner, run on the first call for a (dtype, nvec) pair:
// first the persistent grid (1, 2, 4 or 8 workgroups per compute unit, or
// one row per lane) and, with several columns, the vectors per pass; then,
// at the best of those, the 8- or 4-waves-per-SIMD copy of the kernel (when
// two workgroups' LDS fit a CU) and, for the table searches, the row loop
// or the wave-compacted term loop.  Every candidate computes bitwise the
// same y, so the timing runs also leave the right y behind.  XDG_TUNE_LOG=1
// prints the timings to stderr.
static bool tune_log() {
    static int on = -1;
    if (on < 0) {
        const char *e = getenv("XDG_TUNE_LOG");
        on = e && atoi(e) > 0;
    }
    return on;
}

int apply_tuned(xdg_ham_s *h, const void *x, void *y, int64_t nvec, int dtype, hipStream_t st) {
    TuneKey key{dtype, nvec};
    std::unique_lock<std::mutex> lock(h->tune_mu);
    auto it = h->tuned.find(key);
    if (it != h->tuned.end()) {
        LaunchCfg c = it->second;
        lock.unlock();
        const int rc = apply_launch(h, x, y, nvec, dtype, st, &c);
        if (rc != XDG_ENOMEM || !c.xr) return rc;
        // the copy was set up for a labelling that has been given up, and there is
        // no room for another
        c.xr = 0;
        lock.lock();
        h->tuned[key] = c;
        lock.unlock();
        return apply_launch(h, x, y, nvec, dtype, st, &c);
    }
    const RelabelledRef in = relabelled(h, st);
    const xdg_basis_s *b = product_basis(h, in.get());
    Form f;
    XDG_RETURN_IF(form_of(b, dtype, nvec, &f));
    const int64_t need = (b->dim + APPLY_BLOCK - 1) / APPLY_BLOCK;
    if (b->dim < (int64_t)1024 * APPLY_BLOCK) {   // small blocks: one row per lane
        LaunchCfg c{APPLY_BLOCK, (int)std::min<int64_t>(need, 1 << 30), 8};
        c.small = 1;
        c.few = few_weight(b) < few_line(b, h->n_bonds, f.cols, f.cplx_kernel) &&
                !short_rows(b, in ? h->inner_bonds : h->bonds, h->n_bonds, f.cols, f.cplx_kernel);
        h->tuned[key] = c;
        return apply_launch(h, x, y, nvec, dtype, st, &c);
    }
    hipEvent_t e0, e1;
    XDG_TRY_HIP(hipEventCreate(&e0));
    XDG_TRY_HIP(hipEventCreate(&e1));
    // one warm launch, then the mean of `reps` timed launches (one for large blocks)
    const int reps = b->dim > (int64_t)200000000 ? 1 : 2;
    auto time_cfg = [&](const LaunchCfg &c, float *ms) -> int {
        XDG_RETURN_IF(apply_launch(h, x, y, nvec, dtype, st, &c));
        XDG_TRY_HIP(hipEventRecord(e0, st));
        for (int r = 0; r < reps; ++r) XDG_RETURN_IF(apply_launch(h, x, y, nvec, dtype, st, &c));
        XDG_TRY_HIP(hipEventRecord(e1, st));
        XDG_TRY_HIP(hipEventSynchronize(e1));
        XDG_TRY_HIP(hipEventElapsedTime(ms, e0, e1));
        *ms /= reps;
        if (tune_log()) {
            size_t lds = 0;
            int stg = 0, occ_ok = 0;
            apply_lds(h, dtype, &lds, &stg, &occ_ok);
            fprintf(stderr, "[xdg tune] dim %lld dtype %d nvec %lld (LDS %zu B, tables staged %d, "
                    "8-wave copy possible %d): grid %d nv %d occ %d compact %d xr %d: %.3f ms\n",
                    (long long)b->dim, dtype, (long long)nvec, lds, stg, occ_ok, c.grid, c.nv,
                    c.occ, c.compact, c.xr, *ms);
        }
        return XDG_OK;
    };
    std::vector<LaunchCfg> cands;
    const int cu = device_cu_count();
    for (int mult : {1, 2, 4, 8}) {
        const int g = cu * mult * BLOCKS_PER_1024;
        cands.push_back({APPLY_BLOCK, g, 8});
        // (a number of vectors that an explicit shape may ask for: 1, 2, 4 or 8)
        int half = 1;
        while (half < 8 && half < f.cols / 2) half *= 2;
        if (f.cols > 1 && half < 8) cands.push_back({APPLY_BLOCK, g, half});
    }
    cands.push_back({APPLY_BLOCK, (int)std::min<int64_t>(need, 1 << 30), 8});
    float best = 1e30f;
    LaunchCfg bestc = cands[0];
    int rc = XDG_OK;
    for (const LaunchCfg &c : cands) {
        float ms = 0;
        if ((rc = time_cfg(c, &ms)) != XDG_OK) break;
        if (ms < best) {
            best = ms;
            bestc = c;
        }
    }
    // second phase: kernel copy (occupancy) and, for table searches, the loop form
    if (rc == XDG_OK) {
        std::vector<LaunchCfg> more;
        const bool table = b->plan.kind == K_SUB || b->plan.kind == K_TAB;
        for (int occ : {0, 1})
            for (int cmp : {0, 1}) {
                if (cmp && !table) continue;
                LaunchCfg c = bestc;
                c.occ = occ;
                c.compact = cmp;
                more.push_back(c);
            }
        // sublattice coding: terms reading a rank-addressed copy of x
        if (b->xr_slots && b->plan.kind == K_SUB)
            for (int occ : {0, 1}) {
                LaunchCfg c = bestc;
                c.occ = occ;
                c.compact = 0;
                c.xr = 1;
                more.push_back(c);
            }
        const std::string before = get_error();
        for (const LaunchCfg &c : more) {
            float ms = 0;
            if ((rc = time_cfg(c, &ms)) != XDG_OK) {
                if (c.xr && rc == XDG_ENOMEM) {   // no room for the copy: not a candidate
                    rc = XDG_OK;
                    set_error("%s", before.c_str());
                    continue;
                }
                break;
            }
            if (ms < best) {
                best = ms;
                bestc = c;
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    XDG_RETURN_IF(rc);
    h->tuned[key] = bestc;
    bool xr_used = false;
    for (const auto &kv : h->tuned) xr_used |= kv.second.xr != 0;
    if (!xr_used) {   // free the copy no tuned shape reads
        std::lock_guard<std::mutex> g(h->xr_mu);
        h->xr_slot_bytes = 0;
        h->xr_buf.release();
    }
    return apply_launch(h, x, y, nvec, dtype, st, &bestc);
}

int apply_tuned_config(xdg_ham_s *h, int dtype, int64_t nvec, LaunchCfg *out) {
    std::lock_guard<std::mutex> lock(h->tune_mu);
    auto it = h->tuned.find(TuneKey{dtype, nvec});
    if (it == h->tuned.end()) {
        set_error("no tuned launch shape yet for dtype %d, nvec %lld (apply once first)", dtype,
                  (long long)nvec);
        return XDG_EINVAL;
    }
    *out = it->second;
    return XDG_OK;
}

int ham_count_nnz(xdg_ham_s *h, int64_t *nnz) {
    if (h->nnz >= 0) {
        *nnz = h->nnz;
        return XDG_OK;
    }
    const xdg_basis_s *b = h->basis;
    if (b->dim == 0) {
        h->nnz = 0;
        *nnz = 0;
        return XDG_OK;
    }
    DevBuf cnt;
    XDG_RETURN_IF(cnt.alloc(sizeof(unsigned long long)));
    XDG_TRY_HIP(hipMemset(cnt.p, 0, sizeof(unsigned long long)));
    ApplyArgs A{};
    // in the caller's labels: with repeated bonds the terms of a row depend on
    // which state of its orbit stands for it
    A.one = make_desc(h, nullptr, false, nullptr, nullptr);
    A.count = cnt.as<unsigned long long>();
    A.stage_sub = 1;
    size_t lds = stage_bytes<double>(A.one, b->plan.kind, 1);
    if (lds > lds_budget()) {
        A.stage_sub = 0;
        lds = stage_bytes<double>(A.one, b->plan.kind, 0);
    }
    const unsigned block = APPLY_BLOCK;
    const unsigned grid =
        (unsigned)std::min<int64_t>((b->dim + block - 1) / block, (int64_t)apply_grid_for(2));
    int rc;
    switch (b->plan.kind) {
        case K_U1: rc = launch_count_kind<K_U1>(b->wide, A, grid, block, lds, 0); break;
        case K_AFF: rc = launch_count_kind<K_AFF>(b->wide, A, grid, block, lds, 0); break;
        case K_SUB: rc = launch_count_kind<K_SUB>(b->wide, A, grid, block, lds, 0); break;
        default: rc = launch_count_kind<K_TAB>(b->wide, A, grid, block, lds, 0); break;
    }
    XDG_RETURN_IF(rc);
    unsigned long long c = 0;
    XDG_RETURN_IF(copy_d2h(&c, cnt.p, sizeof c, nullptr));
    h->nnz = b->dim + (int64_t)c;
    *nnz = h->nnz;
    return XDG_OK;
}

static bool runs_packed(const xdg_ham_s *h, const Relabelled *in) {
    const xdg_basis_s *b = product_basis(h, in);
    return b->plan.kind == K_SUB && b->plan.sub.packed();
}

// One part of a batch: the blocks with runs_packed == Q->packed.
static int plan_part(int n, xdg_ham_s *const *hams, const RelabelledRef *in,
                     const void *const *xs, void *const *ys, const BatchMeta &P,
                     uint32_t tile_rows, SectorDesc *descs, uint32_t *prefix, BatchPart *Q) {
    std::vector<int> of;
    for (int i = 0; i < n; ++i)
        if (runs_packed(hams[i], in[i].get()) == (Q->packed != 0)) of.push_back(i);
    Q->n = (int)of.size();
    Q->kind = product_basis(hams[of[0]], in[of[0]].get())->plan.kind;
    // rows per work item: a multiple of the workgroup (default four rows per lane)
    Q->tile_rows = tile_rows ? (tile_rows + APPLY_BLOCK - 1) / APPLY_BLOCK * APPLY_BLOCK
                             : 4 * APPLY_BLOCK;
    size_t lds_full = 0, lds_part = 0;
    // few rows in all: terms shared out over the lanes, about four items per
    // compute unit
    Q->ring = 1;
    int64_t rows = 0, weight = 0, line = INT64_MAX;
    int most_bonds = 0;
    if (Q->kind == K_U1) {   // no group: the loop that the largest block takes alone
        const xdg_ham_s *most = hams[of[0]];
        size_t bonds = 0;
        for (int i : of) {
            if (hams[i]->basis->dim > most->basis->dim) most = hams[i];
            bonds = std::max(bonds, bond_bytes(hams[i]));
        }
        Q->own = u1_own(most, P.single, P.cols) && bonds <= lds_budget();
    }
    auto desc = [&](int i, const void *x, void *y) {
        SectorDesc d = make_desc(hams[i], in[i].get(), P.tsingle, x, y);
        if (Q->own) d.u1 = U1_OWN;
        return d;
    };
    for (int i : of) {
        const SectorDesc d = desc(i, nullptr, nullptr);
        const xdg_basis_s *b = product_basis(hams[i], in[i].get());
        rows += d.dim;
        weight += few_weight(b);
        line = std::min(line, few_line(b, d.n_bonds, P.cols, P.cplx));
        Q->ring &= ring_loop_ok(d, Q->kind, P.wide);
        most_bonds = std::max(most_bonds, d.n_bonds);
        lds_full = std::max(lds_full, P.tsingle ? stage_bytes<float>(d, Q->kind, 1)
                                                : stage_bytes<double>(d, Q->kind, 1));
    }
    if (weight < line && lds_full <= lds_budget() && P.cols < (int64_t)1 << 24) {
        int few = 0, block = 0;
        size_t lds = 0;
        if (few_shape(rows, most_bonds, P.cplx, P.tsingle, lds_full, &few, &block, &lds)) {
            const int64_t per = (int64_t)few * (block / 64);
            const int64_t want = (rows + 4 * (int64_t)device_cu_count() - 1) /
                                 (4 * (int64_t)device_cu_count());
            Q->few = few;
            Q->few_off = (uint32_t)a16(lds_full);
            Q->few_block = block;
            Q->few_lds = lds;
            Q->tile_rows = (uint32_t)std::max<int64_t>(1, (want + per - 1) / per * per);
        }
    }
    uint64_t acc = 0;
    for (int k = 0; k < Q->n; ++k) {
        const int i = of[k];
        const SectorDesc d = desc(i, xs[i], ys[i]);
        const uint64_t tiles = (hams[i]->basis->dim + Q->tile_rows - 1) / Q->tile_rows;
        if (acc + tiles >= 0xFFFFFFFFull) {
            set_error("too many row tiles in the batch");
            return XDG_EINVAL;
        }
        if (prefix) prefix[k] = (uint32_t)acc;
        acc += tiles;
        if (descs) descs[k] = d;
        const size_t f0 = P.tsingle ? stage_bytes<float>(d, Q->kind, 0)
                                    : stage_bytes<double>(d, Q->kind, 0);
        lds_part = std::max(lds_part, f0);
    }
    if (prefix) prefix[Q->n] = (uint32_t)acc;
    Q->n_tiles = (uint32_t)acc;
    Q->stage_sub = lds_full <= lds_budget();
    Q->lds = Q->stage_sub ? lds_full : lds_part;
    return XDG_OK;
}

int batch_plan_host(int n, xdg_ham_s *const *hams, const RelabelledRef *in,
                    const void *const *xs, void *const *ys, int64_t nvec, int dtype, BatchMeta *P,
                    SectorDesc *descs, uint32_t *prefix, uint32_t tile_rows) {
    if (n < 1) {
        set_error("batched apply needs at least one block");
        return XDG_EINVAL;
    }
    const xdg_basis_s *b0 = hams[0]->basis;
    bool any_cplx = false;
    for (int i = 0; i < n; ++i) {
        const xdg_basis_s *b = hams[i]->basis;
        if (b->plan.kind != b0->plan.kind || b->wide != b0->wide) {
            set_error("batched blocks must share the search kind and the state word width");
            return XDG_EINVAL;
        }
        if (b->is_complex && !dtype_complex(dtype)) {
            set_error("block %d is complex: vectors must be complex", i);
            return XDG_EINVAL;
        }
        any_cplx |= b->is_complex;
    }
    if (dtype < XDG_F64 || dtype > XDG_C64 || nvec < 1) {
        set_error("bad dtype or nvec");
        return XDG_EINVAL;
    }
    P->wide = b0->wide;
    P->single = dtype_single(dtype);
    P->acc64 = !P->single || !(b0->plan.flags & XDG_FLAG_F32_ACCUMULATE);
    P->tsingle = P->single && !P->acc64;
    P->cplx = any_cplx;
    P->cols = (dtype_complex(dtype) && !any_cplx) ? 2 * nvec : nvec;
    // the parts: every block runs the search that its products run alone, so that
    // a batch gives the same bits
    P->n_parts = 0;
    int placed = 0;
    for (const bool packed : {true, false}) {
        int in_part = 0;
        for (int i = 0; i < n; ++i) in_part += runs_packed(hams[i], in[i].get()) == packed;
        if (!in_part) continue;
        BatchPart &Q = P->part[P->n_parts];
        Q = BatchPart{};
        Q.packed = packed;
        Q.first = placed;
        XDG_RETURN_IF(plan_part(n, hams, in, xs, ys, *P, tile_rows,
                                descs ? descs + placed : nullptr,
                                prefix ? prefix + placed + P->n_parts : nullptr, &Q));
        placed += in_part;
        ++P->n_parts;
    }
    return XDG_OK;
}

int batch_prepare(int n, xdg_ham_s *const *hams, const RelabelledRef *in, const void *const *xs,
                  void *const *ys, int64_t nvec, int dtype, BatchPlan *P, uint32_t tile_rows) {
    if (n < 1) {
        set_error("batched apply needs at least one block");
        return XDG_EINVAL;
    }
    std::vector<SectorDesc> descs(n);
    std::vector<uint32_t> prefix(n + 2, 0);
    XDG_RETURN_IF(batch_plan_host(n, hams, in, xs, ys, nvec, dtype, P, descs.data(),
                                  prefix.data(), tile_rows));
    XDG_RETURN_IF(P->descs.upload(descs.data(), sizeof(SectorDesc) * n));
    XDG_RETURN_IF(P->prefix.upload(prefix.data(), sizeof(uint32_t) * (n + P->n_parts)));
    XDG_RETURN_IF(P->queue.alloc(sizeof(uint32_t)));
    return XDG_OK;
}

static int part_launch(const BatchMeta &P, const BatchPart &Q, const SectorDesc *d_descs,
                       const uint32_t *d_prefix, uint32_t *d_queue, int grid, int nv_cap,
                       hipStream_t st) {
    if (Q.n_tiles == 0) return XDG_OK;
    ApplyArgs A{};
    A.descs = d_descs;
    A.tile_prefix = d_prefix;
    A.n_secs = Q.n;
    A.n_tiles = Q.n_tiles;
    A.tile_rows = Q.tile_rows;
    A.queue = d_queue;
    A.nvec = P.cols;
    A.stage_sub = Q.stage_sub;
    A.packed = Q.packed;
    A.occ = Q.stage_sub ? occ_for(Q.lds) : 0;
    A.ring = Q.ring;
    A.own = Q.own;
    if (Q.few) {   // one launch for all vectors
        A.few = Q.few;
        A.few_off = Q.few_off;
        A.occ = 0;
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, st, A.queue);
        XDG_TRY_HIP(hipGetLastError());
        const unsigned gf = std::min<unsigned>(Q.n_tiles, 2u * (unsigned)device_cu_count());
        return launch_dispatch(Q.kind, P.wide, P.single, P.acc64, P.cplx, 1, A, gf,
                               (unsigned)Q.few_block, Q.few_lds, st);
    }
    const unsigned g = (unsigned)(grid > 0 ? grid : apply_grid_for(2));
    for (int64_t v0 = 0; v0 < P.cols;) {
        const int nv = pick_nv(P.cols - v0, nv_cap > 0 ? nv_cap : 8);
        A.v0 = (int)v0;
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, st, A.queue);
        XDG_TRY_HIP(hipGetLastError());
        XDG_RETURN_IF(
            launch_dispatch(Q.kind, P.wide, P.single, P.acc64, P.cplx, nv, A, g, APPLY_BLOCK,
                            Q.lds, st));
        v0 += nv;
    }
    return XDG_OK;
}

// The parts follow each other on the stream and share the queue counter.
int batch_launch_raw(const BatchMeta &P, const SectorDesc *d_descs, const uint32_t *d_prefix,
                     uint32_t *d_queue, int grid, int nv_cap, hipStream_t st) {
    for (int p = 0; p < P.n_parts; ++p) {
        const BatchPart &Q = P.part[p];
        XDG_RETURN_IF(part_launch(P, Q, d_descs + Q.first, d_prefix + Q.first + p, d_queue, grid,
                                  nv_cap, st));
    }
    return XDG_OK;
}

int batch_launch(const BatchPlan &P, int grid, int nv_cap, hipStream_t st) {
    return batch_launch_raw(P, P.descs.as<SectorDesc>(), P.prefix.as<uint32_t>(),
                            P.queue.as<uint32_t>(), grid, nv_cap, st);
}

// ------------------------------------------------- batched launch shape --
// Chosen once per set of blocks (and nvec, dtype) and remembered: the
// persistent grid (1, 2 or 4 workgroups per compute unit), then the rows per
// work item (1k - 16k), then the vectors per pass (8, 4, 2).  XDG_TUNE_LOG=1
// prints the timings.
namespace {
std::mutex g_shape_mu;
std::map<std::vector<const void *>, BatchShape> g_shape_cache;

std::vector<const void *> shape_key(int n, xdg_ham_s *const *hams, int64_t nvec, int dtype) {
    std::vector<const void *> key;
    for (int i = 0; i < n; ++i) {
        key.push_back(hams[i]);
        key.push_back(reinterpret_cast<const void *>((uintptr_t)hams[i]->serial));
    }
    key.push_back(reinterpret_cast<const void *>((intptr_t)(nvec * 8 + dtype)));
    return key;
}
}  // namespace

bool batch_shape_cached(int n, xdg_ham_s *const *hams, int64_t nvec, int dtype, BatchShape *out) {
    std::lock_guard<std::mutex> lock(g_shape_mu);
    auto it = g_shape_cache.find(shape_key(n, hams, nvec, dtype));
    if (it == g_shape_cache.end()) return false;
    *out = it->second;
    return true;
}

int batch_shape_tuned(int n, xdg_ham_s *const *hams, const RelabelledRef *in,
                      const void *const *xs, void *const *ys, int64_t nvec, int dtype,
                      hipStream_t st, BatchShape *out) {
    const auto key = shape_key(n, hams, nvec, dtype);
    std::lock_guard<std::mutex> lock(g_shape_mu);
    auto it = g_shape_cache.find(key);
    if (it != g_shape_cache.end()) {
        *out = it->second;
        return XDG_OK;
    }
    BatchShape best_shape{apply_grid_for(2), 4 * 1024, 8};
    BatchMeta meta;
    XDG_RETURN_IF(batch_plan_host(n, hams, in, xs, ys, nvec, dtype, &meta, nullptr, nullptr));
    bool few = true;
    for (int p = 0; p < meta.n_parts; ++p) few &= meta.part[p].few != 0;
    if (few) {   // its shape follows from the sizes
        g_shape_cache[key] = best_shape;
        *out = best_shape;
        return XDG_OK;
    }
    hipEvent_t e0, e1;
    XDG_TRY_HIP(hipEventCreate(&e0));
    XDG_TRY_HIP(hipEventCreate(&e1));
    float best = 1e30f;
    int64_t cols = 1;
    auto time_shape = [&](const BatchShape &sh) -> int {
        BatchPlan P;
        XDG_RETURN_IF(batch_prepare(n, hams, in, xs, ys, nvec, dtype, &P, sh.tile));
        cols = P.cols;
        XDG_RETURN_IF(batch_launch(P, sh.grid, sh.nv, st));
        XDG_TRY_HIP(hipEventRecord(e0, st));
        XDG_RETURN_IF(batch_launch(P, sh.grid, sh.nv, st));
        XDG_TRY_HIP(hipEventRecord(e1, st));
        XDG_TRY_HIP(hipEventSynchronize(e1));
        float ms = 0;
        XDG_TRY_HIP(hipEventElapsedTime(&ms, e0, e1));
        if (tune_log())
            fprintf(stderr, "[xdg tune] batched %d blocks nvec %lld: grid %d tile %u nv %d: "
                    "%.3f ms\n", n, (long long)nvec, sh.grid, sh.tile, sh.nv, ms);
        if (ms < best) {
            best = ms;
            best_shape = sh;
        }
        return XDG_OK;
    };
    int rc = XDG_OK;
    for (int mult : {1, 2, 4})
        if (rc == XDG_OK) rc = time_shape({apply_grid_for(mult), 4 * 1024, 8});
    const BatchShape g = best_shape;
    for (uint32_t tile : {1024u, 2048u, 8192u, 16384u})
        if (rc == XDG_OK) rc = time_shape({g.grid, tile, g.nv});
    const BatchShape t = best_shape;
    for (int nv : {4, 2})
        if (rc == XDG_OK && nv < cols) rc = time_shape({t.grid, t.tile, nv});
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    XDG_RETURN_IF(rc);
    g_shape_cache[key] = best_shape;
    *out = best_shape;
    return XDG_OK;
}

// ------------------------------------------------- allocation-free batch --
// One file-scope device array per GPU holds everything the batched launch
// needs beyond the caller's vectors: the queue counter, the tile prefix and
// the sector descriptors.  Its address is taken once per device with
// hipGetSymbolAddress (the array's name is a host-side stand-in, not a device
// address); descriptors reach it through the arguments of a small fill
// kernel, so nothing is allocated and no host buffer must outlive the call.
constexpr int NOALLOC_MAX_SECTORS = 128;
constexpr size_t NOALLOC_PREFIX_OFF = 256;
constexpr size_t NOALLOC_DESC_OFF =
    a16(NOALLOC_PREFIX_OFF + sizeof(uint32_t) * (NOALLOC_MAX_SECTORS + 2));
constexpr size_t NOALLOC_BYTES = NOALLOC_DESC_OFF + sizeof(SectorDesc) * NOALLOC_MAX_SECTORS;
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

constexpr int FILL_PER_LAUNCH = 4;
struct FillArgs {
    SectorDesc d[FILL_PER_LAUNCH];
    uint32_t prefix[FILL_PER_LAUNCH + 2];   // the last launch also writes the entries behind
    int first, count, n_prefix;
    unsigned char *base;
};
static_assert(sizeof(FillArgs) <= 4096, "fill kernel arguments");

static __global__ void k_fill_batch(FillArgs a) {
    const int i = threadIdx.x;
    if (i < a.count)
        reinterpret_cast<SectorDesc *>(a.base + NOALLOC_DESC_OFF)[a.first + i] = a.d[i];
    if (i < a.n_prefix)
        reinterpret_cast<uint32_t *>(a.base + NOALLOC_PREFIX_OFF)[a.first + i] = a.prefix[i];
}

static int scratch_address(unsigned char **out) {
    static std::mutex mu;
    static void *ptr[64] = {};
    int dev = 0;
    XDG_TRY_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) {
        set_error("device %d out of range for the allocation-free path", dev);
        return XDG_EINVAL;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        XDG_TRY_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) {
            set_error("hipGetSymbolAddress returned no address for the scratch array");
            return XDG_EHIP;
        }
        ptr[dev] = p;
    }
    *out = static_cast<unsigned char *>(ptr[dev]);
    return XDG_OK;
}

int apply_batched_noalloc(int n, xdg_ham_s *const *hams, const void *const *xs,
                          void *const *ys, int64_t nvec, int dtype, hipStream_t st) {
    if (n < 1 || n > NOALLOC_MAX_SECTORS) {
        set_error("allocation-free batched apply takes 1 to %d blocks (got %d); its scratch "
                  "array holds %zu bytes", NOALLOC_MAX_SECTORS, n, NOALLOC_BYTES);
        return XDG_EINVAL;
    }
    for (int i = 0; i < n; ++i)
        if (!hams[i] || !xs[i] || !ys[i] || xs[i] == ys[i]) {
            set_error("batched apply: null handle/pointer or x == y at %d", i);
            return XDG_EINVAL;
        }
    thread_local SectorDesc descs[NOALLOC_MAX_SECTORS];
    thread_local uint32_t prefix[NOALLOC_MAX_SECTORS + 2];
    BatchShape sh;     // a shape tuned earlier for these blocks, else the default
    const bool tuned = batch_shape_cached(n, hams, nvec, dtype, &sh);
    BatchMeta M;
    const std::vector<RelabelledRef> in = relabelled(n, hams, st);
    XDG_RETURN_IF(batch_plan_host(n, hams, in.data(), xs, ys, nvec, dtype, &M, descs, prefix,
                                  tuned ? sh.tile : 0));
    unsigned char *base = nullptr;
    XDG_RETURN_IF(scratch_address(&base));
    for (int first = 0; first < n; first += FILL_PER_LAUNCH) {
        FillArgs a{};
        a.first = first;
        a.count = std::min(FILL_PER_LAUNCH, n - first);
        a.n_prefix = a.count + (first + a.count == n ? M.n_parts : 0);
        for (int i = 0; i < a.count; ++i) a.d[i] = descs[first + i];
        for (int i = 0; i < a.n_prefix; ++i) a.prefix[i] = prefix[first + i];
        a.base = base;
        hipLaunchKernelGGL(k_fill_batch, dim3(1), dim3(64), 0, st, a);
        XDG_TRY_HIP(hipGetLastError());
    }
    return batch_launch_raw(M, reinterpret_cast<const SectorDesc *>(base + NOALLOC_DESC_OFF),
                            reinterpret_cast<const uint32_t *>(base + NOALLOC_PREFIX_OFF),
                            reinterpret_cast<uint32_t *>(base), tuned ? sh.grid : 0,
                            tuned ? sh.nv : 8, st);
}

int apply_batched_launch(int n, xdg_ham_s *const *hams, const void *const *xs, void *const *ys,
                         int64_t nvec, int dtype, hipStream_t st, uint32_t *, int grid, int) {
    for (int i = 0; i < n; ++i)
        if (!hams[i] || !xs[i] || !ys[i] || xs[i] == ys[i]) {
            set_error("batched apply: null handle/pointer or x == y at %d", i);
            return XDG_EINVAL;
        }
    // plans are cached by the exact argument tuple so that repeated calls
    // (iterative methods) upload nothing; a Hamiltonian enters the key by its
    // serial number too, since a new one may reuse a freed one's address, and by
    // its labelling, which it may lose (and never gets again)
    struct Key {
        std::vector<const void *> p;
        int64_t nvec;
        int dtype;
        bool operator==(const Key &o) const { return p == o.p && nvec == o.nvec && dtype == o.dtype; }
    };
    thread_local std::vector<std::pair<Key, std::unique_ptr<BatchPlan>>> cache;
    const std::vector<RelabelledRef> in = relabelled(n, hams, st);
    Key k;
    for (int i = 0; i < n; ++i) {
        k.p.push_back(hams[i]);
        k.p.push_back(reinterpret_cast<const void *>((uintptr_t)hams[i]->serial));
        k.p.push_back(in[i].get());
        k.p.push_back(xs[i]);
        k.p.push_back(ys[i]);
    }
    k.nvec = nvec;
    k.dtype = dtype;
    BatchShape sh;
    XDG_RETURN_IF(batch_shape_tuned(n, hams, in.data(), xs, ys, nvec, dtype, st, &sh));
    k.p.push_back(reinterpret_cast<const void *>((uintptr_t)sh.tile));
    BatchPlan *P = nullptr;
    for (auto &e : cache)
        if (e.first == k) P = e.second.get();
    if (!P) {
        auto up = std::make_unique<BatchPlan>();
        XDG_RETURN_IF(batch_prepare(n, hams, in.data(), xs, ys, nvec, dtype, up.get(), sh.tile));
        if (cache.size() >= 8) cache.erase(cache.begin());
        cache.emplace_back(k, std::move(up));
        P = cache.back().second.get();
    }
    return batch_launch(*P, grid > 0 ? grid : sh.grid, sh.nv, st);
}

}  // namespace xdg
