// The matrix-free application y = H x on a sector (apply, Sec. 3.6; the
// on-the-fly element loop of Sec. 5.1 and the indexing of Sec. 5.2).
//
// Pull form: every output row r (a basis state) is summed by one lane.  For every bond
// with unequal spins it forms t = r with both spins exchanged, finds the
// representative s of t, a group element u with u.t = s (the first one the
// search meets: when s is in the block, chi is 1 on Stab(s), so every such u
// has the same chi(u)) and the number of such elements (= |Stab(s)|), looks
// up the index of s, and adds
//      (Jxy/2) chi(u) sqrt(|Stab s| / |Stab r|) x[idx(s)]
// to the row, after the diagonal Sum_b Jz_b (+-1/4) x[r].  The row is
// written once: no atomics, bitwise reproducible for any launch shape.
// Up to NV vectors of the [dim][nvec] block share each search and lookup.
// Workgroups are up to 1024 lanes so that the tables staged in LDS (bonds,
// characters, search tables) are shared by 16 waves.
#pragma once

#include <type_traits>

#include "device_common.hpp"

namespace xdg {

#ifndef XDG_APPLY_BLOCK
#define XDG_APPLY_BLOCK 1024
#endif
constexpr int APPLY_BLOCK = XDG_APPLY_BLOCK;
// Occupancy variant: at most 64 VGPRs (8 waves per SIMD, two 1024-lane
// workgroups per CU), chosen when two workgroups' LDS fit in one CU.
constexpr int OCC_WAVES = 8;
constexpr int BLOCKS_PER_1024 = 1024 / APPLY_BLOCK;   // grid scale for smaller workgroups

// The loops over a launch's rows (see process_range).
enum : int {
    LOOP_ROW = 0, LOOP_CMP = 1, LOOP_FEW = 2, LOOP_PACKED = 3, LOOP_RING = 4, LOOP_OWN = 5,
    LOOP_BLOCKS = 6, LOOP_BATCH_PACKED = 7, LOOP_BATCH_BLOCKS = 8
};
// Sublattice searches: either, the packed one, the one by blocks.
enum : int { FORM_ANY = 0, FORM_PACKED = 1, FORM_BLOCKS = 2 };
constexpr int form_of_loop(int loop) {
    return loop == LOOP_PACKED || loop == LOOP_BATCH_PACKED   ? FORM_PACKED
           : loop == LOOP_BLOCKS || loop == LOOP_BATCH_BLOCKS ? FORM_BLOCKS
                                                              : FORM_ANY;
}

template <class T> struct Vec2;
template <> struct Vec2<float> { using type = float2; };
template <> struct Vec2<double> { using type = double2; };

template <class T>
__device__ __forceinline__ T fmadd(T a, T b, T c) {
    if constexpr (sizeof(T) == 4)
        return __builtin_fmaf(a, b, c);
    else
        return __builtin_fma(a, b, c);
}

template <class T> struct BondT;
template <> struct BondT<float> { using type = BondF; };
template <> struct BondT<double> { using type = BondD; };

// Blocks without a group: all lanes on one bond, far exchanges through Lin's
// tables or the rank tables in LDS; or every lane on its own bonds (LOOP_OWN).
enum : int { U1_LIN = 0, U1_RANK = 1, U1_OWN = 2 };

// Everything one sector needs on the device (type-erased pointers).
struct SectorDesc {
    const void *reps;            // u32 / u64 [dim]
    const uint16_t *stab;        // [dim]
    int64_t dim;
    const void *hash;
    uint64_t n_lines;
    uint64_t empty;
    const uint2 *rwords;         // rank index (null: hash)
    uint64_t n_rwords;
    const void *rtab;            // colex chunk tables (layout rl)
    RankLayout rl;
    int n_up;
    const uint32_t *lin;         // Lin tables (U(1))
    int nlo;
    const uint32_t *u1_adj;      // U(1): C(i, k) [n_sites][n_up + 1]
    int u1;                      // U(1): form of the loop, U1_*
    int n_sites, n_sym, n_bonds;
    const AffineElem *aff;
    int ring;                    // 0, 1 (all rotations), 2 (and all reflections)
    const int16_t *ring_gidx;    // [2 n_sites]
    const uint64_t *bytetab;
    int n_bchunks;
    const uint16_t *mintop;
    const uint32_t *cand_off;
    const uint16_t *cand_list;
    const uint32_t *sp;
    const uint16_t *tperm;
    int n_s, m, pb, n_perm;
    uint32_t n_cand;
    int subf;                    // sublattice tables in the packed form (staged kernels)
    const uint32_t *pk_tab;      // its block table and candidate lists
    const uint16_t *pk_cand;
    uint32_t n_pk;
    int pk_nb;
    const BondX *bx;             // per-bond data of the packed form [n_bonds]
    const void *bonds;           // BondD / BondF [n_bonds]
    const void *chi;             // double2 / float2 [n_sym]
    const void *sqrtt;           // T [2 (n_sym + 1)]: sqrt(c), then 1/sqrt(c)
    double jz_quarter;           // (1/4) sum_b Jz_b: the diagonal of the all-aligned state
    int ring_bonds;              // 1: n_bonds = n_sites and bond b joins sites b and b + 1 mod N
    int ring_eq;                 // 1: the same, with equal couplings
    int chi_one;                 // 1: every character is exactly 1
    // rank-addressed x (sublattice coding): slot top_rank(s) of xr holds the
    // row of representative s when s is a basis state, zeros otherwise, so a
    // term reads x without the index lookup (null: through the rank index)
    const void *xr;
    const uint64_t *xr_top;      // [2^m] first rank of each top block, ~0 if none
    const uint32_t *xr_top32;    // the same in 4 bytes (0xFFFFFFFF if none), when all fit; or null
    uint64_t xr_slots;           // slots of xr (beyond the last one: not in the block)
    int xr_cols;                 // columns of a slot (see xr_columns)
    int xr_bits;                 // sites below the top block
    const uint32_t *xr_rtab;     // the rank tables' rows for the chunks below it, 4-byte entries
    int xr_rows;                 // rows of xr_rtab
    // packed form: the slots of block_slot instead (null: the ranks above)
    const uint32_t *xb_ent, *xb_off;
    const uint2 *xb_top;
    int xb_w32;
    // relabelled sector: position in x and y of the orbit of basis state k,
    // bit 31 where its sign differs (sublattice kind only; null: k itself)
    const uint32_t *umap;
    const void *x;
    void *y;
};

struct ApplyArgs {
    SectorDesc one;              // used when descs == nullptr
    const SectorDesc *descs;     // batched: device array [n_secs]
    const uint32_t *tile_prefix; // batched: [n_secs + 1] cumulative tile counts
    int n_secs;
    uint32_t n_tiles;
    uint32_t tile_rows;
    uint32_t *queue;             // batched: work counter, zero at launch
    int64_t nvec;
    int v0;                      // first vector of this pass
    int stage_sub;               // copy sublattice tables into LDS
    int occ;                     // use the 8-waves-per-SIMD variant
    int compact;                 // table searches: wave-compacted term loop
    int few;                     // rows per wave of the few-rows loop (0: another loop)
    int ring;                    // every block takes the ring loop (see ring_loop_ok)
    int own;                     // no group: the loop over own bonds
    int packed;                  // batch: every block in the packed sublattice form
    uint32_t few_off;            // byte offset of its terms behind the staged tables
    unsigned long long *count;   // nnz counting mode (nullptr otherwise)
};

__host__ __device__ constexpr size_t a16(size_t x) { return (x + 15) & ~(size_t)15; }

__host__ __device__ inline size_t sub_table_bytes(const SectorDesc &d) {
    const size_t NV = (size_t)d.n_s << d.m;
    if (d.subf)
        return packed_entry_bytes(d.n_sym) + packed_table_bytes(d.n_pk, d.n_perm, d.m, d.pb);
    return a16(2 * NV) + a16(4 * (NV + 1)) + a16(2 * (size_t)d.n_cand) +
           a16(4 * (size_t)d.n_sym * d.n_s) +
           a16(2 * (size_t)d.n_perm * 2 * ((size_t)1 << d.pb));
}

__host__ __device__ inline size_t rank_table_bytes(const SectorDesc &d) {
    if (!d.rwords && d.u1 != U1_RANK) return 0;
    // the rank-addressed x reads only its 4-byte rows of the chunks below the top block
    if (d.xr && d.xb_ent) return 0;
    if (d.xr) return ((size_t)d.xr_rows << d.rl.cb) * 4;
    return ((size_t)d.rl.rows << d.rl.cb) * (d.rl.e32 ? 4 : 8);
}

// bytes of the first-rank table of the rank-addressed x in LDS
__host__ __device__ inline size_t xr_top_bytes(const SectorDesc &d) {
    if (d.xb_ent) {   // entries, offsets, tops
        const size_t m1 = (size_t)d.m + 1;
        return a16((size_t)4 << d.m) + a16(4 * m1 * m1 * m1) + ((size_t)8 << d.m);
    }
    return ((size_t)1 << d.m) * (d.xr_top32 ? 4 : 8);
}

// The ring loop (process_ring): a full ring of more than half a state's bits
// with equal neighbour bonds and the rank index.
inline bool ring_loop_ok(const SectorDesc &d, int kind, bool wide) {
    return kind == K_AFF && (d.dim == 0 || (d.ring && d.ring_eq && d.rwords)) &&
           (wide ? d.n_sites > 32 && d.n_sites < 64 : d.n_sites > 16);
}

// LDS bytes needed to stage a sector's tables.
template <class T>
__host__ __device__ inline size_t stage_bytes(const SectorDesc &d, int kind, int stage_sub) {
    size_t n = a16(sizeof(typename BondT<T>::type) * d.n_bonds);
    // no group: one bond for all lanes is read with scalar loads, so any number
    // of them fits
    if (kind == K_U1)
        return d.u1 == U1_OWN
                   ? n
                   : a16(4 * (size_t)d.n_sites * (d.n_up + 1)) + a16(rank_table_bytes(d));
    n += a16(sizeof(typename Vec2<T>::type) * d.n_sym);
    n += a16(sizeof(T) * 2 * (d.n_sym + 1));
    n += a16(rank_table_bytes(d));
    if (kind == K_AFF) n += a16(sizeof(AffineElem) * d.n_sym) + a16(4 * (size_t)d.n_sites);
    if (kind == K_AFF && d.ring_eq)
        n += a16(sizeof(T) * (d.n_sym + 1)) + a16(sizeof(T) * (d.n_bonds + 1));
    if (kind == K_SUB && stage_sub) n += sub_table_bytes(d);
    if (kind == K_SUB && stage_sub && d.xr) n += a16(xr_top_bytes(d));
    return n;
}

template <class T>
struct Staged {
    const typename BondT<T>::type *bonds;
    const typename Vec2<T>::type *chi;
    const T *sq;       // sqrt(c)
    const T *rsq;      // 1/sqrt(c)
    const AffineElem *aff;
    const int16_t *ring_gidx;
    const T *hs, *jsum;    // ring loop: see process_ring
    const void *rtab;
    const uint32_t *adj;   // U(1): see process_row_u1
    SubCtx sub;
    bool subf;             // packed sublattice search
    PackedCtx pk;
    SlotCtx slot;          // rank-addressed x of a packed sector
    const uint64_t *xr_top;   // first rank of each top block (rank-addressed x)
    const uint32_t *xr_top32; // the same in 4 bytes (xr_w32) at the same place
    bool xr_w32;
};

template <class E>
__device__ inline E *stage_copy(unsigned char *smem, size_t &off, const E *src, size_t n) {
    E *dst = reinterpret_cast<E *>(smem + off);
    off = a16(off + sizeof(E) * n);
    for (size_t e = threadIdx.x; e < n; e += blockDim.x) dst[e] = src[e];
    return dst;
}

// STAGE: the sublattice tables go to LDS too (otherwise they are read from
// global memory); a compile-time choice so that every table pointer has a
// known address space.
template <int KIND, class T, bool STAGE, int LOOP = LOOP_ROW>
__device__ inline void stage(const SectorDesc &d, unsigned char *smem, Staged<T> &S) {
    using B = typename BondT<T>::type;
    using T2 = typename Vec2<T>::type;
    size_t off = 0;
    // packed sublattice search: the elements' entries come first, so that
    // their LDS addresses fit the 16 bits of a candidate
    if constexpr (KIND == K_SUB && STAGE)
        if (d.subf) off = packed_entry_bytes(d.n_sym);
    if constexpr (KIND == K_U1 && LOOP != LOOP_OWN)
        S.bonds = reinterpret_cast<const B *>(d.bonds);
    else
        S.bonds = stage_copy(smem, off, reinterpret_cast<const B *>(d.bonds), d.n_bonds);
    S.sub = SubCtx{d.mintop, d.cand_off, d.cand_list, d.sp, d.tperm, d.n_s, d.m, d.pb};
    S.subf = false;
    S.xr_top = d.xr_top;
    S.xr_top32 = d.xr_top32;
    S.xr_w32 = d.xr_top32 != nullptr;
    if constexpr (KIND == K_U1 && LOOP != LOOP_OWN) {
        S.adj = stage_copy(smem, off, d.u1_adj, (size_t)d.n_sites * (d.n_up + 1));
        S.rtab = stage_copy(smem, off, reinterpret_cast<const uint32_t *>(d.rtab),
                            rank_table_bytes(d) / 4);
    }
    if constexpr (KIND != K_U1) {
        S.chi = stage_copy(smem, off, reinterpret_cast<const T2 *>(d.chi), d.n_sym);
        const T *ls = stage_copy(smem, off, reinterpret_cast<const T *>(d.sqrtt), 2 * (d.n_sym + 1));
        S.sq = ls;
        S.rsq = ls + d.n_sym + 1;
        S.rtab = stage_copy(smem, off,
                            reinterpret_cast<const uint32_t *>(d.xr ? d.xr_rtab : d.rtab),
                            rank_table_bytes(d) / 4);
        if constexpr (KIND == K_AFF) {
            S.aff = stage_copy(smem, off, d.aff, d.n_sym);
            int16_t *lg = reinterpret_cast<int16_t *>(smem + off);
            off = a16(off + 4 * (size_t)d.n_sites);
            if (d.ring)
                for (int e = threadIdx.x; e < 2 * d.n_sites; e += blockDim.x) {
                    int from = e;
                    if constexpr (LOOP == LOOP_RING)   // by the site read first (see ring_scan_big)
                        from = (e + 1) % d.n_sites == 0 ? e + 1 - d.n_sites : e + 1;
                    lg[e] = d.ring_gidx[from];
                }
            S.ring_gidx = lg;
            if constexpr (LOOP == LOOP_RING) {
                const B b0 = *reinterpret_cast<const B *>(d.bonds);
                T *hs = reinterpret_cast<T *>(smem + off);
                off = a16(off + sizeof(T) * ((size_t)d.n_sym + 1));
                T *js = reinterpret_cast<T *>(smem + off);
                off = a16(off + sizeof(T) * ((size_t)d.n_bonds + 1));
                for (int e = threadIdx.x; e <= d.n_sym; e += blockDim.x)
                    hs[e] = b0.h * reinterpret_cast<const T *>(d.sqrtt)[e];
                for (int e = threadIdx.x; e <= d.n_bonds; e += blockDim.x) {
                    T sum = 0;
                    for (int b = 0; b < e; ++b) sum += b0.jz;
                    js[e] = sum;
                }
                S.hs = hs;
                S.jsum = js;
            }
        }
        if constexpr (KIND == K_SUB) {
            if constexpr (STAGE) {
                const size_t NV = (size_t)d.n_s << d.m;
                const size_t ntp = (size_t)d.n_perm * 2 * ((size_t)1 << d.pb);
                constexpr int form = form_of_loop(LOOP);
                auto packed = [&] {
                    const PackedSrc src{d.pk_tab, d.pk_cand, d.sp, d.tperm, d.n_pk, d.pk_nb,
                                        d.n_sym, d.n_perm, d.m, d.pb};
                    S.pk = stage_packed(src, smem, off);
                    S.subf = true;
                    // unused, but addresses in LDS as in the other form: a pointer
                    // into either memory makes every table read a flat one (5x6
                    // square numbered row by row, 15 up, FP64: 2.70 against 2.59 ms)
                    if constexpr (form == FORM_ANY) {
                        const uint16_t *lds = reinterpret_cast<const uint16_t *>(smem);
                        S.sub.mintop = S.sub.cand_list = S.sub.tperm = lds;
                        S.sub.cand_off = S.sub.sp = reinterpret_cast<const uint32_t *>(smem);
                    }
                };
                auto blocks = [&] {
                    S.sub.mintop = stage_copy(smem, off, d.mintop, NV);
                    S.sub.cand_off = stage_copy(smem, off, d.cand_off, NV + 1);
                    S.sub.cand_list = stage_copy(smem, off, d.cand_list, d.n_cand);
                    S.sub.sp = stage_copy(smem, off, d.sp, (size_t)d.n_sym * d.n_s);
                    S.sub.tperm = stage_copy(smem, off, d.tperm, ntp);
                };
                if constexpr (form == FORM_PACKED) packed();
                else if constexpr (form == FORM_BLOCKS) blocks();
                else if (d.subf) packed();
                else blocks();
                // the first-rank table at one LDS address whatever its entry
                // size (both pointers always address LDS here: LDS reads)
                unsigned char *tp = smem + off;
                if (d.xr && d.xb_ent) {
                    const uint32_t base =
                        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
                    const uint32_t m1 = (uint32_t)d.m + 1, V = 1u << d.m;
                    S.slot.ent = base + (uint32_t)off;
                    stage_copy(smem, off, d.xb_ent, V);
                    const uint32_t oa = base + (uint32_t)off;
                    stage_copy(smem, off, d.xb_off, (size_t)m1 * m1 * m1);
                    S.slot.top = base + (uint32_t)off;
                    uint2 *lt = reinterpret_cast<uint2 *>(smem + off);
                    for (uint32_t e = threadIdx.x; e < V; e += blockDim.x) {
                        const uint2 t = d.xb_top[e];
                        lt[e] = make_uint2(t.x, t.y + oa);
                    }
                    off = a16(off + 8 * (size_t)V);
                    S.slot.m = d.m;
                    S.slot.w32 = d.xb_w32 != 0;
                } else if (d.xr) {
                    if (d.xr_top32)
                        stage_copy(smem, off, d.xr_top32, (size_t)1 << d.m);
                    else
                        stage_copy(smem, off, d.xr_top, (size_t)1 << d.m);
                }
                S.xr_top32 = reinterpret_cast<const uint32_t *>(tp);
                S.xr_top = reinterpret_cast<const uint64_t *>(tp);
            }
        }
    }
}

// Positions of 32-bit states are below C(32, 16) < 2^31: 32-bit indices.
template <class W> struct IndexT { using type = int64_t; };
template <> struct IndexT<uint32_t> { using type = int32_t; };

// Locate the representative of t and its index; returns -1 when the orbit
// is not in the block.  On success writes u and |Stab(s)|.  key: t's key for
// the packed sublattice search (computed here from t when null and that
// search is on).  XR: the position is the slot in the rank-addressed x
// (sublattice coding with d.xr set); XR = 2: every character is 1, so the
// search does not keep the element (u is left unset).  FORM: the sublattice
// search of the block, FORM_ANY where the sector tells.
template <class W, int KIND, class T, int XR = 0, int FORM = FORM_ANY>
__device__ __forceinline__ typename IndexT<W>::type locate(const SectorDesc &d, const Staged<T> &S,
                                                           W t, int &u, int &cnt,
                                                           const SubKey *key = nullptr) {
    using I = typename IndexT<W>::type;
    if constexpr (KIND == K_U1) {
        const uint64_t lo = (uint64_t)t & ((1ull << d.nlo) - 1);
        const uint64_t hi = (uint64_t)t >> d.nlo;
        const uint32_t *lin = d.lin;
        u = 0;
        cnt = 1;
        return (I)((int64_t)gld(lin + (1ull << d.nlo) + hi) + (int64_t)gld(lin + lo));
    } else {
        W rep;
        if constexpr (KIND == K_AFF) {
            if (d.ring)
                ring_search<W>(S.ring_gidx, d.ring, d.n_sites, t, rep, u, cnt);
            else
                aff_search<W>(S.aff, d.n_sym, d.n_sites, t, rep, u, cnt);
        } else if constexpr (KIND == K_SUB) {
            if (FORM == FORM_PACKED || (FORM == FORM_ANY && S.subf)) {
                uint32_t top, low;
                sub_search_packed<XR != 2>(S.pk, key ? *key : sub_key<W>(t, d.m, d.pb), top, low,
                                           u, cnt);
                if constexpr (XR != 0) return (I)block_slot_lds(S.slot, top, low);
                rep = ((W)top << (3 * d.m)) | (W)low;
            } else if (d.n_s == 4)
                sub_search<W, 4>(S.sub, t, rep, u, cnt);
            else
                sub_search<W, 0>(S.sub, t, rep, u, cnt);
        } else {
            tab_search<W>(d.bytetab, d.n_bchunks, d.n_sym, t, rep, u, cnt);
        }
        if constexpr (KIND == K_SUB && XR != 0) {
            // the slot of rep in the rank-addressed x (zeros unless rep is a basis state)
            if (d.xb_ent) {
                const int B = 3 * d.m;
                return (I)block_slot_lds(S.slot, (uint32_t)(rep >> B),
                                         (uint32_t)rep & ((1u << B) - 1u));
            }
            const uint32_t *T32 = static_cast<const uint32_t *>(S.rtab);
            const uint64_t r = S.xr_w32
                                   ? top_rank32<W>(T32, d.rl, d.xr_bits, S.xr_top32, rep)
                                   : top_rank<W>(T32, d.rl, d.xr_bits, S.xr_top, rep);
            return r < d.xr_slots ? (I)r : (I)-1;
        }
        if (d.rwords) {
            if constexpr (sizeof(W) == 4) {
                const uint64_t r = colex_rank<W>(S.rtab, d.rl, rep);
                return rank_find32(d.rwords, (uint32_t)d.n_rwords, (uint32_t)r);
            } else {
                // 4-byte entries: every basis state's rank is below 2^32 - 1
                if (d.rl.e32) {
                    const uint32_t r =
                        colex_rank_sat<W>(static_cast<const uint32_t *>(S.rtab), d.rl, rep);
                    return r == 0xFFFFFFFFu ? -1
                                            : rank_find_r32(d.rwords, (uint32_t)d.n_rwords, r);
                }
                return rank_find(d.rwords, d.n_rwords, colex_rank<W>(S.rtab, d.rl, rep));
            }
        }
        return (I)hash_find<W>(d.hash, d.n_lines, (W)d.empty, rep);
    }
}

// Position of basis state k in the caller's vectors; flips the sign of `f`
// where the caller's symmetric state differs by one.
template <class A>
__device__ __forceinline__ int64_t user_pos(const SectorDesc &d, int64_t k, A &f) {
    const uint32_t v = gld(d.umap + k);
    f = v >> 31 ? -f : f;
    return (int64_t)(v & 0x7FFFFFFFu);
}

// A row of a block without a group.  All lanes take the same bond, whose data
// are scalars: neighbouring rows agree in their upper sites, so most of a
// wave's gathers are consecutive.  Exchanging sites i and i + 1 moves the
// position by C(i, k), k the up spins below i (the colex rank's Pascal step),
// read from LDS; far exchanges take the rank of the new state.  The loads of
// U bonds are in flight together.  Walking each lane's own bonds with two Lin
// table reads before every gather kept the vector memory units busy with 64
// separate lines an instruction (ring N = 28, 40 M rows, FP64: 1.87 ms).
template <class W, class T, class A, int NV>
__device__ __forceinline__ void process_row_u1(const SectorDesc &d, const Staged<A> &S,
                                               int64_t row, int64_t nvec, int v0) {
    using B = typename BondT<A>::type;
    constexpr int U = NV <= 2 ? 4 : NV <= 4 ? 2 : 1;
    const W s = gld(reinterpret_cast<const W *>(d.reps) + row);
    const W pairs = s ^ (s >> 1);   // bit i: sites i and i + 1 differ
    const uint32_t r32 = (uint32_t)row;   // positions are below 2^32
    const T *X = reinterpret_cast<const T *>(d.x) + v0;
    T *Y = reinterpret_cast<T *>(d.y);
    const int nb = d.n_bonds;
    const uint32_t stride = (uint32_t)d.n_up + 1u, cols = (uint32_t)nvec;
    A junq = 0, acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0;
    for (int b0 = 0; b0 < nb; b0 += U) {
        bool off[U];
        A h[U];
        T xv[U][NV];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            off[k] = false;
            h[k] = 0;
#pragma unroll
            for (int v = 0; v < NV; ++v) xv[k][v] = T(0);
            if (b0 + k >= nb) continue;
            const B bd = sld(reinterpret_cast<const B *>(d.bonds) + b0 + k);
            const uint32_t lo = bd.i < bd.j ? bd.i : bd.j, hi = bd.i < bd.j ? bd.j : bd.i;
            h[k] = bd.h;
            const W bit = W(1) << lo;
            uint32_t at;
            if (hi == lo + 1) {
                off[k] = (pairs & bit) != 0;
                const W under = s & (bit - 1);
                const uint32_t below = (uint32_t)(sizeof(W) == 4 ? __popc((uint32_t)under)
                                                                 : __popcll((uint64_t)under));
                const uint32_t move = S.adj[lo * stride + below];
                // up if the spin at lo is: row + move, else row - move
                const uint32_t neg =
                    sizeof(W) == 4 ? (uint32_t)__builtin_amdgcn_sbfe((int)~(uint32_t)s, lo, 1)
                                   : ((s & bit) ? 0u : ~0u);
                at = (move ^ neg) + (r32 - neg);
            } else {
                const W mask = bit | (W(1) << hi), both = s & mask;
                off[k] = both != 0 && both != mask;
                at = r32;
                if (off[k]) {
                    if (d.u1 == U1_RANK) {
                        at = (uint32_t)colex_rank<W>(S.rtab, d.rl, s ^ mask);
                    } else {
                        int u, cnt;
                        at = (uint32_t)locate<W, K_U1, A>(d, S, s ^ mask, u, cnt);
                    }
                }
            }
            at = off[k] ? at : r32;   // spins equal: the own row is read and not added
            junq = fmadd<A>(off[k] ? A(1) : A(0), bd.jz, junq);
            const T *q = X + (uint64_t)at * cols;
#pragma unroll
            for (int v = 0; v < NV; ++v) xv[k][v] = gld(q + v);
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int v = 0; v < NV; ++v)
                acc[v] = fmadd<A>(h[k], off[k] ? (A)xv[k][v] : A(0), acc[v]);
    }
    const size_t base = (size_t)row * nvec + v0;
    const A diag = (A)d.jz_quarter - A(0.5) * junq;
    T xd[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) xd[v] = gld(X + (size_t)row * nvec + v);
#pragma unroll
    for (int v = 0; v < NV; ++v) gst(Y + base + v, (T)fmadd<A>(diag, (A)xd[v], acc[v]));
}

// A row of a block without a group, each lane walking its own unequal-spin
// bonds (a mask of 32 bonds at a time, lowest first) with Lin's tables: the
// same terms in the same order, and the same bits, as process_row_u1.  It waits
// for two dependent gathers a term, but takes no bond whose spins agree, and so
// serves fillings and lattices where most do (see u1_own): 6x6, 7 of 36 up,
// FP64 735 -> 538 us, 3 up 37 -> 12 us; ring N = 40, 5 up, FP32 29 -> 21.7 us.
template <class W, class T, class A, int NV>
__device__ __forceinline__ void process_row_own(const SectorDesc &d, const Staged<A> &S,
                                                int64_t row, int64_t nvec, int v0) {
    using B = typename BondT<A>::type;
    const W s = gld(reinterpret_cast<const W *>(d.reps) + row);
    const T *X = reinterpret_cast<const T *>(d.x) + v0;
    T *Y = reinterpret_cast<T *>(d.y) + v0;
    const int nb = d.n_bonds;
    A junq = 0, acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0;
    const W walls = d.ring_bonds ? (s ^ rotr_n<W>(s, 1, d.n_sites)) : W(0);
    for (int b0 = 0; b0 < nb; b0 += 32) {
        const int bn = nb - b0 < 32 ? nb - b0 : 32;
        uint32_t act = 0;
        if (d.ring_bonds) {   // bond b joins sites b and b + 1: bit b of the walls
            act = (uint32_t)(walls >> b0) & (bn == 32 ? ~0u : ((1u << bn) - 1u));
        } else {
            for (int k = 0; k < bn; ++k) {
                const B bd = S.bonds[b0 + k];
                act |= (((uint32_t)(s >> bd.i) ^ (uint32_t)(s >> bd.j)) & 1u) << k;
            }
        }
        while (act) {
            const int b = b0 + __builtin_ctz(act);
            act &= act - 1;
            const B bd = S.bonds[b];
            junq += bd.jz;
            int u, cnt;
            const auto at = locate<W, K_U1, A>(d, S, s ^ ((W(1) << bd.i) | (W(1) << bd.j)), u, cnt);
            const T *q = X + (sizeof(W) == 4 ? (uint64_t)(uint32_t)at * (uint32_t)nvec
                                             : (uint64_t)at * (uint64_t)nvec);
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] = fmadd<A>(bd.h, (A)gld(q + v), acc[v]);
        }
    }
    const size_t base = (size_t)row * nvec;
    const A diag = (A)d.jz_quarter - A(0.5) * junq;
    T xd[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) xd[v] = gld(X + base + v);
#pragma unroll
    for (int v = 0; v < NV; ++v) gst(Y + base + v, (T)fmadd<A>(diag, (A)xd[v], acc[v]));
}

// A row of a block with a group.  FORM: as for locate (the packed one comes with
// its bond records).
// T: storage type of x and y; A: type of the amplitudes and of the per-row
// accumulation (each output element is rounded to T once, at the store).
// XR: the terms read the rank-addressed x (sublattice coding, d.xr set);
// XR = 2: every character is 1 (the amplitude skips chi(u), a product by
// exactly 1).  PIPE: each term's gather is added at the next term of the row
// (or after its last bond), so that its latency overlaps the next search;
// the same fused multiply-adds in the same order.
template <class W, int KIND, class T, class A, bool CPLX, int NV, int XR = 0,
          bool PIPE = false, int FORM = FORM_ANY>
__device__ __forceinline__ void process_row(const SectorDesc &d, const Staged<A> &S, int64_t row,
                                            int64_t nvec, int v0) {
    static_assert(KIND != K_U1, "process_row_u1");
    using B = typename BondT<A>::type;
    constexpr int C = CPLX ? 2 : 1;
    const W s = gld(reinterpret_cast<const W *>(d.reps) + row);
    const T *X = reinterpret_cast<const T *>(d.x);
    T *Y = reinterpret_cast<T *>(d.y);
    // the terms' x: rank-addressed (the same values at other places) or x itself
    const T *XT = XR != 0 ? reinterpret_cast<const T *>(d.xr) : X;
    static_assert(XR != 2 || (PIPE && !CPLX), "trivial characters: real blocks, pipelined loop");
    const int nb = d.n_bonds;
    // Diagonal: sum_b Jz_b (+1/4 if the spins of b are equal, -1/4 if not)
    // = (1/4) sum_b Jz_b - (1/2) sum over the unequal-spin bonds of Jz_b; the
    // second sum is taken in the walk over those bonds below.
    A junq = 0;
    A acc[NV * C];
#pragma unroll
    for (int v = 0; v < NV * C; ++v) acc[v] = 0;
    A rn = S.rsq[gld(d.stab + row)];
    // explicit fused multiply-adds: a complex kernel on a block with real
    // characters (ai = 0) rounds exactly like the real kernel
    auto add = [&](A ar, A ai, const T *xv) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if constexpr (CPLX) {
                const A xr = xv[2 * v], xi = xv[2 * v + 1];
                acc[2 * v] = fmadd<A>(-ai, xi, fmadd<A>(ar, xr, acc[2 * v]));
                acc[2 * v + 1] = fmadd<A>(ai, xr, fmadd<A>(ar, xi, acc[2 * v + 1]));
            } else {
                acc[v] = fmadd<A>(ar, (A)xv[v], acc[v]);
            }
        }
    };
    // PIPE: the pending term.  ALL: every term has a slot (packed form of the
    // rank-addressed x), so none is tested; the first one pending adds 0 * 0.
    constexpr bool ALL = FORM == FORM_PACKED && XR != 0;
    bool p_ok = ALL;
    A p_ar = 0, p_ai = 0;
    T p_x[NV * C];
#pragma unroll
    for (int v = 0; v < NV * C; ++v) p_x[v] = T(0);
    // key: the packed sublattice search's key of the term's state, if given
    auto term = [&](const B &bd, W t, const SubKey *key) {
        int u, cnt;
        auto idx = locate<W, KIND, A, XR, FORM>(d, S, t, u, cnt, key);
        A hs = bd.h;
        if constexpr (KIND == K_SUB && XR == 0)
            if (d.umap && idx >= 0) idx = user_pos<A>(d, idx, hs);
        if constexpr (PIPE) {
            // the gather is issued for every term (row 0 when the orbit is
            // not in the block: a valid address, never added)
            const bool ok = ALL || idx >= 0;
            A ar = 0, ai = 0;
            if (ok) {
                const A f = hs * S.sq[cnt];
                if constexpr (XR == 2) {
                    ar = f;   // chi(u) = 1
                } else {
                    const auto c = S.chi[u];
                    ar = f * c.x;
                    if constexpr (CPLX) ai = f * c.y;
                }
            }
            // the previous gather (issued one search ago) is added first, so
            // that the new one can land in the same registers
            if (ALL || p_ok) add(p_ar, p_ai, p_x);
            const size_t xb =
                ((size_t)(ok ? idx : 0) * (XR != 0 ? (int64_t)d.xr_cols : nvec) + v0) * C;
#pragma unroll
            for (int v = 0; v < NV * C; ++v) p_x[v] = gld(XT + xb + v);
            p_ok = ALL || ok;
            p_ar = ar;
            p_ai = ai;
            return;
        }
        if (idx < 0) return;
        const A f = hs * S.sq[cnt];   // times 1/sqrt|Stab r| once per row
        const auto c = S.chi[u];
        const A ar = f * c.x;
        A ai = 0;
        if constexpr (CPLX) ai = f * c.y;
        // 32-bit states: positions below 2^31, one 32 x 32 -> 64-bit multiply-add
        const size_t xb = sizeof(W) == 4
                              ? (uint64_t)(uint32_t)idx * (uint32_t)(nvec * C) + (uint64_t)(v0 * C)
                              : ((size_t)idx * nvec + v0) * C;
        // explicit fused multiply-adds: a complex kernel on a block with real
        // characters (ai = 0) rounds exactly like the real kernel
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if constexpr (CPLX) {
                const A xr = gld(XT + xb + 2 * v), xi = gld(XT + xb + 2 * v + 1);
                acc[2 * v] = fmadd<A>(-ai, xi, fmadd<A>(ar, xr, acc[2 * v]));
                acc[2 * v + 1] = fmadd<A>(ai, xr, fmadd<A>(ar, xi, acc[2 * v + 1]));
            } else {
                acc[v] = fmadd<A>(ar, (A)gld(XT + xb + v), acc[v]);
            }
        }
    };
    if constexpr (KIND == K_AFF) {
        // Cheap searches: per group of 32 bonds, a mask of the bonds with
        // unequal spins, walked lowest first (the order of the plain bond
        // loop), so that a wave iterates over its lanes' active bonds only.
        // Bonds b = (b, b + 1 mod N) in order: bit b of s ^ rotr(s, 1).
        const W walls = d.ring_bonds ? (s ^ rotr_n<W>(s, 1, d.n_sites)) : W(0);
        for (int b0 = 0; b0 < nb; b0 += 32) {
            const int bn = nb - b0 < 32 ? nb - b0 : 32;
            uint32_t act = 0;
            if (d.ring_bonds) {
                act = (uint32_t)(walls >> b0) & (bn == 32 ? ~0u : ((1u << bn) - 1u));
            } else {
                for (int k = 0; k < bn; ++k) {
                    const B bd = S.bonds[b0 + k];
                    act |= (((uint32_t)(s >> bd.i) ^ (uint32_t)(s >> bd.j)) & 1u) << k;
                }
            }
            while (act) {
                const int b = b0 + __builtin_ctz(act);
                act &= act - 1;
                const B bd = S.bonds[b];
                junq += bd.jz;
                term(bd, s ^ ((W(1) << bd.i) | (W(1) << bd.j)), nullptr);
            }
        }
    } else {
        // Table searches: all lanes take the same bond at the same time, so
        // that neighbouring rows walk similar table entries and look up
        // neighbouring index words.
        bool done = false;
        if constexpr (KIND == K_SUB && FORM != FORM_BLOCKS) {
            if (FORM == FORM_PACKED || (S.subf && d.bx)) {
                // packed form: the bond comes with scalar loads, the term's key
                // is the row's key with the bond's bits flipped
                const SubKey kr = sub_key<W>(s, d.m, d.pb);
                for (int b = 0; b < nb; ++b) {
                    const BondX x = sld(d.bx + b);
                    const B bd = sld(reinterpret_cast<const B *>(d.bonds) + b);
                    const W fl = (W)x.flip, sf = s & fl;
                    if (sf == 0 || sf == fl) continue;
                    junq += bd.jz;
                    const SubKey kt = sub_key_flip(kr, x);
                    term(bd, s ^ fl, &kt);
                }
                if constexpr (PIPE) {
                    if (ALL || p_ok) add(p_ar, p_ai, p_x);
                }
                done = true;
            }
        }
        if constexpr (FORM != FORM_PACKED) if (!done) {
            for (int b = 0; b < nb; ++b) {
                const B bd = S.bonds[b];
                if (((s >> bd.i) & 1) == ((s >> bd.j) & 1)) continue;
                junq += bd.jz;
                term(bd, s ^ ((W(1) << bd.i) | (W(1) << bd.j)), nullptr);
            }
            if constexpr (PIPE) {
                if (ALL || p_ok) add(p_ar, p_ai, p_x);
                p_ok = false;
            }
        }
    }
    // (the caller's position is read here and not before the terms: a register
    // pair held over the search costs the 64-register copies spills)
    int64_t orow = row;
    if constexpr (KIND == K_SUB)
        if (d.umap) orow = user_pos<A>(d, row, rn);
    const size_t base = ((size_t)orow * nvec + v0) * C;
    const A diag = (A)d.jz_quarter - A(0.5) * junq;
    // the row's x is read before its first store: y may alias x for the
    // compiler, and with a read between any two stores the parts of a row's
    // line left the L2 one by one (ring N = 28, every momentum, complex64 x 8:
    // 8.22 -> 6.06 ms, 7.7 -> 2.57 GB written, 32 -> 15.6 GB fetched)
    T xd[NV * C];
#pragma unroll
    for (int v = 0; v < NV * C; ++v) xd[v] = gld(X + base + v);
#pragma unroll
    for (int v = 0; v < NV * C; ++v)
        gst(Y + base + v, (T)fmadd<A>(diag, (A)xd[v], rn * acc[v]));
}

// A row of a full ring with equal neighbour bonds: the terms, their order and
// every rounding of the general loop, so the results agree bitwise.  What
// bounds it is the number of vector instructions of a term (32 sites: 112 of
// them, 88 % of the issue slots in the general loop).  The exchanged pair is
// made from the lowest set bit of the walls; the amplitudes h sqrt(c) and the
// sums of k equal Jz are tables, rounded as the loop rounds them; the search
// tests no rotation length.  TRIV, every character 1: all orbits are in the
// block and no element is needed, so neither the index bit nor the character
// is looked at.  Ring N = 32, k = 0, FP32: 1.166 -> 0.974 ms; N = 28, every
// momentum, complex64 x 8: 6.06 -> 5.71 ms.  (The 64-register copy kept 27
// vector and 35 scalar registers in memory in the general loop, here 3 and 0.)
template <class W, class T, class A, bool CPLX, int NV, bool FULL, bool TRIV>
__device__ __forceinline__ void process_ring(const SectorDesc &d, const Staged<A> &S, int64_t row,
                                             int64_t nvec, int v0) {
    constexpr int C = CPLX ? 2 : 1;
    const int N = FULL ? 8 * (int)sizeof(W) : d.n_sites;
    const W mask = FULL ? ~W(0) : (W(1) << N) - 1;
    const W s = gld(reinterpret_cast<const W *>(d.reps) + row);
    const T *X = reinterpret_cast<const T *>(d.x) + (size_t)v0 * C;
    T *Y = reinterpret_cast<T *>(d.y) + (size_t)v0 * C;
    const bool dense = nvec == NV;   // one pass: the row stride is a constant
    W act = s ^ rot_r<W, FULL>(s, 1, N, mask);   // bit b: the spins of bond b differ
    const A junq = S.jsum[sizeof(W) == 4 ? __popc((uint32_t)act) : __popcll((uint64_t)act)];
    A acc[NV * C];
#pragma unroll
    for (int v = 0; v < NV * C; ++v) acc[v] = 0;
    while (act) {
        const W bit = act & (W(0) - act);
        act ^= bit;
        const W t = s ^ (bit | rot_l<W, FULL>(bit, 1, N, mask));
        W rep;
        int u, cnt;
        ring_scan_big<W, FULL, TRIV, true>(t, N, mask, S.ring_gidx, rep, u, cnt);
        if (d.ring == 2)
            ring_scan_big<W, FULL, TRIV, false>(rev_n<W>(t, N), N, mask, S.ring_gidx + N, rep, u,
                                                cnt);
        typename IndexT<W>::type idx;
        if constexpr (sizeof(W) == 4) {
            const uint32_t r = (uint32_t)colex_rank<W>(S.rtab, d.rl, rep);
            if constexpr (TRIV) {
                const uint64_t e = gld(reinterpret_cast<const uint64_t *>(d.rwords) + (r >> 5));
                idx = (int32_t)((uint32_t)e +
                                __popc((uint32_t)(e >> 32) & ((1u << (r & 31u)) - 1u)));
            } else {
                idx = rank_find32(d.rwords, (uint32_t)d.n_rwords, r);
            }
        } else if (d.rl.e32) {
            const uint32_t r = colex_rank_sat<W>(static_cast<const uint32_t *>(S.rtab), d.rl, rep);
            idx = r == 0xFFFFFFFFu ? -1 : rank_find_r32(d.rwords, (uint32_t)d.n_rwords, r);
        } else {
            idx = rank_find(d.rwords, d.n_rwords, colex_rank<W>(S.rtab, d.rl, rep));
        }
        if (!(TRIV && sizeof(W) == 4) && idx < 0) continue;
        const A f = S.hs[cnt];
        A ar = f, ai = 0;
        if constexpr (!TRIV) {
            const auto c = S.chi[u];
            ar = f * c.x;
            if constexpr (CPLX) ai = f * c.y;
        }
        const size_t at = sizeof(W) == 4 ? (size_t)(uint32_t)idx : (size_t)idx;
        const T *q = X + (dense ? at * (NV * C)
                          : sizeof(W) == 4 ? (uint64_t)(uint32_t)at * (uint32_t)(nvec * C)
                                           : at * (size_t)(nvec * C));
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if constexpr (CPLX) {
                const A xr = gld(q + 2 * v), xi = gld(q + 2 * v + 1);
                acc[2 * v] = fmadd<A>(-ai, xi, fmadd<A>(ar, xr, acc[2 * v]));
                acc[2 * v + 1] = fmadd<A>(ai, xr, fmadd<A>(ar, xi, acc[2 * v + 1]));
            } else {
                acc[v] = fmadd<A>(ar, (A)gld(q + v), acc[v]);
            }
        }
    }
    const A rn = S.rsq[gld(d.stab + row)];
    const size_t base = (size_t)row * nvec * C;
    const A diag = (A)d.jz_quarter - A(0.5) * junq;
    T xd[NV * C];
#pragma unroll
    for (int v = 0; v < NV * C; ++v) xd[v] = gld(X + base + v);
#pragma unroll
    for (int v = 0; v < NV * C; ++v)
        gst(Y + base + v, (T)fmadd<A>(diag, (A)xd[v], rn * acc[v]));
}

// ------------------------------------------------ wave-compacted term loop --
// For the table searches (sublattice coding, byte tables) the row loop above
// takes every bond with all lanes of the wave at once, so on each bond only
// the lanes whose spins differ there (about half) do a term.  Here a wave
// owns a window of 64 + CMP_EXTRA consecutive rows (a second row on the
// first CMP_EXTRA lanes) and, bond by bond, packs the unequal-spin terms of
// the window into passes of up to 64: every lane of a pass takes the same
// bond, as in the row loop, but most lanes have a term.  Terms move between
// lanes with cross-lane permutes (no LDS): each owner pushes its row to the
// lane that will do its term, that lane pulls the row state, computes the
// term, and the owner pulls the amplitude and the gathered x back and adds
// them with the same fused multiply-adds, in bond order, so that both loops
// give bitwise identical rows.
constexpr int CMP_EXTRA = 48;
constexpr int CMP_ROWS = 64 + CMP_EXTRA;   // rows per wave window

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

__device__ __forceinline__ int rank_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ int pull32(int src_lane, int v) {
    return __builtin_amdgcn_ds_bpermute(src_lane << 2, v);
}

template <class V>
__device__ __forceinline__ V pull(int src_lane, V v) {
    if constexpr (sizeof(V) == 4) {
        return __builtin_bit_cast(V, pull32(src_lane, __builtin_bit_cast(int, v)));
    } else {
        static_assert(sizeof(V) == 8, "8-byte value");
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const int lo = pull32(src_lane, (int)(uint32_t)u);
        const int hi = pull32(src_lane, (int)(uint32_t)(u >> 32));
        return __builtin_bit_cast(V, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    }
}

// Lanes with `mine` send `val` to lane `dest` (dest distinct, all inside the
// range [lo, hi)); every other lane sends to one of the lanes outside that
// range, so that the permute is a bijection (a lane that is not a
// destination of any sender would receive an undefined value).  Returns what
// this lane received.
__device__ __forceinline__ int push_range(bool mine, int dest, int lo, int hi, int val) {
    const uint64_t other = __ballot(!mine);
    const int d = mine ? dest : ((hi + rank_below(other)) & 63);
    (void)lo;
    return __builtin_amdgcn_ds_permute(d << 2, val);
}

template <class W, int KIND, class T, class A, bool CPLX, int NV>
__device__ __forceinline__ void process_window(const SectorDesc &d, const Staged<A> &S,
                                               int64_t w0, int64_t r1, int64_t nvec, int v0) {
    using B = typename BondT<A>::type;
    constexpr int C = CPLX ? 2 : 1;
    const int lane = lane_id();
    const int64_t row0 = w0 + lane, row1 = w0 + 64 + lane;
    const bool ok0 = row0 < r1, ok1 = lane < CMP_EXTRA && row1 < r1;
    const W *R = reinterpret_cast<const W *>(d.reps);
    const W s0 = ok0 ? gld(R + row0) : W(0);
    const W s1 = ok1 ? gld(R + row1) : W(0);
    const T *X = reinterpret_cast<const T *>(d.x);
    T *Y = reinterpret_cast<T *>(d.y);
    const int nb = d.n_bonds;
    A acc0[NV * C], acc1[NV * C];
#pragma unroll
    for (int v = 0; v < NV * C; ++v) acc0[v] = acc1[v] = 0;
    auto unequal = [](W s, const B &bd) -> bool {
        return (((uint32_t)(s >> bd.i)) ^ ((uint32_t)(s >> bd.j))) & 1u;
    };
    auto add = [&](A *acc, A ar, A ai, const T *xq) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if constexpr (CPLX) {
                const A xr = xq[2 * v], xi = xq[2 * v + 1];
                acc[2 * v] = fmadd<A>(-ai, xi, fmadd<A>(ar, xr, acc[2 * v]));
                acc[2 * v + 1] = fmadd<A>(ai, xr, fmadd<A>(ar, xi, acc[2 * v + 1]));
            } else {
                acc[v] = fmadd<A>(ar, (A)xq[v], acc[v]);
            }
        }
    };
    for (int b = 0; b < nb; ++b) {
        const B bd = S.bonds[b];
        const bool a0 = ok0 && unequal(s0, bd), a1 = ok1 && unequal(s1, bd);
        const uint64_t M0 = __ballot(a0), M1 = __ballot(a1);
        const int n0 = __popcll(M0), n = n0 + __popcll(M1);
        // term index of this lane's row-0 and row-1 terms (row 0 terms first)
        const int e0 = rank_below(M0), e1 = n0 + rank_below(M1);
        const W flip = (W(1) << bd.i) | (W(1) << bd.j);
        for (int p = 0; p < n; p += 64) {
            const int take = n - p < 64 ? n - p : 64;
            // pass lanes [lo0, hi0) take row-0 terms, [hi0, take) row-1 terms
            const int lo0 = 0, hi0 = n0 - p < 0 ? 0 : (n0 - p < take ? n0 - p : take);
            const bool m0 = a0 && e0 >= p && e0 < p + take;
            const bool m1 = a1 && e1 >= p && e1 < p + take;
            const int g0 = push_range(m0, e0 - p, lo0, hi0, lane);
            const int g1 = push_range(m1, e1 - p, hi0, take, lane);
            const bool has = lane < take;
            const bool second = lane >= hi0;
            const int src = second ? g1 : g0;   // owner lane of this pass lane's term
            const W t0 = pull<W>(src, s0), t1 = pull<W>(src, s1);
            bool ok = false;
            A ar = 0, ai = 0;
            T xv[NV * C];
#pragma unroll
            for (int v = 0; v < NV * C; ++v) xv[v] = T(0);
            if (has) {
                const W t = (second ? t1 : t0) ^ flip;
                int u, cnt;
                auto idx = locate<W, KIND, A>(d, S, t, u, cnt);
                if (idx >= 0) {
                    ok = true;
                    A hs = bd.h;
                    if constexpr (KIND == K_SUB)
                        if (d.umap) idx = user_pos<A>(d, idx, hs);
                    const A f = hs * S.sq[cnt];
                    const auto c = S.chi[u];
                    ar = f * c.x;
                    if constexpr (CPLX) ai = f * c.y;
                    const size_t xb = sizeof(W) == 4
                                          ? (uint64_t)(uint32_t)idx * (uint32_t)(nvec * C) +
                                                (uint64_t)(v0 * C)
                                          : ((size_t)idx * nvec + v0) * C;
#pragma unroll
                    for (int v = 0; v < NV * C; ++v) xv[v] = gld(X + xb + v);
                }
            }
            // owners pull their terms back: row 0, then row 1
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool mine = h == 0 ? m0 : m1;
                const int from = mine ? (h == 0 ? e0 : e1) - p : lane;
                const bool okq = pull32(from, (int)ok) != 0;
                const A arq = pull<A>(from, ar);
                A aiq = 0;
                if constexpr (CPLX) aiq = pull<A>(from, ai);
                T xq[NV * C];
#pragma unroll
                for (int v = 0; v < NV * C; ++v) xq[v] = pull<T>(from, xv[v]);
                if (mine && okq) add(h == 0 ? acc0 : acc1, arq, aiq, xq);
            }
        }
    }
    // the diagonal, (1/4) sum_b Jz_b - (1/2) sum over the unequal-spin bonds
    // (bond order, as in the row loop), and the stores
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const bool okh = h == 0 ? ok0 : ok1;
        if (!okh) continue;
        const W sh = h == 0 ? s0 : s1;
        const int64_t row = h == 0 ? row0 : row1;
        A junq = 0;
        for (int b = 0; b < nb; ++b) {
            const B bd = S.bonds[b];
            if (unequal(sh, bd)) junq += bd.jz;
        }
        A rn = S.rsq[gld(d.stab + row)];
        int64_t orow = row;
        if constexpr (KIND == K_SUB)
            if (d.umap) orow = user_pos<A>(d, row, rn);
        const size_t base = ((size_t)orow * nvec + v0) * C;
        const A diag = (A)d.jz_quarter - A(0.5) * junq;
        const A *acc = h == 0 ? acc0 : acc1;
#pragma unroll
        for (int v = 0; v < NV * C; ++v)
            gst(Y + base + v, (T)fmadd<A>(diag, (A)gld(X + base + v), rn * acc[v]));
    }
}

// --------------------------------------------------------- few-rows loop --
// A block of few rows leaves most of the chip idle when every lane owns a
// row, and the time is one lane's chain of n_bonds searches (6x6 triangular
// lattice, 1772 rows: 1.0 ms).  Here a wave takes `few` rows at once: first
// its lanes share out the (row, bond) pairs and leave each term's amplitude
// and position in LDS, then a lane per (row, vector) adds the terms in bond
// order with the fused multiply-adds of the row loop, so that both loops give
// the same bits.  All vectors share the search, whatever their number.
constexpr uint32_t NO_TERM = 0xFFFFFFFFu;

template <class A>
__host__ __device__ constexpr size_t few_bytes(bool cplx, int terms) {
    return ((size_t)terms * (sizeof(A) * (cplx ? 2 : 1) + 4) + 15) & ~(size_t)15;
}

template <class W, int KIND, class T, class A, bool CPLX>
__device__ __forceinline__ void process_few(const SectorDesc &d, const Staged<A> &S, int64_t r0,
                                            int64_t r1, int64_t wave, int64_t waves, int few,
                                            unsigned char *scratch, int64_t nvec) {
    static_assert(KIND != K_U1, "a term without a group is too cheap to share out");
    using B = typename BondT<A>::type;
    constexpr int C = CPLX ? 2 : 1;
    const int lane = (int)__lane_id();
    const uint32_t nb = (uint32_t)d.n_bonds, cols = (uint32_t)nvec;
    const W *R = reinterpret_cast<const W *>(d.reps);
    const T *X = reinterpret_cast<const T *>(d.x);
    T *Y = reinterpret_cast<T *>(d.y);
    A *amp = reinterpret_cast<A *>(scratch);
    uint32_t *pos = reinterpret_cast<uint32_t *>(amp + (size_t)few * nb * C);
    for (int64_t w0 = r0 + wave * few; w0 < r1; w0 += waves * few) {
        const uint32_t nr = (uint32_t)(r1 - w0 < few ? r1 - w0 : few);
        for (uint32_t e = lane; e < nr * nb; e += 64) {
            const uint32_t r = e / nb, b = e - r * nb;
            const W s = gld(R + w0 + r);
            const B bd = S.bonds[b];
            uint32_t at = NO_TERM;
            if (((s >> bd.i) & 1) != ((s >> bd.j) & 1)) {
                int u, cnt;
                auto idx = locate<W, KIND, A>(d, S, s ^ ((W(1) << bd.i) | (W(1) << bd.j)), u, cnt);
                if (idx >= 0) {
                    A hs = bd.h;
                    if constexpr (KIND == K_SUB)
                        if (d.umap) idx = user_pos<A>(d, idx, hs);
                    const A f = hs * S.sq[cnt];
                    const auto c = S.chi[u];
                    if constexpr (CPLX) amp[2 * e + 1] = f * c.y;
                    amp[C * e] = f * c.x;
                    at = (uint32_t)idx;
                }
            }
            pos[e] = at;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t q = lane; q < nr * cols; q += 64) {
            const uint32_t r = q / cols, v = q - r * cols;
            const int64_t row = w0 + r;
            const W s = gld(R + row);
            A junq = 0, re = 0, im = 0;
#pragma unroll 4
            for (uint32_t b = 0; b < nb; ++b) {
                const B bd = S.bonds[b];
                const bool off = ((s >> bd.i) & 1) != ((s >> bd.j) & 1);
                junq = off ? junq + bd.jz : junq;
                const uint32_t e = r * nb + b, at = pos[e];
                // no term: position 0 is read and not added
                const size_t xb = ((size_t)(at == NO_TERM ? 0u : at) * cols + v) * C;
                const A ar = at == NO_TERM ? A(0) : amp[C * e];
                const A xr = (A)gld(X + xb);
                if constexpr (CPLX) {
                    const A ai = at == NO_TERM ? A(0) : amp[2 * e + 1];
                    const A xi = (A)gld(X + xb + 1);
                    const A nr_ = fmadd<A>(-ai, xi, fmadd<A>(ar, xr, re));
                    const A ni_ = fmadd<A>(ai, xr, fmadd<A>(ar, xi, im));
                    re = at == NO_TERM ? re : nr_;
                    im = at == NO_TERM ? im : ni_;
                } else {
                    const A n_ = fmadd<A>(ar, xr, re);
                    re = at == NO_TERM ? re : n_;
                }
            }
            A rn = S.rsq[gld(d.stab + row)];
            int64_t orow = row;
            if constexpr (KIND == K_SUB)
                if (d.umap) orow = user_pos<A>(d, row, rn);
            const size_t base = ((size_t)orow * cols + v) * C;
            const A diag = (A)d.jz_quarter - A(0.5) * junq;
            gst(Y + base, (T)fmadd<A>(diag, (A)gld(X + base), rn * re));
            if constexpr (CPLX)
                gst(Y + base + 1, (T)fmadd<A>(diag, (A)gld(X + base + 1), rn * im));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// rows [r0, r1) of a sector.  LOOP_CMP: windows of CMP_ROWS rows per wave
// (every lane of a wave takes part in its permutes; `first` and `stride`
// count lanes, so wave w of the launch starts at window w); LOOP_FEW: `few`
// rows per wave, all vectors; otherwise a lane per row, reading the
// rank-addressed x when XR.  LOOP_PACKED, LOOP_BLOCKS: the lane-per-row loop of
// a single block in that sublattice form and nothing else, LOOP_BATCH_*: of a
// batch of such blocks (see launch_nv);
// LOOP_RING: the rows of process_ring; LOOP_OWN: those of process_row_own.
template <class W, int KIND, class T, class A, bool CPLX, int NV, int LOOP, int XR, bool PIPE>
__device__ __forceinline__ void process_range(const SectorDesc &d, const Staged<A> &S, int64_t r0,
                                              int64_t r1, int64_t first, int64_t stride,
                                              int64_t nvec, int v0, int few,
                                              unsigned char *few_terms) {
    constexpr int form = form_of_loop(LOOP);
    if constexpr (LOOP == LOOP_FEW) {
        process_few<W, KIND, T, A, CPLX>(
            d, S, r0, r1, (first - lane_id()) / 64, stride / 64, few,
            few_terms + (threadIdx.x / 64) * few_bytes<A>(CPLX, few * d.n_bonds), nvec);
    } else if constexpr (LOOP == LOOP_RING) {
        auto rows = [&](auto full, auto one) {
            for (int64_t row = r0 + first; row < r1; row += stride)
                process_ring<W, T, A, CPLX, NV, decltype(full)::value, decltype(one)::value>(
                    d, S, row, nvec, v0);
        };
        using std::false_type;
        using std::true_type;
        auto form = [&](auto full) {
            if constexpr (CPLX) {
                rows(full, false_type{});
            } else {
                if (d.chi_one) rows(full, true_type{});
                else rows(full, false_type{});
            }
        };
        if constexpr (sizeof(W) == 4) {
            if (d.n_sites == 32) form(true_type{});
            else form(false_type{});
        } else {
            form(false_type{});
        }
    } else if constexpr (LOOP == LOOP_CMP) {
        const int64_t wave = (first - lane_id()) / 64, waves = stride / 64;
        for (int64_t w0 = r0 + wave * CMP_ROWS; w0 < r1; w0 += waves * CMP_ROWS)
            process_window<W, KIND, T, A, CPLX, NV>(d, S, w0, r1, nvec, v0);
    } else {
        for (int64_t row = r0 + first; row < r1; row += stride)
            if constexpr (LOOP == LOOP_OWN)
                process_row_own<W, T, A, NV>(d, S, row, nvec, v0);
            else if constexpr (KIND == K_U1)
                process_row_u1<W, T, A, NV>(d, S, row, nvec, v0);
            else
                process_row<W, KIND, T, A, CPLX, NV, XR, PIPE, form>(d, S, row, nvec, v0);
    }
}

// count of the off-diagonal terms of a row that land in the block
template <class W, int KIND>
__device__ __forceinline__ uint32_t count_row(const SectorDesc &d, const Staged<double> &S,
                                              int64_t row) {
    const W s = reinterpret_cast<const W *>(d.reps)[row];
    uint32_t n = 0;
    for (int b = 0; b < d.n_bonds; ++b) {
        const BondD bd = S.bonds[b];
        if (((s >> bd.i) & 1) == ((s >> bd.j) & 1)) continue;
        const W t = s ^ ((W(1) << bd.i) | (W(1) << bd.j));
        int u, cnt;
        if (locate<W, KIND, double>(d, S, t, u, cnt) >= 0) ++n;
    }
    return n;
}

template <class W, int KIND, class T, class AC, bool CPLX, int NV, bool STAGE, bool OCC,
          int LOOP, int XR>
__global__ __launch_bounds__(APPLY_BLOCK, OCC ? OCC_WAVES : 1) void k_apply(ApplyArgs A) {
    // the sublattice row loop pipelines its gathers
    constexpr bool SINGLE = LOOP == LOOP_PACKED || LOOP == LOOP_BLOCKS;
    constexpr bool BATCH = LOOP == LOOP_BATCH_PACKED || LOOP == LOOP_BATCH_BLOCKS;
    constexpr bool PIPE = KIND == K_SUB && (LOOP == LOOP_ROW || SINGLE || BATCH);
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *few_terms = smem + A.few_off;
    __shared__ uint32_t s_tile;
    __shared__ SectorDesc s_desc;
    Staged<AC> S;
    if constexpr (!BATCH) if (SINGLE || A.descs == nullptr) {
        const SectorDesc &d = A.one;
        stage<KIND, AC, STAGE, LOOP>(d, smem, S);
        __syncthreads();
        const int64_t stride = (int64_t)gridDim.x * blockDim.x;
        process_range<W, KIND, T, AC, CPLX, NV, LOOP, XR, PIPE>(
            d, S, 0, d.dim, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride, A.nvec, A.v0,
            A.few, few_terms);
        return;
    }
    // persistent: (sector, row tile) items from one queue
    if constexpr (!SINGLE) for (int cur = -1;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(A.queue, 1u);
        __syncthreads();
        const uint32_t tile = s_tile;
        if (tile >= A.n_tiles) break;
        int lo = 0, hi = A.n_secs - 1;   // last sector with tile_prefix <= tile
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (A.tile_prefix[mid] <= tile) lo = mid; else hi = mid - 1;
        }
        if (lo != cur) {
            // no group: a word per lane.  As one lane's copy it held 64 registers,
            // which cost kernels of three vectors the second workgroup of a compute
            // unit (ring N = 24, FP32 x 3: 89 -> 67 us); with the searches of the
            // other kinds the loop spills 8 bytes more instead.
            if constexpr (KIND == K_U1) {
                for (uint32_t e = threadIdx.x; e < sizeof(SectorDesc) / 4; e += blockDim.x)
                    reinterpret_cast<uint32_t *>(&s_desc)[e] =
                        reinterpret_cast<const uint32_t *>(A.descs + lo)[e];
            } else {
                if (threadIdx.x == 0) s_desc = A.descs[lo];
            }
            __syncthreads();
            stage<KIND, AC, STAGE, LOOP>(s_desc, smem, S);
            __syncthreads();
            cur = lo;
        }
        const SectorDesc &d = s_desc;
        const int64_t r0 = (int64_t)(tile - A.tile_prefix[lo]) * A.tile_rows;
        int64_t r1 = r0 + A.tile_rows;
        r1 = r1 < d.dim ? r1 : d.dim;
        process_range<W, KIND, T, AC, CPLX, NV, LOOP, XR, PIPE>(
            d, S, r0, r1, threadIdx.x, blockDim.x, A.nvec, A.v0, A.few, few_terms);
        __syncthreads();
    }
}

template <class W, int KIND, bool STAGE>
__global__ __launch_bounds__(APPLY_BLOCK) void k_count(ApplyArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned long long s_sum;
    Staged<double> S;
    const SectorDesc &d = A.one;
    stage<KIND, double, STAGE>(d, smem, S);
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    unsigned long long n = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < d.dim; row += stride)
        n += count_row<W, KIND>(d, S, row);
    atomicAdd(&s_sum, n);
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(A.count, s_sum);
}

static __global__ void k_zero_u32(uint32_t *p) { *p = 0; }

// Host launcher for one search kind (instantiated in one translation unit per
// kind).  `single`: FP32 vectors; `acc64`: FP64 amplitudes and accumulation
// (always for FP64 vectors).
template <int KIND>
int launch_kind(bool wide, bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A,
                unsigned grid, unsigned block, size_t lds, hipStream_t st);

template <int KIND>
int launch_count_kind(bool wide, const ApplyArgs &A, unsigned grid, unsigned block, size_t lds,
                      hipStream_t st);

// The sublattice kernels whose terms read the rank-addressed x: any
// characters, and every character 1 (one translation unit each).
int launch_sub_xr(bool wide, bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A,
                  unsigned grid, unsigned block, size_t lds, hipStream_t st);
int launch_sub_xr_trivial(bool wide, bool single, bool acc64, int nv, const ApplyArgs &A,
                          unsigned grid, unsigned block, size_t lds, hipStream_t st);

// Kernels with 64 VGPRs, by the accumulator scalars of a lane: with more than
// two it spills them (complex 8-vector passes: 200 bytes); the rank-addressed
// kernels up to four.
constexpr int occ_scalars(int xr) { return xr ? 4 : 2; }
// Vectors per pass of the rank-addressed kernels: at most eight scalars.
constexpr int xr_max_nv(bool cplx) { return cplx ? 4 : 8; }

template <class W, int KIND, class T, class AC, bool CPLX, bool STAGE, bool OCC, int LOOP, int XR,
          int NV = 1>
void (*apply_kernel(int nv))(ApplyArgs) {
    constexpr int most = LOOP == LOOP_CMP ? 2 : XR ? xr_max_nv(CPLX) : 8;
    constexpr int limit = OCC ? occ_scalars(XR) / (CPLX ? 2 : 1) : most;
    if constexpr (NV <= (limit < most ? limit : most)) {
        if (nv == NV) return k_apply<W, KIND, T, AC, CPLX, NV, STAGE, OCC, LOOP, XR>;
        return apply_kernel<W, KIND, T, AC, CPLX, STAGE, OCC, LOOP, XR, NV + 1>(nv);
    }
    return nullptr;
}

template <class W, int KIND, class T, class AC, bool CPLX, int XR>
int launch_nv(int nv, const ApplyArgs &A, unsigned grid, unsigned block, size_t lds,
              hipStream_t st) {
    void (*f)(ApplyArgs) = nullptr;
    const bool occ = A.occ && nv * (CPLX ? 2 : 1) <= occ_scalars(XR);
    // the compacted loop takes passes of one or two vectors, the row loop the others
    const bool cmp = A.compact && nv <= 2;
    if constexpr (KIND == K_SUB && !(XR == 2 && CPLX)) {
        // The row loop of each search, for one block and for a batch, is a kernel of
        // its own: with both searches and both launches in one it held 128 registers
        // (one block: packed 47, by blocks 45), and its 64-register copy kept 290
        // bytes in memory.  5x6 square numbered row by row, 15 up, 2.6 M rows, FP64:
        // 2.75 ms with both, 2.59 apart; eight vectors 3.70 and 3.04 ms; a batch of
        // two 4x6 J1-J2 blocks, 9 up: 123 and 118 us.
        const bool packed = A.descs ? A.packed != 0 : A.one.subf && A.one.bx;
        auto row = [&](auto loop) {
            constexpr int L = decltype(loop)::value;
            f = occ ? apply_kernel<W, KIND, T, AC, CPLX, true, true, L, XR>(nv)
                    : apply_kernel<W, KIND, T, AC, CPLX, true, false, L, XR>(nv);
        };
        if constexpr (XR != 0) {   // single blocks with their tables in LDS
            if (A.stage_sub && packed)
                row(std::integral_constant<int, LOOP_PACKED>{});
            else if (A.stage_sub)
                row(std::integral_constant<int, LOOP_BLOCKS>{});
        } else if (!A.stage_sub) {
            f = cmp ? apply_kernel<W, KIND, T, AC, CPLX, false, false, LOOP_CMP, 0>(nv)
                    : apply_kernel<W, KIND, T, AC, CPLX, false, false, LOOP_ROW, 0>(nv);
        } else if (A.few) {
            f = k_apply<W, KIND, T, AC, CPLX, 1, true, false, LOOP_FEW, 0>;
        } else if (cmp) {
            row(std::integral_constant<int, LOOP_CMP>{});
        } else if (A.descs) {
            if (packed)
                row(std::integral_constant<int, LOOP_BATCH_PACKED>{});
            else
                row(std::integral_constant<int, LOOP_BATCH_BLOCKS>{});
        } else if (packed) {
            row(std::integral_constant<int, LOOP_PACKED>{});
        } else {
            row(std::integral_constant<int, LOOP_BLOCKS>{});
        }
    } else if constexpr (KIND != K_SUB) {
        auto row = [&](auto loop) {
            constexpr int L = decltype(loop)::value;
            f = occ ? apply_kernel<W, KIND, T, AC, CPLX, true, true, L, 0>(nv)
                    : apply_kernel<W, KIND, T, AC, CPLX, true, false, L, 0>(nv);
        };
        if constexpr (KIND == K_U1) {
            if (A.own)
                row(std::integral_constant<int, LOOP_OWN>{});
            else
                row(std::integral_constant<int, LOOP_ROW>{});
        } else if (A.few) {
            f = k_apply<W, KIND, T, AC, CPLX, 1, true, false, LOOP_FEW, 0>;
        } else if (KIND == K_AFF && A.ring) {
            if constexpr (KIND == K_AFF) row(std::integral_constant<int, LOOP_RING>{});
        } else if (KIND == K_TAB && cmp) {
            if constexpr (KIND == K_TAB) row(std::integral_constant<int, LOOP_CMP>{});
        } else {
            row(std::integral_constant<int, LOOP_ROW>{});
        }
    }
    if (!f) {
        set_error("no kernel for %d vectors per pass (1 to 8; the rank-addressed x: at most eight "
                  "scalars, tables in LDS)", nv);
        return XDG_EINVAL;
    }
    if (lds > 65536)
        XDG_TRY_HIP(hipFuncSetAttribute((const void *)f,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(f, dim3(grid), dim3(block), lds, st, A);
    XDG_TRY_HIP(hipGetLastError());
    return XDG_OK;
}

template <class W, int KIND, bool CPLX, int XR>
int launch_prec(bool single, bool acc64, int nv, const ApplyArgs &A, unsigned grid,
                unsigned block, size_t lds, hipStream_t st) {
    if (!single) return launch_nv<W, KIND, double, double, CPLX, XR>(nv, A, grid, block, lds, st);
    if (acc64) return launch_nv<W, KIND, float, double, CPLX, XR>(nv, A, grid, block, lds, st);
    return launch_nv<W, KIND, float, float, CPLX, XR>(nv, A, grid, block, lds, st);
}

// One state width (a translation unit each for the sublattice kernels).
template <class W, int KIND, int XR = 0>
int launch_width(bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A, unsigned grid,
                 unsigned block, size_t lds, hipStream_t st) {
    if constexpr (KIND == K_U1) {
        if (cplx) {
            set_error("complex kernel requested for a U(1) block");
            return XDG_EINVAL;
        }
        return launch_prec<W, KIND, false, XR>(single, acc64, nv, A, grid, block, lds, st);
    } else {
        return cplx ? launch_prec<W, KIND, true, XR>(single, acc64, nv, A, grid, block, lds, st)
                    : launch_prec<W, KIND, false, XR>(single, acc64, nv, A, grid, block, lds, st);
    }
}

template <int KIND, int XR = 0>
int launch_kind_impl(bool wide, bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A,
                     unsigned grid, unsigned block, size_t lds, hipStream_t st) {
    return wide ? launch_width<uint64_t, KIND, XR>(single, acc64, cplx, nv, A, grid, block, lds, st)
                : launch_width<uint32_t, KIND, XR>(single, acc64, cplx, nv, A, grid, block, lds, st);
}

int launch_sub_wide(bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A, unsigned grid,
                    unsigned block, size_t lds, hipStream_t st);
int launch_sub_xr_wide(bool single, bool acc64, bool cplx, int nv, const ApplyArgs &A,
                       unsigned grid, unsigned block, size_t lds, hipStream_t st);

template <int KIND>
int launch_count_impl(bool wide, const ApplyArgs &A, unsigned grid, unsigned block, size_t lds,
                      hipStream_t st) {
    void (*f)(ApplyArgs) = wide ? k_count<uint64_t, KIND, true> : k_count<uint32_t, KIND, true>;
    if constexpr (KIND == K_SUB)
        if (!A.stage_sub)
            f = wide ? k_count<uint64_t, KIND, false> : k_count<uint32_t, KIND, false>;
    if (lds > 65536)
        XDG_TRY_HIP(hipFuncSetAttribute((const void *)f,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(f, dim3(grid), dim3(block), lds, st, A);
    XDG_TRY_HIP(hipGetLastError());
    return XDG_OK;
}

}  // namespace xdg
