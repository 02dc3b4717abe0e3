// Sector basis on the GPU (Spinhalf(N, nup[, irrep]), Sec. 3.1 and 3.11):
// ascending enumeration of popcount-n_up states in independent chunks
// (colex unranking + next-same-popcount), representative and compatibility
// test per candidate, count -> scan -> ordered fill; then the device index
// (Lin tables for the U(1) block, Sec. 5.2; a line-bucketed hash for
// representatives).  Also the counter-based random state generator.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "device_common.hpp"

namespace xdg {

// ------------------------------------------------------------------ utils --
// Device memory held by the library's buffers, and the caller's limit on it
// (0 = none), see xdg_set_device_memory_limit.
static std::atomic<uint64_t> g_dev_bytes{0};
static std::atomic<uint64_t> g_dev_limit{0};

static thread_local uint64_t g_missing = 0;

uint64_t take_missing_memory() {
    const uint64_t n = g_missing;
    g_missing = 0;
    return n;
}

void set_device_memory_limit(uint64_t bytes) { g_dev_limit.store(bytes); }
uint64_t device_memory_in_use() { return g_dev_bytes.load(); }

void DevBuf::release() {
    if (p) {
        (void)hipFree(p);
        g_dev_bytes.fetch_sub(bytes);
    }
    p = nullptr;
    bytes = 0;
}

int DevBuf::alloc(size_t n) {
    release();
    if (n == 0) return XDG_OK;
    const uint64_t limit = g_dev_limit.load();
    const uint64_t held = g_dev_bytes.fetch_add(n) + n;
    if (limit && held > limit) {
        g_dev_bytes.fetch_sub(n);
        g_missing = held - limit;
        set_error("device memory limit: %zu more bytes would bring the library to %llu of %llu",
                  n, (unsigned long long)held, (unsigned long long)limit);
        return XDG_ENOMEM;
    }
    hipError_t e = hipMalloc(&p, n);
    if (e != hipSuccess) {
        g_dev_bytes.fetch_sub(n);
        p = nullptr;
        size_t room = 0, all = 0;
        if (e == hipErrorOutOfMemory && hipMemGetInfo(&room, &all) == hipSuccess)
            g_missing = n > room ? n - room : 1;
        (void)hipGetLastError();
        set_error("hipMalloc(%zu bytes) failed: %s", n, hipGetErrorString(e));
        return XDG_ENOMEM;
    }
    bytes = n;
    return XDG_OK;
}

int DevBuf::upload(const void *host, size_t n) {
    XDG_RETURN_IF(alloc(n));
    if (n) XDG_RETURN_IF(copy_h2d(p, host, n, nullptr));
    return XDG_OK;
}

// Host <-> device transfers go through a page-locked buffer owned by the
// library (per thread, grown on demand, chunks of at most 64 MiB) with an
// explicit wait after every chunk: no DMA ever targets pageable caller
// memory, and no transfer is still in flight when the call returns.
namespace {
// (kept until the process ends: freeing it from a thread-exit destructor
// could run after the HIP runtime has shut down)
struct PinnedStage {
    void *p = nullptr;
    size_t cap = 0;
    int reserve(size_t n) {
        if (n <= cap) return XDG_OK;
        if (p) (void)hipHostFree(p);
        p = nullptr;
        cap = 0;
        hipError_t e = hipHostMalloc(&p, n, hipHostMallocPortable | hipHostMallocMapped);
        if (e != hipSuccess) {
            p = nullptr;
            (void)hipGetLastError();
            set_error("hipHostMalloc(%zu bytes) failed: %s", n, hipGetErrorString(e));
            return XDG_ENOMEM;
        }
        cap = n;
        return XDG_OK;
    }
};
thread_local PinnedStage g_stage, g_scalars;
constexpr size_t STAGE_CHUNK = (size_t)64 << 20;
}  // namespace

int copy_d2h(void *dst, const void *src, size_t n, hipStream_t st) {
    size_t done = 0;
    while (done < n) {
        const size_t len = std::min(STAGE_CHUNK, n - done);
        XDG_RETURN_IF(g_stage.reserve(len));
        XDG_TRY_HIP(hipMemcpyAsync(g_stage.p, static_cast<const char *>(src) + done, len,
                                   hipMemcpyDeviceToHost, st));
        XDG_TRY_HIP(hipStreamSynchronize(st));
        std::memcpy(static_cast<char *>(dst) + done, g_stage.p, len);
        done += len;
    }
    return XDG_OK;
}

int copy_h2d(void *dst, const void *src, size_t n, hipStream_t st) {
    size_t done = 0;
    while (done < n) {
        const size_t len = std::min(STAGE_CHUNK, n - done);
        XDG_RETURN_IF(g_stage.reserve(len));
        std::memcpy(g_stage.p, static_cast<const char *>(src) + done, len);
        XDG_TRY_HIP(hipMemcpyAsync(static_cast<char *>(dst) + done, g_stage.p, len,
                                   hipMemcpyHostToDevice, st));
        XDG_TRY_HIP(hipStreamSynchronize(st));
        done += len;
    }
    return XDG_OK;
}

int host_scalars(size_t n, double **out) {
    XDG_RETURN_IF(g_scalars.reserve(n * sizeof(double)));
    *out = static_cast<double *>(g_scalars.p);
    return XDG_OK;
}

int device_cu_count() {
    static int cached = 0;
    if (!cached) {
        int dev = 0, cu = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            cu > 0)
            cached = cu;
        else
            cached = 256;
    }
    return cached;
}

size_t lds_limit() {
    static size_t cached = 0;
    if (!cached) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
            v > 0)
            cached = (size_t)v;
        else
            cached = 65536;
    }
    return cached;
}

__host__ __device__ static inline size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// ------------------------------------------------------------ enumeration --
// Candidates: for every segment, prefix | low << shift over the integers
// `low` of `bits` bits and k set bits, ascending; ascending segments, so that
// candidate number r is ascending too.  What a representative must look like
// keeps the list short:
//   sublattice coding: its top block is the minimal top of its own content (26
//     of 512 contents on the 6x6 lattice): one segment per such content, the
//     sites below it free.  4.2e8 candidates instead of 9.1e9 there.
//   a full ring: the lowest site is up (else the state shifted down is
//     smaller) and the top one down, unless all sites agree: one segment of
//     N - 2 free sites, a quarter of the states.
//   otherwise: one segment, all states.
struct EnumSeg {
    uint64_t base;      // number of the segment's first candidate
    uint64_t prefix;
    uint64_t k;
};

template <class W>
struct EnumArgs {
    int N, n_sym;
    int bits, shift, n_seg;
    const EnumSeg *segs;       // [n_seg + 1], the last one's base is the total
    uint64_t total, n_chunks;
    uint32_t chunk_len;        // a multiple of 32 if larger
    const uint64_t *binom;     // [65][65]
    uint32_t *counts;          // [n_chunks] (count pass)
    uint32_t *keep;            // [ceil(chunk_len / 32)][n_chunks] kept candidates, or null
    const uint64_t *offsets;   // [n_chunks] (fill passes; NULL = the number itself)
    W *reps;
    uint16_t *stab;
    uint64_t dim;
    const double2 *chi;
    const AffineElem *aff;
    const uint64_t *bytetab;
    int n_bchunks;
    const uint16_t *mintop;
    const uint32_t *cand_off;
    const uint16_t *cand_list;
    const uint32_t *sp;
    const uint16_t *tperm;
    int n_s, m, pb, n_perm;
    uint32_t n_cand;
    int stage_sub;
    PackedSrc packed;          // K_PACKED
    int chi_one;               // every character is exactly 1
};

template <class W>
struct Candidates {
    const EnumArgs<W> &A;
    int seg;
    W low;
    uint64_t r, end;    // this candidate's number, and the segment's end
    __device__ __forceinline__ Candidates(const EnumArgs<W> &A_, uint64_t r0) : A(A_), r(r0) {
        int lo = 0, hi = A.n_seg - 1;   // last segment with base <= r0
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (A.segs[mid].base <= r0) lo = mid; else hi = mid - 1;
        }
        seg = lo;
        end = A.segs[seg + 1].base;
        low = unrank_colex<W>(r0 - A.segs[seg].base, A.bits, (int)A.segs[seg].k, A.binom);
    }
    __device__ __forceinline__ W state() const { return (W)A.segs[seg].prefix | (low << A.shift); }
    __device__ __forceinline__ void next() {
        if (++r < end) {
            low = next_same_popcount<W>(low);
        } else {
            ++seg;
            end = A.segs[seg + 1].base;
            low = (W(1) << A.segs[seg].k) - 1;   // every segment is shorter than W here
        }
    }
};

// 16 waves share the staged tables; lists too short to fill the chip that way
// take workgroups of one wave
constexpr int ENUM_BLOCK = 1024;

// Sublattice coding in the packed form (sub_rep_packed).  The test by early
// exits takes each lane through lists of its own, and the products' search
// forms the whole minimum (6x6 lattice, Gamma A1: count pass 11.0 and 8.8 ms,
// 2.9 ms with this; k_stab 0.43 -> 0.16 ms).
constexpr int K_PACKED = 5;

// Representative test of the enumeration with the tables in LDS.
template <class W, int KIND>
struct RepTest {
    const EnumArgs<W> &A;
    const double2 *chi;
    const AffineElem *aff;
    SubCtx C;
    PackedCtx P;
    __device__ __forceinline__ RepTest(const EnumArgs<W> &A_, unsigned char *smem) : A(A_) {
        if constexpr (KIND == K_PACKED) {
            size_t at = packed_entry_bytes(A.n_sym);
            P = stage_packed(A.packed, smem, at);
            __syncthreads();
            return;
        }
        C = SubCtx{A.mintop, A.cand_off, A.cand_list, A.sp, A.tperm, A.n_s, A.m, A.pb};
        double2 *lchi = reinterpret_cast<double2 *>(smem);
        size_t off = align16(sizeof(double2) * A.n_sym);
        for (int g = threadIdx.x; g < A.n_sym; g += blockDim.x) lchi[g] = A.chi[g];
        chi = lchi;
        aff = A.aff;
        if constexpr (KIND == K_AFF) {
            AffineElem *laff = reinterpret_cast<AffineElem *>(smem + off);
            for (int g = threadIdx.x; g < A.n_sym; g += blockDim.x) laff[g] = A.aff[g];
            aff = laff;
        }
        if constexpr (KIND == K_SUB) {
            if (A.stage_sub) {
                auto copy = [&](auto *src, uint32_t n) {
                    using E = std::remove_const_t<std::remove_pointer_t<decltype(src)>>;
                    auto *dst = reinterpret_cast<E *>(smem + off);
                    off = align16(off + sizeof(*src) * (size_t)n);
                    for (uint32_t e = threadIdx.x; e < n; e += blockDim.x) dst[e] = src[e];
                    return dst;
                };
                const uint32_t NV = (uint32_t)A.n_s << A.m;
                C.mintop = copy(A.mintop, NV);
                C.cand_off = copy(A.cand_off, NV + 1);
                C.cand_list = copy(A.cand_list, A.n_cand);
                C.sp = copy(A.sp, (uint32_t)A.n_sym * A.n_s);
                C.tperm = copy(A.tperm, (uint32_t)A.n_perm * 2u << A.pb);
            }
        }
        __syncthreads();
    }
    // s is the representative of an orbit that carries a symmetric state (the
    // stabiliser sum of chi is nonzero); st = |Stab(s)|
    __device__ __forceinline__ bool operator()(W s, int &st) const {
        if constexpr (KIND == K_PACKED) {
            const int B = 3 * A.m;
            int n = 0;
            double cr = 0.0, ci = 0.0;
            auto same = [&](uint32_t g) {
                ++n;
                const double2 c = A.chi_one ? make_double2(1.0, 0.0) : A.chi[g];
                cr += c.x;
                ci += c.y;
            };
            const bool rep = sub_rep_packed(P, sub_key<W>(s, A.m, A.pb), (uint32_t)(s >> B),
                                            (uint32_t)(s & ((W(1) << B) - 1)), same) &&
                             cr * cr + ci * ci > 0.25;
            st = n;
            return rep;
        }
        double cr = 0.0, ci = 0.0;
        bool rep = false;
        if constexpr (KIND == K_AFF)
            rep = aff_is_rep<W>(aff, A.n_sym, A.N, s, chi, st, cr, ci);
        else if constexpr (KIND == K_SUB)
            rep = sub_is_rep<W>(C, s, chi, st, cr, ci);
        else if constexpr (KIND == K_TAB)
            rep = tab_is_rep<W>(A.bytetab, A.n_bchunks, A.n_sym, s, chi, st, cr, ci);
        return rep && (cr * cr + ci * ci > 0.25);
    }
};

// A lane per chunk of candidates: how many are kept and, with A.keep, which
// (FILL = false); the kept ones at their place, tested again (FILL = true,
// byte tables, whose bits would take more memory than the index).
template <class W, int KIND, bool FILL>
__global__ __launch_bounds__(ENUM_BLOCK) void k_enum(EnumArgs<W> A) {
    extern __shared__ __align__(16) unsigned char smem[];
    const RepTest<W, KIND> test(A, smem);
    const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= A.n_chunks) return;
    const uint64_t r0 = c * A.chunk_len;
    const uint64_t r1 = r0 + A.chunk_len < A.total ? r0 + A.chunk_len : A.total;
    Candidates<W> cand(A, r0);
    uint64_t pos = FILL ? A.offsets[c] : 0;
    uint32_t cnt = 0, bits = 0;
    for (uint64_t r = r0; r < r1; ++r) {
        const W s = cand.state();
        int st;
        if (test(s, st)) {
            if constexpr (FILL) {
                A.reps[pos] = s;
                A.stab[pos] = (uint16_t)st;
                ++pos;
            }
            ++cnt;
            bits |= 1u << (uint32_t)((r - r0) & 31);
        }
        if (!FILL && A.keep && (((r - r0) & 31) == 31 || r + 1 == r1)) {
            A.keep[((r - r0) >> 5) * A.n_chunks + c] = bits;
            bits = 0;
        }
        if (r + 1 < r1) cand.next();
    }
    if constexpr (!FILL) A.counts[c] = cnt;
}

// The kept candidates at their place: all of them (U(1)) or those of A.keep.
template <class W>
__global__ __launch_bounds__(256) void k_enum_fill(EnumArgs<W> A) {
    const uint64_t c = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= A.n_chunks) return;
    const uint64_t r0 = c * A.chunk_len;
    const uint64_t r1 = r0 + A.chunk_len < A.total ? r0 + A.chunk_len : A.total;
    Candidates<W> cand(A, r0);
    uint64_t pos = A.offsets ? A.offsets[c] : r0;
    for (uint64_t b0 = r0; b0 < r1; b0 += 32) {
        const uint64_t b1 = b0 + 32 < r1 ? b0 + 32 : r1;
        const uint32_t bits = A.keep ? A.keep[((b0 - r0) >> 5) * A.n_chunks + c] : ~0u;
        for (uint64_t r = b0; r < b1; ++r) {
            if ((bits >> (uint32_t)(r - b0)) & 1u) A.reps[pos++] = cand.state();
            if (r + 1 < r1) cand.next();
        }
    }
}

// |Stab| of every basis state (all lanes busy, unlike in the count pass,
// where one candidate in 13 is kept on the 6x6 lattice)
template <class W, int KIND>
__global__ __launch_bounds__(ENUM_BLOCK) void k_stab(EnumArgs<W> A) {
    extern __shared__ __align__(16) unsigned char smem[];
    const RepTest<W, KIND> test(A, smem);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < A.dim; i += stride) {
        int st;
        (void)test(A.reps[i], st);
        A.stab[i] = (uint16_t)st;
    }
}

// ------------------------------------------------------------------- scan --
// Exclusive scan of u32 counts into u64 offsets, three passes with
// 1024-element tiles; fixed order, no atomics.
__device__ uint64_t block_exclusive_scan(uint64_t v, uint64_t *sh, uint64_t *total) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int d = 1; d < (int)blockDim.x; d <<= 1) {
        uint64_t add = t >= d ? sh[t - d] : 0;
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    const uint64_t incl = sh[t];
    if (total) *total = sh[blockDim.x - 1];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(1024) void k_scan_tiles(const uint32_t *counts, uint64_t n,
                                                     uint64_t *tile_sums) {
    __shared__ uint64_t sh[1024];
    const uint64_t i = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
    uint64_t v = i < n ? counts[i] : 0;
    uint64_t tot;
    block_exclusive_scan(v, sh, &tot);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_sums(uint64_t *tile_sums, uint64_t n_tiles,
                                                    uint64_t *grand_total) {
    __shared__ uint64_t sh[1024];
    const uint64_t per = (n_tiles + 1023) / 1024;
    const uint64_t b0 = threadIdx.x * per;
    uint64_t local = 0;
    for (uint64_t b = b0; b < b0 + per && b < n_tiles; ++b) local += tile_sums[b];
    uint64_t tot;
    uint64_t base = block_exclusive_scan(local, sh, &tot);
    for (uint64_t b = b0; b < b0 + per && b < n_tiles; ++b) {
        uint64_t v = tile_sums[b];
        tile_sums[b] = base;
        base += v;
    }
    if (threadIdx.x == 0) *grand_total = tot;
}

__global__ __launch_bounds__(1024) void k_scan_apply(const uint32_t *counts, uint64_t n,
                                                     const uint64_t *tile_base, uint64_t *offsets) {
    __shared__ uint64_t sh[1024];
    const uint64_t i = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
    uint64_t v = i < n ? counts[i] : 0;
    uint64_t ex = block_exclusive_scan(v, sh, nullptr);
    if (i < n) offsets[i] = ex + tile_base[blockIdx.x];
}

// ------------------------------------------------------------------- hash --
template <class W>
__global__ __launch_bounds__(256) void k_hash_insert(const W *reps, uint64_t dim, void *table,
                                                     uint64_t n_lines, W empty) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= dim) return;
    const W key = reps[i];
    uint64_t line = hash_line<W>(key, n_lines);
    for (;;) {
        if constexpr (sizeof(W) == 4) {
            Line32 *L = reinterpret_cast<Line32 *>(table) + line;
            for (int s = 0; s < 8; ++s) {
                uint32_t old = atomicCAS(&L->k[s], (uint32_t)empty, (uint32_t)key);
                if (old == (uint32_t)empty) {
                    L->v[s] = (uint32_t)i;
                    return;
                }
            }
        } else {
            Line64 *L = reinterpret_cast<Line64 *>(table) + line;
            for (int s = 0; s < 5; ++s) {
                unsigned long long old =
                    atomicCAS(reinterpret_cast<unsigned long long *>(&L->k[s]),
                              (unsigned long long)empty, (unsigned long long)key);
                if (old == (unsigned long long)empty) {
                    L->v[s] = (uint32_t)i;
                    return;
                }
            }
        }
        line = line + 1 == n_lines ? 0 : line + 1;
    }
}

// ------------------------------------------------------------------- rank --
// Sets the bit of every basis state; the first state of each word (the reps
// are ascending and the colex rank preserves their order) writes its index
// as the word's count.
template <class W>
__global__ __launch_bounds__(256) void k_rank_build(const W *reps, uint64_t dim, const void *T,
                                                    RankLayout L, uint2 *words) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= dim) return;
    const uint64_t r = colex_rank<W>(T, L, reps[i]);
    const uint64_t w = r >> 5;
    atomicOr(&words[w].y, 1u << (uint32_t)(r & 31));
    if (i == 0 || (colex_rank<W>(T, L, reps[i - 1]) >> 5) != w) words[w].x = (uint32_t)i;
}

// index of arbitrary states (-1 when absent)
struct RankArgs {
    const uint2 *words;
    uint64_t n_words;   // 0: no rank index
    const void *tab;
    RankLayout L;
};

template <class W>
__global__ __launch_bounds__(256) void k_lookup(const uint64_t *states, int64_t n, int64_t *out,
                                                int N, int n_up, int u1, const uint32_t *lin,
                                                int nlo, const void *table, uint64_t n_lines,
                                                W empty, RankArgs R) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t s = states[i];
    int64_t r = -1;
    const bool in_range = N == 64 || (s >> N) == 0;
    if (in_range && __popcll(s) == n_up) {
        if (u1) {
            const uint64_t lo = s & ((1ull << nlo) - 1), hi = s >> nlo;
            r = (int64_t)lin[(1ull << nlo) + hi] + (int64_t)lin[lo];
        } else if (R.n_words) {
            r = rank_find(R.words, R.n_words, colex_rank<W>(R.tab, R.L, (W)s));
        } else if (n_lines) {
            r = hash_find<W>(table, n_lines, empty, (W)s);
        }
    }
    out[i] = r;
}

// ----------------------------------------------------------------- random --
__device__ __forceinline__ uint64_t splitmix_out(uint64_t seed, uint64_t n) {
    uint64_t z = seed + n * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ double u53(uint64_t z) {
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

template <class T>
__global__ __launch_bounds__(256) void k_random(uint64_t n, uint64_t seed, int kind, T *out) {
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
         q += (uint64_t)gridDim.x * blockDim.x) {
        const double u1 = u53(splitmix_out(seed, 2 * q + 1));
        double v;
        if (kind == 0) {
            v = 2.0 * u1 - 1.0;
        } else {
            const double u2 = u53(splitmix_out(seed, 2 * q + 2));
            v = sqrt(-2.0 * log1p(-u1)) * cos(2.0 * M_PI * u2);
        }
        out[q] = (T)v;
    }
}

int random_fill(int64_t n_scalars, uint64_t seed, int kind, bool single, void *out,
                hipStream_t st) {
    if (n_scalars <= 0) return XDG_OK;
    const int block = 256;
    const uint64_t want = ((uint64_t)n_scalars + block - 1) / block;
    const int grid = (int)std::min<uint64_t>(want, (uint64_t)device_cu_count() * 16);
    if (single)
        hipLaunchKernelGGL(k_random<float>, dim3(grid), dim3(block), 0, st, (uint64_t)n_scalars,
                           seed, kind, (float *)out);
    else
        hipLaunchKernelGGL(k_random<double>, dim3(grid), dim3(block), 0, st,
                           (uint64_t)n_scalars, seed, kind, (double *)out);
    XDG_TRY_HIP(hipGetLastError());
    return XDG_OK;
}

// ------------------------------------------------------------- host side --
namespace {

// The candidate segments of a block (see EnumSeg), the last one's end included.
void enum_segments(const xdg_basis_s *b, std::vector<EnumSeg> *segs, int *bits, int *shift) {
    const int N = b->n_sites, n = b->n_up;
    *bits = N;
    *shift = 0;
    uint64_t acc = 0;
    auto add = [&](uint64_t prefix, int k) {
        segs->push_back({acc, prefix, (uint64_t)k});
        acc += binomial(*bits, k);
    };
    const SublatticeTables &S = b->plan.sub;
    if (b->plan.kind == K_SUB && S.n_s >= 2) {
        *bits = (S.n_s - 1) * S.m;
        for (uint32_t c = 0; c < 1u << S.m; ++c) {
            const int k = n - __builtin_popcount(c);
            if (k < 0 || k > *bits || S.mintop[((size_t)(S.n_s - 1) << S.m) + c] != c) continue;
            add((uint64_t)c << *bits, k);
        }
    } else if (b->plan.kind == K_AFF && b->plan.ring && N >= 3 && n > 0 && n < N) {
        *bits = N - 2;
        *shift = 1;
        add(1, n - 1);
    } else {
        add(0, n);
    }
    segs->push_back({acc, 0, 0});
}

template <class W>
int enumerate(xdg_basis_s *b, const std::vector<uint64_t> &binom) {
    const int kind = b->plan.kind;
    EnumArgs<W> A{};
    std::vector<EnumSeg> segs;
    enum_segments(b, &segs, &A.bits, &A.shift);
    const uint64_t total = segs.back().base;
    if (total == 0) {
        b->dim = 0;
        return XDG_OK;
    }
    DevBuf consts;
    DevView segs_v, binom_v;
    UploadArena ar;
    ar.add(segs_v, segs.data(), segs.size() * sizeof(EnumSeg));
    ar.add(binom_v, binom.data(), binom.size() * 8);
    XDG_RETURN_IF(ar.commit(consts));
    A.segs = segs_v.as<EnumSeg>();
    A.n_seg = (int)segs.size() - 1;
    A.N = b->n_sites;
    A.n_sym = b->n_sym;
    A.total = total;
    A.binom = binom_v.as<uint64_t>();
    A.chi = b->chi_d.as<double2>();
    A.aff = b->t_aff.as<AffineElem>();
    A.bytetab = b->t_bytes.as<uint64_t>();
    A.n_bchunks = b->plan.bytes.n_chunks;
    A.mintop = b->t_mintop.as<uint16_t>();
    A.cand_off = b->t_candoff.as<uint32_t>();
    A.cand_list = b->t_candlist.as<uint16_t>();
    A.sp = b->t_pid.as<uint32_t>();
    A.tperm = b->t_tperm.as<uint16_t>();
    A.n_s = b->plan.sub.n_s;
    A.m = b->plan.sub.m;
    A.pb = b->plan.sub.pb;
    A.n_perm = b->plan.sub.n_perm;
    A.n_cand = (uint32_t)b->plan.sub.cand_list.size();

    // a lane per chunk: enough lanes for the chip twice over, chunks long
    // enough to pay for their first state
    const uint64_t lanes_target = (uint64_t)device_cu_count() * 4096;
    uint64_t cl = std::max<uint64_t>(4, std::min<uint64_t>(4096, total / lanes_target));
    // without a group nothing is tested and the stores are the work: lanes next
    // to each other fill the same lines (ring N = 28, 40 M states: 260, 202,
    // 320 and 525 us with 4, 8, 16 and 152 states a lane)
    if (kind == K_U1) cl = 8;
    else if (cl > 32) cl = cl / 32 * 32;
    A.chunk_len = (uint32_t)cl;
    A.n_chunks = (total + cl - 1) / cl;

    size_t lds = 0;
    if (kind != K_U1) {
        lds = align16(sizeof(double2) * b->n_sym);
        if (kind == K_AFF) lds += align16(sizeof(AffineElem) * b->n_sym);
        if (kind == K_SUB) {
            const size_t NV = (size_t)A.n_s << A.m;
            const size_t GS = (size_t)A.n_sym * A.n_s;
            size_t need = align16(2 * NV) + align16(4 * (NV + 1)) + align16(2 * (size_t)A.n_cand) +
                          align16(4 * GS) +
                          align16(2 * ((size_t)A.n_perm * 2 << A.pb));
            if (lds + need <= lds_limit()) {
                A.stage_sub = 1;
                lds += need;
            }
        }
    }
    A.chi_one = b->chi_trivial;
    bool packed = kind == K_SUB && b->plan.sub.packed();
    if (packed) {
        const SublatticeTables &S = b->plan.sub;
        A.packed = PackedSrc{b->t_pktab.as<uint32_t>(), b->t_pkcand.as<uint16_t>(), A.sp, A.tperm,
                             (uint32_t)S.pk_cand.size(), S.pk_nb, b->n_sym, A.n_perm, A.m, A.pb};
        const size_t need = packed_entry_bytes(b->n_sym) +
                            packed_table_bytes(A.packed.n_cand, A.n_perm, A.m, A.pb);
        packed = need <= lds_limit();
        if (packed) lds = need;
    }
    auto blocks_of = [](uint64_t lanes, int block) { return (lanes + block - 1) / block; };
    if (blocks_of(A.n_chunks, 256) > 0x7fffffffull) {
        set_error("enumeration grid too large");
        return XDG_EINVAL;
    }
    const int block =
        A.n_chunks >= (uint64_t)device_cu_count() * ENUM_BLOCK ? ENUM_BLOCK : 64;
    const unsigned grid = (unsigned)blocks_of(A.n_chunks, block);
    const unsigned fill_grid = (unsigned)blocks_of(A.n_chunks, 256);
    void (*kcount)(EnumArgs<W>) = nullptr, (*kfill)(EnumArgs<W>) = nullptr,
        (*kstab)(EnumArgs<W>) = nullptr;
    if (kind == K_AFF) {
        kcount = k_enum<W, K_AFF, false>;
        kstab = k_stab<W, K_AFF>;
    } else if (packed) {
        kcount = k_enum<W, K_PACKED, false>;
        kstab = k_stab<W, K_PACKED>;
    } else if (kind == K_SUB) {
        kcount = k_enum<W, K_SUB, false>;
        kstab = k_stab<W, K_SUB>;
    } else if (kind == K_TAB) {
        kcount = k_enum<W, K_TAB, false>;
        kfill = k_enum<W, K_TAB, true>;
    }
    for (auto f : {kcount, kfill, kstab})
        if (f && lds > 65536)
            XDG_TRY_HIP(hipFuncSetAttribute((const void *)f,
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));

    DevBuf temp;
    uint64_t dim;
    if (kind == K_U1) {
        dim = total;
    } else {
        // one allocation: total, tile sums, offsets, counts, kept bits
        const uint64_t n_tiles = (A.n_chunks + 1023) / 1024;
        const uint64_t keep_words = kind == K_TAB ? 0 : (cl + 31) / 32 * A.n_chunks;
        XDG_RETURN_IF(temp.alloc(8 * (1 + n_tiles + A.n_chunks) + 4 * (A.n_chunks + keep_words)));
        uint64_t *tot = temp.as<uint64_t>(), *tiles = tot + 1, *offsets = tiles + n_tiles;
        A.counts = reinterpret_cast<uint32_t *>(offsets + A.n_chunks);
        A.keep = keep_words ? A.counts + A.n_chunks : nullptr;
        hipLaunchKernelGGL(kcount, dim3(grid), dim3(block), lds, 0, A);
        XDG_TRY_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)n_tiles), dim3(1024), 0, 0,
                           A.counts, A.n_chunks, tiles);
        hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, 0, tiles, n_tiles, tot);
        hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)n_tiles), dim3(1024), 0, 0,
                           A.counts, A.n_chunks, tiles, offsets);
        XDG_TRY_HIP(hipGetLastError());
        XDG_RETURN_IF(copy_d2h(&dim, tot, sizeof dim, nullptr));
        A.offsets = offsets;
    }
    if (dim >= 0xFFFFFFFFull) {
        set_error("block dimension %llu needs 64-bit indices (limit 2^32 - 1)",
                  (unsigned long long)dim);
        return XDG_EINVAL;
    }
    b->dim = (int64_t)dim;
    if (dim == 0) return XDG_OK;
    XDG_RETURN_IF(b->reps.alloc(sizeof(W) * dim));
    if (kind != K_U1) XDG_RETURN_IF(b->stab.alloc(sizeof(uint16_t) * dim));
    A.reps = b->reps.as<W>();
    A.stab = b->stab.as<uint16_t>();
    A.dim = dim;
    if (kfill) {
        hipLaunchKernelGGL(kfill, dim3(grid), dim3(block), lds, 0, A);
    } else {
        hipLaunchKernelGGL(k_enum_fill<W>, dim3(fill_grid), dim3(256), 0, 0, A);
        XDG_TRY_HIP(hipGetLastError());
        if (kstab) {
            const unsigned g = (unsigned)std::min<uint64_t>(blocks_of(dim, block),
                                                            (uint64_t)device_cu_count() * 2);
            hipLaunchKernelGGL(kstab, dim3(g), dim3(block), lds, 0, A);
        }
    }
    XDG_TRY_HIP(hipGetLastError());
    XDG_TRY_HIP(hipDeviceSynchronize());
    return XDG_OK;
}

template <class W>
int build_hash(xdg_basis_s *b) {
    const uint64_t dim = (uint64_t)b->dim;
    const int slots = sizeof(W) == 4 ? 8 : 5;
    const double load = 0.5;   // mean occupied slots per slot
    uint64_t n_lines = (uint64_t)std::ceil((double)dim / (slots * load));
    n_lines = std::max<uint64_t>(n_lines, 1);
    if (n_lines >= (1ull << 32)) {
        set_error("hash index too large");
        return XDG_EINVAL;
    }
    XDG_RETURN_IF(b->hash.alloc(64 * n_lines));
    const W empty = b->n_up == b->n_sites ? W(0) : ~W(0);
    XDG_TRY_HIP(hipMemset(b->hash.p, empty ? 0xFF : 0x00, 64 * n_lines));
    b->hidx.n_lines = n_lines;
    b->hidx.slots = slots;
    const int block = 256;
    hipLaunchKernelGGL(k_hash_insert<W>, dim3((unsigned)((dim + block - 1) / block)), dim3(block),
                       0, 0, b->reps.as<W>(), dim, b->hash.p, n_lines, empty);
    XDG_TRY_HIP(hipGetLastError());
    XDG_TRY_HIP(hipDeviceSynchronize());
    return XDG_OK;
}

// Chunk tables of the colex rank (the layout read by colex_rank): the entry
// of chunk k, below set bits under it, chunk bits v is the sum over the set
// bits of v, the i-th (from the bottom) at site p = k cb + q, of
// C(p, below + i); sites beyond N contribute nothing.  Rows only for below
// in [rank_lo, rank_hi] of each chunk.  32-bit states: four chunks of 8
// sites, u32 entries.  Wider states: the widest chunk (fewest reads) whose
// table stays within 32 KiB (the apply kernels stage it in LDS), with u32
// entries saturating at 2^32 - 1 when max_rank, the largest rank the block
// must resolve, leaves room below that, u64 entries otherwise.
RankLayout rank_layout(int N, int n_up, bool wide, uint64_t max_rank) {
    RankLayout L{};
    auto rows_of = [&](int cb, int nc) {
        int rows = 0;
        for (int k = 0; k < nc; ++k) rows += rank_hi(n_up, cb, k) - rank_lo(N, n_up, cb, k) + 1;
        return rows;
    };
    if (!wide) {
        L.cb = RANK_CB32;
        L.nc = RANK_NC32;
        L.e32 = 1;
    } else {
        L.e32 = max_rank < 0xFFFFFFFFull - 64 ? 1 : 0;
        const size_t esz = L.e32 ? 4 : 8;
        for (L.cb = 8; L.cb > 4; --L.cb) {
            L.nc = (N + L.cb - 1) / L.cb;
            if (((size_t)rows_of(L.cb, L.nc) << L.cb) * esz <= 32768) break;
        }
        L.nc = (N + L.cb - 1) / L.cb;
    }
    int row = 0;
    for (int k = 0; k < L.nc; ++k) {
        const int lo = rank_lo(N, n_up, L.cb, k);
        L.rbase[k] = row - lo;
        row += rank_hi(n_up, L.cb, k) - lo + 1;
    }
    L.rows = row;
    return L;
}

template <class E>
void rank_tables(int N, int n_up, const RankLayout &L, std::vector<E> &T) {
    const int cb = L.cb;
    T.assign((size_t)L.rows << cb, 0);
    for (int k = 0; k < L.nc; ++k) {
        const int lo = rank_lo(N, n_up, cb, k), hi = rank_hi(n_up, cb, k);
        for (int below = lo; below <= hi; ++below) {
            const size_t row = (size_t)(L.rbase[k] + below);
            for (uint32_t v = 0; v < (1u << cb); ++v) {
                uint64_t r = 0;
                int c = below;
                for (int q = 0; q < cb; ++q) {
                    if (!((v >> q) & 1)) continue;
                    ++c;
                    const int p = k * cb + q;
                    if (p < N) r += binomial(p, c);
                }
                if (sizeof(E) == 4 && r > 0xFFFFFFFFull) r = 0xFFFFFFFFull;
                T[(row << cb) | v] = (E)r;
            }
        }
    }
}

uint64_t colex_rank_host(uint64_t s) {
    uint64_t r = 0;
    int c = 0;
    for (int p = 0; p < 64; ++p)
        if ((s >> p) & 1) r += binomial(p, ++c);
    return r;
}

// The rows of the chunk tables (layout L) for the chunks below B, in 4-byte
// entries: shares of sites below 32 are exact; larger ones (read only for
// bits above B, which the rank clears) saturate.
template <class E>
int xr_lower_rows(const RankLayout &L, const E *T, int B, int n_up, std::vector<uint32_t> &out) {
    const int nlc = (B + L.cb - 1) / L.cb;
    const int rows = L.rbase[nlc - 1] + rank_hi(n_up, L.cb, nlc - 1) + 1;
    out.resize((size_t)rows << L.cb);
    for (size_t e = 0; e < out.size(); ++e)
        out[e] = T[e] > (E)0xFFFFFFFFu ? 0xFFFFFFFFu : (uint32_t)T[e];
    return rows;
}

// First rank of every top block for rank-addressed vectors (top_rank): the
// blocks that are the minimal top of their own content, ascending, each
// followed by the colex ranks of the states of the remaining popcount on the
// B sites below it.  Not set up when the blocks do not tile the sites or B
// exceeds 31.  T: the block's chunk tables (u32 or u64 entries, layout L);
// first, last: its smallest and largest basis states.
template <class W>
int build_xr(xdg_basis_s *b, const void *T, const RankLayout &L, W first, W last) {
    const SublatticeTables &S = b->plan.sub;
    const int n_s = S.n_s, m = S.m, B = (n_s - 1) * m;
    if (n_s < 2 || n_s * m != b->n_sites || B < 1 || B > 31 || m > 16) return XDG_OK;
    const uint32_t V = 1u << m;
    std::vector<uint64_t> top(V, ~0ull);
    uint64_t acc = 0;
    for (uint32_t c = 0; c < V; ++c) {
        if (S.mintop[(size_t)(n_s - 1) * V + c] != c) continue;
        const int k = b->n_up - __builtin_popcount(c);
        if (k < 0 || k > B) continue;
        top[c] = acc;
        acc += binomial(B, k);
    }
    if (S.packed()) {   // the slots of block_slot
        if (acc >= 1ull << 40) return XDG_OK;
        std::vector<uint32_t> ent(V), off((size_t)(m + 1) * (m + 1) * (m + 1), 0);
        std::vector<uint32_t> seen(m + 1, 0);
        for (uint32_t v = 0; v < V; ++v) {
            const int p = __builtin_popcount(v);
            ent[v] = slot_entry(seen[p]++, (uint32_t)binomial(m, p), p, m);
        }
        for (int pc = 0; pc <= m; ++pc) {
            uint64_t o = 0;
            for (int p2 = 0; p2 <= m; ++p2)
                for (int p1 = 0; p1 <= m; ++p1) {
                    const int p0 = b->n_up - pc - p2 - p1;
                    if (p0 < 0 || p0 > m) continue;
                    off[((size_t)pc * (m + 1) + p2) * (m + 1) + p1] = (uint32_t)o;
                    o += binomial(m, p2) * binomial(m, p1) * binomial(m, p0);
                }
        }
        std::vector<uint2> tops(V);
        for (uint32_t c = 0; c < V; ++c) {
            const uint64_t t = top[c] == ~0ull ? 0 : top[c];
            const uint32_t row = 4u * (uint32_t)(__builtin_popcount(c) * (m + 1) * (m + 1));
            tops[c] = make_uint2((uint32_t)t, (uint32_t)(t >> 32) << 24 | row);
        }
        auto in = [&](W s) {
            const uint32_t c = (uint32_t)((uint64_t)s >> B);
            return top[c] != ~0ull && block_slot(ent.data(), off.data(), tops.data(), m, c,
                                                 (uint32_t)s & ((1u << B) - 1u)) < acc;
        };
        if (!in(first) || !in(last)) {
            set_error("internal: a representative lies outside the slot space");
            return XDG_EINVAL;
        }
        UploadArena ar;
        ar.add(b->xb_ent, ent.data(), 4 * ent.size());
        ar.add(b->xb_off, off.data(), 4 * off.size());
        ar.add(b->xb_top, tops.data(), 8 * tops.size());
        XDG_RETURN_IF(ar.commit(b->xb_buf));
        b->xr_slots = acc;
        b->xr_bits = B;
        return XDG_OK;
    }
    std::vector<uint32_t> low;
    const int rows = L.e32 ? xr_lower_rows(L, static_cast<const uint32_t *>(T), B, b->n_up, low)
                           : xr_lower_rows(L, static_cast<const uint64_t *>(T), B, b->n_up, low);
    const uint64_t r0 = top_rank<W>(low.data(), L, B, top.data(), first);
    const uint64_t r1 = top_rank<W>(low.data(), L, B, top.data(), last);
    if (r0 == ~0ull || r1 == ~0ull || r0 > r1 || r1 >= acc) {
        set_error("internal: a representative lies outside the top-block rank space");
        return XDG_EINVAL;
    }
    XDG_RETURN_IF(b->xr_top.upload(top.data(), sizeof(uint64_t) * V));
    if (acc < 0xFFFFFFFFull) {   // 4-byte first ranks for the kernels' LDS
        std::vector<uint32_t> t32(V);
        for (uint32_t c = 0; c < V; ++c) t32[c] = top[c] == ~0ull ? 0xFFFFFFFFu : (uint32_t)top[c];
        XDG_RETURN_IF(b->xr_top32.upload(t32.data(), sizeof(uint32_t) * V));
    }
    XDG_RETURN_IF(b->xr_rtab.upload(low.data(), sizeof(uint32_t) * low.size()));
    b->xr_rows = rows;
    b->xr_slots = r1 + 1;
    b->xr_bits = B;
    return XDG_OK;
}

// Rank index when it fits (see XDG_INDEX_RANK); returns XDG_OK with
// b->n_rwords = 0 when the hash index should be used instead.
template <class W>
int build_rank(xdg_basis_s *b) {
    const uint64_t dim = (uint64_t)b->dim;
    if (b->plan.flags & XDG_FLAG_HASH_INDEX) return XDG_OK;
    uint64_t last = 0;
    XDG_RETURN_IF(copy_d2h(&last, b->reps.as<W>() + (dim - 1), sizeof(W), nullptr));
    const uint64_t n_words = (colex_rank_host(last) >> 5) + 1;
    const int slots = sizeof(W) == 4 ? 8 : 5;
    const double hash_bytes = 64.0 * std::ceil((double)dim / (slots * 0.5));
    if ((double)n_words * 8.0 > 4.0 * hash_bytes + 64.0 * (1 << 20)) return XDG_OK;
    const RankLayout L = rank_layout(b->n_sites, b->n_up, sizeof(W) == 8, colex_rank_host(last));
    std::vector<uint32_t> T32;
    std::vector<uint64_t> T64;
    const void *T = nullptr;
    size_t tbytes = 0;
    if (L.e32) {
        rank_tables<uint32_t>(b->n_sites, b->n_up, L, T32);
        T = T32.data();
        tbytes = T32.size() * 4;
    } else {
        rank_tables<uint64_t>(b->n_sites, b->n_up, L, T64);
        T = T64.data();
        tbytes = T64.size() * 8;
    }
    // the table read of the device rank must give the plain colex rank
    if (colex_rank<W>(T, L, (W)last) != colex_rank_host(last)) {
        set_error("internal: colex chunk tables disagree with the colex rank");
        return XDG_EINVAL;
    }
    UploadArena ar;
    ar.add(b->rtab, T, tbytes);
    XDG_RETURN_IF(ar.commit(b->rank_buf));
    XDG_RETURN_IF(b->rwords.alloc(8 * n_words));
    XDG_TRY_HIP(hipMemset(b->rwords.p, 0, 8 * n_words));
    const int block = 256;
    hipLaunchKernelGGL(k_rank_build<W>, dim3((unsigned)((dim + block - 1) / block)), dim3(block), 0,
                       0, b->reps.as<W>(), dim, b->rtab.p, L, b->rwords.as<uint2>());
    XDG_TRY_HIP(hipGetLastError());
    XDG_TRY_HIP(hipDeviceSynchronize());
    b->n_rwords = n_words;
    b->rank = L;
    if (b->plan.kind == K_SUB) {
        W first = 0;
        XDG_RETURN_IF(copy_d2h(&first, b->reps.as<W>(), sizeof(W), nullptr));
        XDG_RETURN_IF(build_xr<W>(b, T, L, first, (W)last));
    }
    return XDG_OK;
}

int build_lin(xdg_basis_s *b) {
    // index(s) = L_hi[hi] + L_lo[lo]: L_lo = colex rank of lo among the
    // lo' with the same popcount, L_hi[hi] = number of basis states whose
    // high part is smaller than hi (Lin's two-table scheme, Sec. 5.2).
    const int N = b->n_sites, n = b->n_up;
    const int nlo = N / 2, nhi = N - nlo;
    std::vector<uint32_t> t((size_t)1 << nlo | 0, 0);
    t.assign(((size_t)1 << nlo) + ((size_t)1 << nhi), 0);
    for (uint64_t lo = 0; lo < (1ull << nlo); ++lo) {
        uint64_t r = 0;
        int k = 0;
        for (int p = 0; p < nlo; ++p)
            if ((lo >> p) & 1) {
                r += binomial(p, k + 1);
                ++k;
            }
        t[lo] = (uint32_t)r;
    }
    uint64_t acc = 0;
    for (uint64_t hi = 0; hi < (1ull << nhi); ++hi) {
        t[((size_t)1 << nlo) + hi] = (uint32_t)acc;
        const int rest = n - __builtin_popcountll(hi);
        if (rest >= 0 && rest <= nlo) acc += binomial(nlo, rest);
    }
    b->lin_nlo = nlo;
    b->lin_nhi = nhi;
    // for the products: position changes of neighbouring sites' exchanges
    std::vector<uint32_t> adj((size_t)N * (n + 1));
    for (int i = 0; i < N; ++i)
        for (int k = 0; k <= n; ++k)
            adj[(size_t)i * (n + 1) + k] =
                (uint32_t)std::min<uint64_t>(binomial(i, k), 0xFFFFFFFFull);
    UploadArena ar;
    ar.add(b->lin, t.data(), t.size() * sizeof(uint32_t));
    ar.add(b->u1_adj, adj.data(), adj.size() * 4);
    return ar.commit(b->tables);
}

}  // namespace

int basis_build_device(xdg_basis_s *b) {
    std::vector<uint64_t> bt(65 * 65);
    for (int a = 0; a <= 64; ++a)
        for (int c = 0; c <= 64; ++c) bt[a * 65 + c] = binomial(a, c);
    UploadArena ar;
    const Plan &P = b->plan;
    if (b->n_sym) {
        ar.add(b->chi_d, b->chi.data(), b->chi.size() * sizeof(double));
        b->chi_trivial = true;
        for (int g = 0; g < b->n_sym; ++g)
            b->chi_trivial &= b->chi[2 * g] == 1.0 && b->chi[2 * g + 1] == 0.0;
        std::vector<float> cf(b->chi.begin(), b->chi.end());
        ar.add(b->chi_f, cf.data(), cf.size() * sizeof(float));
        std::vector<double> sq(2 * (b->n_sym + 1));
        std::vector<float> sqf(2 * (b->n_sym + 1));
        for (int c = 0; c <= b->n_sym; ++c) {
            sq[c] = c ? std::sqrt((double)c) : 0.0;
            sq[b->n_sym + 1 + c] = c ? 1.0 / std::sqrt((double)c) : 0.0;
            sqf[c] = (float)sq[c];
            sqf[b->n_sym + 1 + c] = (float)sq[b->n_sym + 1 + c];
        }
        ar.add(b->sqrt_d, sq.data(), sq.size() * sizeof(double));
        ar.add(b->sqrt_f, sqf.data(), sqf.size() * sizeof(float));
    }
    if (P.kind == K_AFF) {
        ar.add(b->t_aff, P.aff.data(), P.aff.size() * sizeof(AffineElem));
        if (P.ring)
            ar.add(b->t_ring, P.ring_gidx.data(), P.ring_gidx.size() * 2);
    }
    if (P.kind == K_SUB) {
        // device form, one word per (element, block): the offset of the block
        // permutation's tables in tperm, shifted left by 8, or'ed with the
        // first bit of the source block
        const uint64_t E = 1ull << P.sub.pb;
        std::vector<uint32_t> sp(P.sub.pid.size());
        for (size_t e = 0; e < sp.size(); ++e) {
            const uint64_t to = (uint64_t)P.sub.pid[e] * 2u * E;
            const uint32_t so = (uint32_t)(P.sub.src[e] * P.sub.m);
            if (to >= (1ull << 24) || so > 255u) {
                set_error("sublattice tables too large for their packed offsets");
                return XDG_EINVAL;
            }
            sp[e] = (uint32_t)(to << 8) | so;
        }
        ar.add(b->t_pid, sp.data(), sp.size() * 4);
        ar.add(b->t_tperm, P.sub.tperm.data(), P.sub.tperm.size() * 2);
        ar.add(b->t_mintop, P.sub.mintop.data(), P.sub.mintop.size() * 2);
        ar.add(b->t_candoff, P.sub.cand_off.data(), P.sub.cand_off.size() * 4);
        ar.add(b->t_candlist, P.sub.cand_list.data(),
                                           std::max<size_t>(2, P.sub.cand_list.size() * 2));
        ar.add(b->t_pktab, P.sub.pk_tab.data(), P.sub.pk_tab.size() * 4);
        ar.add(b->t_pkcand, P.sub.pk_cand.data(), P.sub.pk_cand.size() * 2);
    }
    if (P.kind == K_TAB)
        ar.add(b->t_bytes, P.bytes.tab.data(), P.bytes.tab.size() * 8);

    if (b->n_sym) XDG_RETURN_IF(ar.commit(b->tables));

    if (b->wide) {
        XDG_RETURN_IF(enumerate<uint64_t>(b, bt));
    } else {
        XDG_RETURN_IF(enumerate<uint32_t>(b, bt));
    }
    if (P.kind == K_U1) {
        XDG_RETURN_IF(build_lin(b));
    } else if (b->dim > 0) {
        if (b->wide) {
            XDG_RETURN_IF(build_rank<uint64_t>(b));
            if (!b->n_rwords) XDG_RETURN_IF(build_hash<uint64_t>(b));
        } else {
            XDG_RETURN_IF(build_rank<uint32_t>(b));
            if (!b->n_rwords) XDG_RETURN_IF(build_hash<uint32_t>(b));
        }
    }
    return XDG_OK;
}

// --------------------------------------------------- second labellings --
namespace {
std::mutex g_inner_mu;
std::vector<xdg_basis_s *> g_inner_of;   // the blocks that have a second labelling
}  // namespace

void offer_relabelled(xdg_basis_s *b, RelabelledRef in) {
    std::lock_guard<std::mutex> all(g_inner_mu);
    std::lock_guard<std::mutex> lock(b->inner_mu);
    b->inner = std::move(in);
    b->has_inner = b->had_inner = true;
    g_inner_of.push_back(b);
}

void forget_relabelled(xdg_basis_s *b) {
    if (!b->had_inner) return;
    // (also where it has been given up: that may still be under way)
    std::lock_guard<std::mutex> all(g_inner_mu);
    g_inner_of.erase(std::remove(g_inner_of.begin(), g_inner_of.end(), b), g_inner_of.end());
}

RelabelledRef relabelled(const xdg_ham_s *h, hipStream_t st) {
    xdg_basis_s *b = h->basis;
    if (!b->has_inner || !h->inner_bonds.d.p) return nullptr;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    bool captured = false;
    if (st) {
        captured = hipStreamIsCapturing(st, &cs) != hipSuccess ||
                   cs != hipStreamCaptureStatusNone;
    }
    std::lock_guard<std::mutex> lock(b->inner_mu);
    b->inner_captured |= captured && b->inner;
    return b->inner;
}

std::vector<RelabelledRef> relabelled(int n, xdg_ham_s *const *hams, hipStream_t st) {
    std::vector<RelabelledRef> in(n);
    for (int i = 0; i < n; ++i) in[i] = relabelled(hams[i], st);
    return in;
}

bool give_up_relabelled() {
    const uint64_t missing = take_missing_memory();
    if (!missing) return false;
    std::vector<RelabelledRef> gone;   // freed after the locks
    {
        std::lock_guard<std::mutex> all(g_inner_mu);
        uint64_t held = 0;
        for (xdg_basis_s *b : g_inner_of) {
            std::lock_guard<std::mutex> lock(b->inner_mu);
            if (b->inner && !b->inner_captured) held += b->inner->bytes;
        }
        if (held < missing) return false;
        for (xdg_basis_s *b : g_inner_of) {
            std::lock_guard<std::mutex> lock(b->inner_mu);
            if (!b->inner || b->inner_captured) continue;
            gone.push_back(std::move(b->inner));
            b->inner = nullptr;
            b->has_inner = false;
        }
        g_inner_of.erase(std::remove_if(g_inner_of.begin(), g_inner_of.end(),
                                        [](xdg_basis_s *b) { return !b->has_inner; }),
                         g_inner_of.end());
    }
    return true;
}

// ------------------------------------------------------- inner labelling --
namespace {

struct UserMapArgs {
    uint8_t site_bit[64];      // inner label of every site
    int N, n_sym;
    uint64_t dim;
    const uint64_t *bytetab;
    int n_bchunks;
    SubCtx sub;                // tables in device memory
    int n_s;                   // 0: byte tables
    RankArgs R;                // index of the caller's basis
    const void *hash;
    uint64_t n_lines;
    uint64_t empty;
    const double2 *chi;
    uint32_t *umap;
};

// umap[k] for the inner representatives: the state in the caller's labels,
// its representative s = u.t there, the position of s, and the sign chi(u)
// by which the two symmetric states differ.
template <class W>
__global__ __launch_bounds__(256) void k_user_map(const W *inner_reps, UserMapArgs A) {
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t k = (uint64_t)blockIdx.x * 256 + threadIdx.x; k < A.dim; k += stride) {
        const W r = inner_reps[k];
        W t = 0;
        for (int i = 0; i < A.N; ++i) t |= ((r >> A.site_bit[i]) & W(1)) << i;
        W s;
        int u, cnt;
        if (A.n_s == 0)
            tab_search<W>(A.bytetab, A.n_bchunks, A.n_sym, t, s, u, cnt);
        else
            sub_search<W, 0>(A.sub, t, s, u, cnt);
        const int64_t p = A.R.n_words
                              ? rank_find(A.R.words, A.R.n_words, colex_rank<W>(A.R.tab, A.R.L, s))
                              : hash_find<W>(A.hash, A.n_lines, (W)A.empty, s);
        // a state without a position (never: same sector) would show as 2^31 - 1
        A.umap[k] = (p < 0 ? 0x7FFFFFFFu : (uint32_t)p) | (A.chi[u].x < 0.0 ? 0x80000000u : 0u);
    }
}

__global__ __launch_bounds__(256) void k_map_check(const uint32_t *umap, uint64_t dim,
                                                   uint32_t *bad) {
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t k = (uint64_t)blockIdx.x * 256 + threadIdx.x; k < dim; k += stride)
        if ((umap[k] & 0x7FFFFFFFu) >= dim) atomicOr(bad, 1u);
}

}  // namespace

// Products with H do not need the caller's site labels: any labelling finds
// the orbit of a state, and a sector's vectors in two labellings differ by the
// order of the orbits and the signs of the characters.  Where the caller's
// labels leave only the byte tables (every element of the group tried for
// every term) or blocks that the packed sublattice search does not take, but
// the group respects some partition into four blocks of 5 to 10 sites, the
// products run in labels by those blocks and go through umap.  Only for
// characters of exactly +-1, so that no product is rounded twice.
// Measured: 6x6 lattice numbered row by row, 12 of 36 spins up, FP64, one
// vector 135.3 -> 3.4 ms (2.1 with the two-step packed search and block slots);
// 6x6 triangular lattice in three blocks of 12, 12 of 36 up, three FP64 vectors
// 25.8 -> 10.7 ms (3.7 with these and one pass for the three vectors).
//
static uint64_t basis_bytes(const xdg_basis_s *b) {
    uint64_t n = 0;
    for (const DevBuf *d : {&b->reps, &b->stab, &b->hash, &b->rwords, &b->rank_buf, &b->xr_top,
                            &b->xr_top32, &b->xr_rtab, &b->xb_buf, &b->tables})
        n += d->bytes;
    return n;
}

// wrong: the map does not fit the block (an error of this library's, returned).
static int build_inner(xdg_basis_s *b, bool few_rows, uint32_t *wrong) {
    const Plan &P = b->plan;
    if (b->dim < 1 || b->dim >= 0x7FFFFFFF || (P.flags & XDG_FLAG_HASH_INDEX)) return XDG_OK;
    if (P.kind != K_TAB && !(P.kind == K_SUB && !P.sub.packed())) return XDG_OK;
    // Blocks below the few-rows line whose tables leave 32 KiB of the LDS for that
    // loop's terms beside the rank tables (32 KiB at most) take it in either labels
    // and are prepared faster in one (4x6 square, 29606 rows, FP64: 89 us a product
    // in the caller's labels, 87 in others, and 3.1 against 5.0 ms before it; with
    // 6 of 24 up 57 and 45 us, 2.9 and 4.8 ms: a hundred and more products make up
    // for that).  Tables without that room keep them out of it (6x6 triangular
    // lattice, 5 of 36 up: 1.99 ms a product, 0.10 in others).
    if (P.kind == K_SUB && few_rows &&
        6 * ((size_t)P.sub.n_s << P.sub.m) + 2 * P.sub.cand_list.size() + 4 * P.sub.pid.size() +
                2 * P.sub.tperm.size() + 64 * 1024 < lds_limit())
        return XDG_OK;
    for (int g = 0; g < b->n_sym; ++g)
        if (std::fabs(b->chi[2 * g]) != 1.0 || b->chi[2 * g + 1] != 0.0) return XDG_OK;
    std::vector<int> pos = four_block_labels(b->n_sites, b->n_sym, b->perm.data());
    if (pos.empty()) return XDG_OK;
    auto rel = std::make_shared<Relabelled>();
    rel->basis = std::make_unique<xdg_basis_s>();
    xdg_basis_s *const in = rel->basis.get();
    in->device = b->device;
    in->n_sites = b->n_sites;
    in->n_up = b->n_up;
    in->n_sym = b->n_sym;
    in->wide = b->wide;
    in->chi = b->chi;
    in->perm = relabel_group(b->n_sites, b->n_sym, b->perm.data(), pos);
    xdg_basis_opts o{};
    o.search = XDG_SEARCH_SUBLATTICE;
    o.n_sublattices = 4;
    o.flags = P.flags;
    int rc = make_plan(in->n_sites, in->n_sym, in->perm.data(), &o, &in->plan, true);
    if (rc == XDG_OK) rc = basis_build_device(in);
    DevBuf &umap = rel->umap, bad;
    if (rc == XDG_OK && in->dim == b->dim) rc = umap.alloc(sizeof(uint32_t) * (size_t)b->dim);
    if (rc == XDG_OK) rc = bad.alloc(sizeof(uint32_t));
    XDG_RETURN_IF(rc);
    if (in->dim != b->dim || !in->n_rwords || !in->plan.sub.packed()) return XDG_OK;
    UserMapArgs A{};
    for (int i = 0; i < b->n_sites; ++i) A.site_bit[i] = (uint8_t)pos[i];
    A.N = b->n_sites;
    A.n_sym = b->n_sym;
    A.dim = (uint64_t)b->dim;
    A.bytetab = b->t_bytes.as<uint64_t>();
    A.n_bchunks = P.bytes.n_chunks;
    A.n_s = P.kind == K_SUB ? P.sub.n_s : 0;
    A.sub = SubCtx{b->t_mintop.as<uint16_t>(), b->t_candoff.as<uint32_t>(),
                   b->t_candlist.as<uint16_t>(), b->t_pid.as<uint32_t>(),
                   b->t_tperm.as<uint16_t>(), P.sub.n_s, P.sub.m, P.sub.pb};
    A.R = RankArgs{b->rwords.as<uint2>(), b->n_rwords, b->rtab.p, b->rank};
    A.hash = b->hash.p;
    A.n_lines = b->hidx.n_lines;
    A.empty = b->n_up == b->n_sites ? 0ull : (b->wide ? ~0ull : 0xFFFFFFFFull);
    A.chi = b->chi_d.as<double2>();
    A.umap = umap.as<uint32_t>();
    const unsigned grid = (unsigned)std::min<int64_t>((b->dim + 255) / 256,
                                                      (int64_t)device_cu_count() * 8);
    XDG_TRY_HIP(hipMemset(bad.p, 0, sizeof(uint32_t)));
    if (b->wide)
        hipLaunchKernelGGL(k_user_map<uint64_t>, dim3(grid), dim3(256), 0, 0,
                           in->reps.as<uint64_t>(), A);
    else
        hipLaunchKernelGGL(k_user_map<uint32_t>, dim3(grid), dim3(256), 0, 0,
                           in->reps.as<uint32_t>(), A);
    hipLaunchKernelGGL(k_map_check, dim3(grid), dim3(256), 0, 0, umap.as<uint32_t>(), A.dim,
                       bad.as<uint32_t>());
    XDG_TRY_HIP(hipGetLastError());
    XDG_RETURN_IF(copy_d2h(wrong, bad.p, sizeof *wrong, nullptr));
    if (*wrong) return XDG_EINVAL;
    rel->pos = std::move(pos);
    bad.release();
    rel->bytes = basis_bytes(in) + umap.bytes;
    // Device memory that the caller's own vectors may want is beyond the library's
    // sight, so the labelling stays only where it is a small part of what is left;
    // the library's own allocations make it give way (give_up_relabelled).
    size_t room = 0, all = 0;
    XDG_TRY_HIP(hipMemGetInfo(&room, &all));
    if (rel->bytes > room / 8) return XDG_OK;
    offer_relabelled(b, std::move(rel));
    return XDG_OK;
}

// The caller's block is complete without the inner one: whatever keeps that from
// being built (no room, a plan or an index that does not apply) leaves the block
// in the caller's labels and the thread's last error as it was.
int basis_build_inner(xdg_basis_s *b, bool few_rows) {
    const std::string before = get_error();
    uint32_t wrong = 0;
    const int rc = build_inner(b, few_rows, &wrong);
    if (rc == XDG_OK) return XDG_OK;
    if (wrong) {
        set_error("internal: an orbit of the relabelled sector has no place in the basis");
        return rc;
    }
    (void)hipGetLastError();
    XDG_TRY_HIP(hipDeviceSynchronize());   // an error that lasts
    set_error("%s", before.c_str());
    return XDG_OK;
}

// Chunk tables of the colex rank of a block without a group (its positions).
int u1_rank_tables(const xdg_basis_s *b, DevBuf *tab, RankLayout *L) {
    *L = rank_layout(b->n_sites, b->n_up, b->wide, (uint64_t)b->dim - 1);
    if (L->e32) {
        std::vector<uint32_t> T;
        rank_tables<uint32_t>(b->n_sites, b->n_up, *L, T);
        return tab->upload(T.data(), T.size() * 4);
    }
    std::vector<uint64_t> T;
    rank_tables<uint64_t>(b->n_sites, b->n_up, *L, T);
    return tab->upload(T.data(), T.size() * 8);
}

int basis_lookup(xdg_basis_s *b, const uint64_t *d_states, int64_t n, int64_t *d_idx,
                 hipStream_t st) {
    if (n <= 0) return XDG_OK;
    const int block = 256;
    const unsigned grid = (unsigned)((n + block - 1) / block);
    const int u1 = b->plan.kind == K_U1;
    const RankArgs R{b->rwords.as<uint2>(), b->n_rwords, b->rtab.p, b->rank};
    if (b->wide) {
        const uint64_t empty = b->n_up == b->n_sites ? 0ull : ~0ull;
        hipLaunchKernelGGL(k_lookup<uint64_t>, dim3(grid), dim3(block), 0, st, d_states, n, d_idx,
                           b->n_sites, b->n_up, u1, b->lin.as<uint32_t>(), b->lin_nlo, b->hash.p,
                           b->dim > 0 ? b->hidx.n_lines : 0, empty, R);
    } else {
        const uint32_t empty = b->n_up == b->n_sites ? 0u : ~0u;
        hipLaunchKernelGGL(k_lookup<uint32_t>, dim3(grid), dim3(block), 0, st, d_states, n, d_idx,
                           b->n_sites, b->n_up, u1, b->lin.as<uint32_t>(), b->lin_nlo, b->hash.p,
                           b->dim > 0 ? b->hidx.n_lines : 0, empty, R);
    }
    XDG_TRY_HIP(hipGetLastError());
    return XDG_OK;
}

}  // namespace xdg
