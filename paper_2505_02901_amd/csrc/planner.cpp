// Host-side planning for a sector: validation of the permutation group and
// its characters (Sec. 3.10.1, 3.10.2), invariance of the bond list
// (well-defined quantum numbers, Sec. 3.6 / 3.10), choice of the
// representative-search kind and construction of its lookup tables
// (Sec. 5.1 backends, Sec. 5.2: lookup tables for the symmetry action,
// sublattice coding).
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <unordered_map>

#include "xdg_internal.hpp"

namespace xdg {

namespace {
thread_local std::string g_err;

struct VecHash {
    size_t operator()(const std::vector<int32_t> &v) const {
        uint64_t h = 1469598103934665603ull;
        for (int32_t x : v) {
            h ^= (uint64_t)(uint32_t)x;
            h *= 1099511628211ull;
        }
        return (size_t)h;
    }
};
}  // namespace

void set_error(const char *fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
}

const char *get_error() { return g_err.c_str(); }

uint64_t binomial(int n, int k) {
    static uint64_t t[65][65];
    static bool ready = false;
    if (!ready) {
        for (int a = 0; a <= 64; ++a) {
            t[a][0] = 1;
            for (int b = 1; b <= a; ++b) t[a][b] = t[a - 1][b - 1] + (b < a ? t[a - 1][b] : 0);
        }
        ready = true;
    }
    if (n < 0 || k < 0 || k > n || n > 64) return 0;
    return t[n][k];
}

// --------------------------------------------------------- group checks --
namespace {

// Fast acceptance of a valid group and character table: true only if every
// check of validate_group below holds.  The products with a few generators
// (found on the way: every element not yet reached becomes one) give the whole
// multiplication table by lookups, f (g h) = (f g) h, instead of a composition
// and a hash search for each of the |G|^2 products (288 elements of 36 sites:
// 11 ms -> 0.9 ms); the characters are still checked for every pair.
bool group_holds(int N, int n_sym, const int32_t *perm, const double *chi) {
    if (n_sym > 4096) return false;
    std::unordered_map<std::vector<int32_t>, int, VecHash> where;
    std::vector<int32_t> row(N);
    int id = -1;
    for (int g = 0; g < n_sym; ++g) {
        uint64_t seen = 0;
        bool same = true;
        for (int i = 0; i < N; ++i) {
            const int32_t v = perm[(size_t)g * N + i];
            if (v < 0 || v >= N || (seen >> v) & 1) return false;
            seen |= 1ull << v;
            same &= v == i;
        }
        row.assign(perm + (size_t)g * N, perm + (size_t)(g + 1) * N);
        if (!where.emplace(row, g).second) return false;
        if (same) id = g;
    }
    if (id < 0) return false;
    // right[h][f] = f o gen_h; elements reached from the identity, with the
    // element and generator they were reached by
    std::vector<std::vector<int>> right;
    std::vector<int> gens, order{id}, from(n_sym, -1), by(n_sym, -1);
    std::vector<char> reached(n_sym, 0);
    reached[id] = 1;
    int next = 0;
    while ((int)order.size() < n_sym) {
        while (reached[next]) ++next;
        if (gens.size() >= 16) return false;
        const int32_t *ph = perm + (size_t)next * N;
        std::vector<int> r(n_sym);
        for (int f = 0; f < n_sym; ++f) {
            for (int i = 0; i < N; ++i) row[i] = perm[(size_t)f * N + ph[i]];
            const auto it = where.find(row);
            if (it == where.end()) return false;
            r[f] = it->second;
        }
        right.push_back(std::move(r));
        gens.push_back(next);
        for (size_t a = 0; a < order.size(); ++a)   // grows while new ones are found
            for (size_t h = 0; h < gens.size(); ++h) {
                const int to = right[h][order[a]];
                if (reached[to]) continue;
                reached[to] = 1;
                from[to] = order[a];
                by[to] = (int)h;
                order.push_back(to);
            }
    }
    // closed under the generators, and generated by them: a group (finite, so
    // inverses are there too)
    if (!chi) return true;
    constexpr double tol = 1e-12;
    for (int g = 0; g < n_sym; ++g) {
        const double a = std::hypot(chi[2 * g], chi[2 * g + 1]);
        if (!std::isfinite(a) || std::fabs(a - 1.0) > tol) return false;
    }
    std::vector<int> prod((size_t)n_sym * n_sym);   // prod[g][f] = f o g
    for (int f = 0; f < n_sym; ++f) prod[(size_t)id * n_sym + f] = f;
    for (size_t a = 1; a < order.size(); ++a) {
        const int g = order[a];
        const int *p = &prod[(size_t)from[g] * n_sym], *r = right[by[g]].data();
        int *q = &prod[(size_t)g * n_sym];
        for (int f = 0; f < n_sym; ++f) q[f] = r[p[f]];
    }
    for (int g = 0; g < n_sym; ++g) {
        const double gr = chi[2 * g], gi = chi[2 * g + 1];
        const int *q = &prod[(size_t)g * n_sym];
        for (int f = 0; f < n_sym; ++f) {
            const double fr = chi[2 * f], fi = chi[2 * f + 1];
            const double dr = fr * gr - fi * gi - chi[2 * q[f]];
            const double di = fr * gi + fi * gr - chi[2 * q[f] + 1];
            if (!(dr * dr + di * di <= 0.25 * tol * tol)) return false;   // the full check decides
        }
    }
    return true;
}

// Fast acceptance of an invariant bond list: couplings summed per pair of
// sites in a table, every pair compared with its image under every element
// (288 elements, 144 bonds: 7 ms -> 0.1 ms).  With a group, a pair whose
// source is no bond is met as the image under the inverse element.
bool bonds_hold(int N, int n_sym, const int32_t *perm, int n_bonds, const int32_t *sites,
                const double *jz, const double *jxy) {
    std::vector<double> z((size_t)N * N, 0.0), x((size_t)N * N, 0.0);
    std::vector<std::pair<int, int>> pairs;
    std::vector<char> have((size_t)N * N, 0);
    double scale = 0.0;
    for (int b = 0; b < n_bonds; ++b) {
        const int i = sites[2 * b], j = sites[2 * b + 1];
        if (i < 0 || j < 0 || i >= N || j >= N || i == j || !std::isfinite(jz[b]) ||
            !std::isfinite(jxy[b]))
            return false;
        const size_t k = (size_t)std::min(i, j) * N + std::max(i, j);
        if (!have[k]) pairs.push_back({std::min(i, j), std::max(i, j)});
        have[k] = 1;
        z[k] += jz[b];
        x[k] += jxy[b];
        scale = std::max(scale, std::max(std::fabs(jz[b]), std::fabs(jxy[b])));
    }
    const double tol = 1e-12 * std::max(scale, 1e-300);
    for (int g = 0; g < n_sym; ++g) {
        const int32_t *pg = perm + (size_t)g * N;
        for (const auto &p : pairs) {
            const int a = pg[p.first], c = pg[p.second];
            const size_t k = (size_t)p.first * N + p.second,
                         q = (size_t)std::min(a, c) * N + std::max(a, c);
            if (!(std::fabs(z[q] - z[k]) <= tol) || !(std::fabs(x[q] - x[k]) <= tol)) return false;
        }
    }
    return true;
}

}  // namespace

int validate_group(int n_sites, int n_sym, const int32_t *perm, const double *chi) {
    if (n_sites < 1 || n_sites > 64) {
        set_error("n_sites = %d outside [1, 64]", n_sites);
        return XDG_EINVAL;
    }
    if (n_sym == 0) return XDG_OK;
    if (n_sym < 0 || !perm) {
        set_error("n_sym = %d with perm %s", n_sym, perm ? "set" : "NULL");
        return XDG_EINVAL;
    }
    const int N = n_sites;
    if (group_holds(N, n_sym, perm, chi)) return XDG_OK;
    // something is wrong (or the group is very large): find out what
    std::unordered_map<std::vector<int32_t>, int, VecHash> where;
    std::vector<int32_t> row(N);
    for (int g = 0; g < n_sym; ++g) {
        std::vector<char> seen(N, 0);
        for (int i = 0; i < N; ++i) {
            int32_t v = perm[(size_t)g * N + i];
            if (v < 0 || v >= N || seen[v]) {
                set_error("permutation %d is not a bijection of the %d sites", g, N);
                return XDG_EINVAL;
            }
            seen[v] = 1;
        }
        row.assign(perm + (size_t)g * N, perm + (size_t)(g + 1) * N);
        if (where.count(row)) {
            set_error("permutation %d appears twice in the group", g);
            return XDG_EGROUP;
        }
        where[row] = g;
    }
    // identity
    for (int i = 0; i < N; ++i) row[i] = i;
    auto it = where.find(row);
    if (it == where.end()) {
        set_error("the group lacks the identity permutation");
        return XDG_EGROUP;
    }
    // inverses
    for (int g = 0; g < n_sym; ++g) {
        for (int i = 0; i < N; ++i) row[perm[(size_t)g * N + i]] = i;
        if (!where.count(row)) {
            set_error("the inverse of permutation %d is missing", g);
            return XDG_EGROUP;
        }
    }
    // closure and the homomorphism property of the characters
    const double tol = 1e-12;
    if (chi) {
        for (int g = 0; g < n_sym; ++g) {
            double a = std::hypot(chi[2 * g], chi[2 * g + 1]);
            if (!std::isfinite(a) || std::fabs(a - 1.0) > tol) {
                set_error("|chi(%d)| = %.17g is not 1", g, a);
                return XDG_ECHAR;
            }
        }
    }
    for (int f = 0; f < n_sym; ++f) {
        const int32_t *pf = perm + (size_t)f * N;
        for (int g = 0; g < n_sym; ++g) {
            const int32_t *pg = perm + (size_t)g * N;
            for (int i = 0; i < N; ++i) row[i] = pf[pg[i]];   // (f o g)(i)
            auto h = where.find(row);
            if (h == where.end()) {
                set_error("product of permutations %d and %d is not in the group", f, g);
                return XDG_EGROUP;
            }
            if (chi) {
                std::complex<double> cf(chi[2 * f], chi[2 * f + 1]);
                std::complex<double> cg(chi[2 * g], chi[2 * g + 1]);
                std::complex<double> ch(chi[2 * h->second], chi[2 * h->second + 1]);
                if (std::abs(cf * cg - ch) > tol) {
                    set_error("characters violate chi(f)chi(g) = chi(fg) for f=%d g=%d", f, g);
                    return XDG_ECHAR;
                }
            }
        }
    }
    return XDG_OK;
}

int validate_bonds(int n_sites, int n_sym, const int32_t *perm, int n_bonds, const int32_t *sites,
                   const double *jz, const double *jxy) {
    if (n_bonds < 0 || (n_bonds > 0 && (!sites || !jz || !jxy))) {
        set_error("bad bond arrays");
        return XDG_EINVAL;
    }
    if (bonds_hold(n_sites, n_sym, perm, n_bonds, sites, jz, jxy)) return XDG_OK;
    std::map<std::pair<int, int>, std::pair<double, double>> agg;
    double scale = 0.0;
    for (int b = 0; b < n_bonds; ++b) {
        int i = sites[2 * b], j = sites[2 * b + 1];
        if (i < 0 || j < 0 || i >= n_sites || j >= n_sites || i == j) {
            set_error("bond %d = (%d, %d) is not a pair of distinct sites in [0, %d)", b, i, j,
                      n_sites);
            return XDG_EINVAL;
        }
        if (!std::isfinite(jz[b]) || !std::isfinite(jxy[b])) {
            set_error("bond %d has a non-finite coupling", b);
            return XDG_EINVAL;
        }
        auto &a = agg[{std::min(i, j), std::max(i, j)}];
        a.first += jz[b];
        a.second += jxy[b];
        scale = std::max(scale, std::max(std::fabs(jz[b]), std::fabs(jxy[b])));
    }
    const double tol = 1e-12 * std::max(scale, 1e-300);
    for (int g = 0; g < n_sym; ++g) {
        const int32_t *pg = perm + (size_t)g * n_sites;
        std::map<std::pair<int, int>, std::pair<double, double>> img;
        for (auto &kv : agg) {
            int i = pg[kv.first.first], j = pg[kv.first.second];
            auto &a = img[{std::min(i, j), std::max(i, j)}];
            a.first += kv.second.first;
            a.second += kv.second.second;
        }
        for (auto &kv : img) {
            auto f = agg.find(kv.first);
            double z = f == agg.end() ? 0.0 : f->second.first;
            double x = f == agg.end() ? 0.0 : f->second.second;
            if (std::fabs(z - kv.second.first) > tol || std::fabs(x - kv.second.second) > tol) {
                set_error("the bond list is not invariant under permutation %d", g);
                return XDG_ENOTSYM;
            }
        }
        for (auto &kv : agg) {
            if (!img.count(kv.first) &&
                (std::fabs(kv.second.first) > tol || std::fabs(kv.second.second) > tol)) {
                set_error("the bond list is not invariant under permutation %d", g);
                return XDG_ENOTSYM;
            }
        }
    }
    return XDG_OK;
}

// --------------------------------------------------------- search kinds --
namespace {

bool detect_affine(int N, int n_sym, const int32_t *perm, std::vector<AffineElem> *out) {
    std::vector<AffineElem> v;
    for (int g = 0; g < n_sym; ++g) {
        const int32_t *p = perm + (size_t)g * N;
        int a = p[0];
        bool plus = true, minus = true;
        for (int i = 0; i < N; ++i) {
            if (p[i] != (a + i) % N) plus = false;
            if (p[i] != ((a - i) % N + N) % N) minus = false;
        }
        if (!plus && !minus) return false;
        // (g.t)_i = t_{g(i)}:  plus  -> image = rotr_N(t, a)
        //                      minus -> image = rotr_N(rev_N(t), (N - 1 - a) mod N)
        if (plus)
            v.push_back({a, +1});
        else
            v.push_back({((N - 1 - a) % N + N) % N, -1});
    }
    if (out) *out = v;
    return true;
}

// Blocks q = sites [q m, (q+1) m).  Stable if every g maps the sites of
// each block onto the sites of one block.
bool detect_sublattice(int N, int n_sym, const int32_t *perm, int n_s, std::vector<uint8_t> *src) {
    if (n_s < 2 || N % n_s) return false;
    const int m = N / n_s;
    std::vector<uint8_t> s((size_t)n_sym * n_s);
    for (int g = 0; g < n_sym; ++g) {
        const int32_t *p = perm + (size_t)g * N;
        for (int a = 0; a < n_s; ++a) {
            int k = p[a * m] / m;
            for (int w = 0; w < m; ++w)
                if (p[a * m + w] / m != k) return false;
            s[(size_t)g * n_s + a] = (uint8_t)k;
        }
    }
    if (src) *src = s;
    return true;
}

void build_sublattice(int N, int n_sym, const int32_t *perm, int n_s, SublatticeTables *T) {
    const int m = N / n_s;
    const int V = 1 << m;
    const int pb = (m + 1) / 2, E = 1 << pb;
    T->n_s = n_s;
    T->m = m;
    T->pb = pb;
    detect_sublattice(N, n_sym, perm, n_s, &T->src);
    // distinct block permutations: image bit w of block a takes source bit
    // p[a m + w] - k m of block k = src[g][a]
    std::map<std::vector<int>, int> ids;
    std::vector<std::vector<int>> perms;
    T->pid.assign((size_t)n_sym * n_s, 0);
    for (int g = 0; g < n_sym; ++g) {
        const int32_t *p = perm + (size_t)g * N;
        for (int a = 0; a < n_s; ++a) {
            const int k = T->src[(size_t)g * n_s + a];
            std::vector<int> bw(m);
            for (int w = 0; w < m; ++w) bw[w] = p[a * m + w] - k * m;
            auto it = ids.find(bw);
            if (it == ids.end()) {
                it = ids.emplace(bw, (int)perms.size()).first;
                perms.push_back(bw);
            }
            T->pid[(size_t)g * n_s + a] = (uint16_t)it->second;
        }
    }
    T->n_perm = (int)perms.size();
    T->tperm.assign((size_t)T->n_perm * 2 * E, 0);
    for (int q = 0; q < T->n_perm; ++q) {
        std::vector<int> dst(m);   // source bit -> image bit
        for (int w = 0; w < m; ++w) dst[perms[q][w]] = w;
        for (int h = 0; h < 2; ++h)
            for (int u = 0; u < E; ++u) {
                uint32_t r = 0;
                for (int j = 0; j < pb; ++j) {
                    const int sb = h * pb + j;
                    if (sb < m && ((u >> j) & 1)) r |= 1u << dst[sb];
                }
                T->tperm[((size_t)q * 2 + h) * E + u] = (uint16_t)r;
            }
    }
    auto image = [&](int g, int a, int v) -> uint32_t {
        const uint16_t *tp = &T->tperm[(size_t)T->pid[(size_t)g * n_s + a] * 2 * E];
        return (uint32_t)tp[v & (E - 1)] | tp[E + (v >> pb)];
    };
    const int top = n_s - 1;
    T->mintop.assign((size_t)n_s * V, 0xFFFF);
    std::vector<std::vector<uint16_t>> lists((size_t)n_s * V);
    for (int g = 0; g < n_sym; ++g) {
        int k = T->src[(size_t)g * n_s + top];
        for (int v = 0; v < V; ++v) {
            const uint16_t im = (uint16_t)image(g, top, v);
            uint16_t &mt = T->mintop[(size_t)k * V + v];
            auto &L = lists[(size_t)k * V + v];
            if (im < mt) {
                mt = im;
                L.clear();
            }
            if (im == mt) L.push_back((uint16_t)g);
        }
    }
    T->cand_off.assign((size_t)n_s * V + 1, 0);
    T->cand_list.clear();
    for (size_t e = 0; e < lists.size(); ++e) {
        T->cand_off[e] = (uint32_t)T->cand_list.size();
        T->cand_list.insert(T->cand_list.end(), lists[e].begin(), lists[e].end());
    }
    T->cand_off.back() = (uint32_t)T->cand_list.size();
    // packed form, where its fields hold everything
    // (2048: more than the kernels' own shared data before the entries)
    if (!sub_packed_ok(n_s, m, pb) || 16 * (n_sym + 1) + 2048 > 65536) return;
    size_t longest = 1, pairs = 0;
    for (const auto &L : lists) {
        longest = std::max(longest, (L.size() + 1) / 2);
        pairs += (L.size() + 1) / 2;
    }
    int nb = 1;
    while (((size_t)1 << nb) <= longest) ++nb;
    if (nb > 31 - m || pairs >= (size_t)1 << (31 - m - nb)) return;
    T->pk_nb = nb;
    for (size_t e = 0; e < lists.size(); ++e) {
        const auto &L = lists[e];
        const uint32_t top_bits = L.empty() ? (uint32_t)V : T->mintop[e];
        T->pk_tab.push_back(top_bits << (31 - m) | (uint32_t)(T->pk_cand.size() / 2) << nb |
                            (uint32_t)((L.size() + 1) / 2));
        for (uint16_t g : L) T->pk_cand.push_back((uint16_t)(g * 16));
        if (L.size() & 1) T->pk_cand.push_back((uint16_t)(n_sym * 16));
    }
}

void build_bytes(int N, int n_sym, const int32_t *perm, ByteTables *B) {
    const int C = (N + 7) / 8;
    B->n_chunks = C;
    B->tab.assign((size_t)n_sym * C * 256, 0);
    std::vector<int> inv(N);
    for (int g = 0; g < n_sym; ++g) {
        const int32_t *p = perm + (size_t)g * N;
        for (int i = 0; i < N; ++i) inv[p[i]] = i;   // bit j of t lands on bit inv[j]
        for (int c = 0; c < C; ++c)
            for (int v = 0; v < 256; ++v) {
                uint64_t r = 0;
                for (int bit = 0; bit < 8; ++bit) {
                    int j = 8 * c + bit;
                    if (j < N && ((v >> bit) & 1)) r |= 1ull << inv[j];
                }
                B->tab[((size_t)g * C + c) * 256 + v] = r;
            }
    }
}

}  // namespace

std::vector<int32_t> relabel_group(int N, int n_sym, const int32_t *perm,
                                   const std::vector<int> &pos) {
    std::vector<int32_t> out((size_t)n_sym * N);
    for (int g = 0; g < n_sym; ++g)
        for (int i = 0; i < N; ++i)
            out[(size_t)g * N + pos[i]] = pos[perm[(size_t)g * N + i]];
    return out;
}

// The partitions of the sites that the group respects: for a transitive group
// the smallest one joining site 0 with site j, for every j, and the joins of
// those found.  Of those with four classes of 5 to 10 sites the one with the
// fewest candidate elements in its search tables is taken.
std::vector<int> four_block_labels(int N, int n_sym, const int32_t *perm) {
    if (N % 4 || !sub_packed_ok(4, N / 4, (N / 4 + 1) / 2) || n_sym < 4 || n_sym > 4096) return {};
    using Classes = std::vector<int>;   // smallest site of each site's class
    struct Join {
        std::vector<int> up;
        int find(int a) {
            while (up[a] != a) a = up[a] = up[up[a]];
            return a;
        }
    };
    // the finest respected partition that joins every pair given
    auto close = [&](std::vector<std::pair<int, int>> pairs) {
        Join u;
        for (int i = 0; i < N; ++i) u.up.push_back(i);
        while (!pairs.empty()) {
            const auto [a, b] = pairs.back();
            pairs.pop_back();
            const int x = u.find(a), y = u.find(b);
            if (x == y) continue;
            u.up[std::max(x, y)] = std::min(x, y);
            for (int g = 0; g < n_sym; ++g) {
                const int32_t *q = perm + (size_t)g * N;
                if (u.find(q[a]) != u.find(q[b])) pairs.push_back({q[a], q[b]});
            }
        }
        Classes c(N);
        for (int i = 0; i < N; ++i) c[i] = u.find(i);
        return c;
    };
    std::vector<Classes> found;
    auto add = [&](Classes c) {
        if (std::find(found.begin(), found.end(), c) == found.end()) found.push_back(std::move(c));
    };
    for (int j = 1; j < N; ++j) add(close({{0, j}}));
    for (size_t a = 0; a < found.size() && found.size() < 64; ++a)
        for (size_t b = 0; b < a && found.size() < 64; ++b) {
            std::vector<std::pair<int, int>> both;
            for (int i = 0; i < N; ++i) {
                both.push_back({i, found[a][i]});
                both.push_back({i, found[b][i]});
            }
            add(close(both));
        }
    std::vector<int> best;
    size_t best_cost = ~(size_t)0;
    for (const Classes &c : found) {
        std::map<int, std::vector<int>> blocks;
        for (int i = 0; i < N; ++i) blocks[c[i]].push_back(i);
        bool ok = blocks.size() == 4;
        for (const auto &b : blocks) ok &= (int)b.second.size() == N / 4;
        if (!ok) continue;
        std::vector<int> pos(N);
        int at = 0;
        for (const auto &b : blocks)
            for (int i : b.second) pos[i] = at++;
        SublatticeTables T;
        build_sublattice(N, n_sym, relabel_group(N, n_sym, perm, pos).data(), 4, &T);
        if (T.cand_list.size() < best_cost) {
            best_cost = T.cand_list.size();
            best = pos;
        }
    }
    return best;
}

int make_plan(int n_sites, int n_sym, const int32_t *perm, const xdg_basis_opts *opts, Plan *plan,
              bool build_tables) {
    const int want = opts ? opts->search : XDG_SEARCH_AUTO;
    const int want_ns = opts ? opts->n_sublattices : 0;
    if (opts) {
        for (int r : opts->reserved)
            if (r != 0) {
                set_error("xdg_basis_opts.reserved must be zero");
                return XDG_EINVAL;
            }
    }
    if (want < XDG_SEARCH_AUTO || want > XDG_SEARCH_TABLE) {
        set_error("unknown search kind %d", want);
        return XDG_EINVAL;
    }
    const int flags = opts ? opts->flags : 0;
    if (flags & ~(XDG_FLAG_F32_ACCUMULATE | XDG_FLAG_HASH_INDEX)) {
        set_error("unknown flags 0x%x", flags);
        return XDG_EINVAL;
    }
    Plan p;
    p.flags = flags;
    if (n_sym == 0) {
        if (want != XDG_SEARCH_AUTO && want != XDG_SEARCH_U1) {
            set_error("search kind %d needs a permutation group", want);
            return XDG_EINVAL;
        }
        p.kind = XDG_SEARCH_U1;
        *plan = std::move(p);
        return XDG_OK;
    }
    if (want == XDG_SEARCH_U1) {
        set_error("XDG_SEARCH_U1 given together with a permutation group");
        return XDG_EINVAL;
    }
    if (n_sym > 65535) {
        set_error("groups of more than 65535 elements are not supported");
        return XDG_EINVAL;
    }
    const int N = n_sites;
    if (want == XDG_SEARCH_AUTO || want == XDG_SEARCH_AFFINE) {
        if (detect_affine(N, n_sym, perm, &p.aff)) {
            p.kind = XDG_SEARCH_AFFINE;
            std::vector<int16_t> gi(2 * (size_t)N, -1);
            int n_rot = 0, n_ref = 0;
            for (int g = 0; g < n_sym; ++g) {
                const AffineElem &e = p.aff[g];
                int16_t &slot = gi[(e.eps > 0 ? 0 : N) + e.a];
                if (slot < 0) {
                    slot = (int16_t)g;
                    (e.eps > 0 ? n_rot : n_ref)++;
                }
            }
            if (n_rot == N && (n_ref == 0 || n_ref == N) && n_sym == n_rot + n_ref && N <= 64) {
                p.ring = n_ref ? 2 : 1;
                p.ring_gidx = gi;
            }
            *plan = std::move(p);
            return XDG_OK;
        }
        if (want == XDG_SEARCH_AFFINE) {
            set_error("the group is not made of ring translations/reflections i -> +-i + a");
            return XDG_EINVAL;
        }
    }
    if (want == XDG_SEARCH_AUTO || want == XDG_SEARCH_SUBLATTICE) {
        int chosen = 0;
        if (want_ns) {
            if (N % want_ns == 0 && N / want_ns <= 16 && detect_sublattice(N, n_sym, perm, want_ns, nullptr))
                chosen = want_ns;
        } else {
            for (int ns = 2; ns <= 8 && !chosen; ++ns)
                if (N % ns == 0 && N / ns <= 12 && detect_sublattice(N, n_sym, perm, ns, nullptr))
                    chosen = ns;
        }
        if (chosen) {
            p.kind = XDG_SEARCH_SUBLATTICE;
            if (build_tables) build_sublattice(N, n_sym, perm, chosen, &p.sub);
            p.sub.n_s = chosen;
            p.sub.m = N / chosen;
            *plan = std::move(p);
            return XDG_OK;
        }
        if (want == XDG_SEARCH_SUBLATTICE) {
            set_error("the labelling has no stable block partition into %d sublattices",
                      want_ns);
            return XDG_EINVAL;
        }
    }
    p.kind = XDG_SEARCH_TABLE;
    if (build_tables) build_bytes(N, n_sym, perm, &p.bytes);
    p.bytes.n_chunks = (N + 7) / 8;
    *plan = std::move(p);
    return XDG_OK;
}

}  // namespace xdg
