// Host-side construction of the H^2 structure (Sec. 4.6 "ab initio"
// generation): KD-tree bisection of the points, tight boxes, and the dual
// traversal that splits the matrix into admissible (coupling) blocks at every
// level and dense blocks at the leaf level (Sec. 2.2), each level kept as
// block-sparse rows (Sec. 4.3, Fig. 5).
//
// Rules taken where the paper leaves the choice open:
//  - leaf level q is the smallest with n <= leaf * 2^q, and every node above
//    it is bisected (a complete tree, as the per-level batch sizes of the
//    upsweep and downsweep algorithms imply);
//  - a node is split along the widest axis of its tight box (lowest axis on
//    ties), its points ordered by (coordinate, input index), the first half
//    (rounded down) going to the first child;
//  - boxes are tight; an axis of zero extent is widened symmetrically to
//    1e-12 * max(1, widest extent of the root box);
//  - (s, t) is admissible when max(diam s, diam t) <= eta * dist(s, t) > 0,
//    with Euclidean box diameters and box gap.
#include "h2_structure.h"

#include <algorithm>
#include <cmath>
#include <future>
#include <numeric>
#include <thread>

namespace h2 {
namespace {

// Splits node v of a level.  Its points need a full order only at the last
// split, where each half becomes a leaf (the order is total, so which points
// go to which child does not depend on how they are selected).
struct Key {
    double c;
    int64_t i;
    bool operator<(const Key &o) const { return c < o.c || (c == o.c && i < o.i); }
};

void split_node(const double *points, int dim, int level, int64_t v, Structure &s, std::vector<Key> &keys) {
    const int64_t b = s.begin[v], e = s.end[v], mid = b + (e - b) / 2;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = b; i < e; ++i)
        for (int a = 0; a < dim; ++a) {
            const double c = points[s.perm[i] * dim + a];
            lo[a] = std::min(lo[a], c);
            hi[a] = std::max(hi[a], c);
        }
    int axis = 0;
    for (int a = 1; a < dim; ++a)
        if (hi[a] - lo[a] > hi[axis] - lo[axis]) axis = a;
    keys.resize(size_t(e - b));
    for (int64_t i = b; i < e; ++i) keys[size_t(i - b)] = {points[s.perm[i] * dim + axis], s.perm[i]};
    if (level == s.q - 1) std::sort(keys.begin(), keys.end());
    else std::nth_element(keys.begin(), keys.begin() + (mid - b), keys.end());
    for (int64_t i = b; i < e; ++i) s.perm[i] = keys[size_t(i - b)].i;
    s.begin[2 * v + 1] = b;
    s.end[2 * v + 1] = mid;
    s.begin[2 * v + 2] = mid;
    s.end[2 * v + 2] = e;
}

// Splits all levels (with the traversal on the host threads below, the
// structure of 65,536 points in 2-D takes 6.8 instead of 32 ms on 8 threads,
// 4,096 points on one 0.9 instead of 2.2): those of few nodes one after the other, nodes spread
// over the host threads, then every subtree below them by one thread.
void split_levels(const double *points, int dim, Structure &s) {
    const int top = s.n < 8192 ? 0 : std::min(s.q, 4);
    for (int l = 0; l < top; ++l)
        parallel_ranges(int64_t(1) << l, 1, [&](int64_t j0, int64_t j1) {
            std::vector<Key> keys;
            for (int64_t j = j0; j < j1; ++j) split_node(points, dim, l, Structure::first(l) + j, s, keys);
        });
    parallel_ranges(int64_t(1) << top, 1, [&](int64_t j0, int64_t j1) {
        std::vector<Key> keys;
        for (int64_t j = j0; j < j1; ++j)
            for (int l = top; l < s.q; ++l)
                for (int64_t i = j << (l - top); i < (j + 1) << (l - top); ++i)
                    split_node(points, dim, l, Structure::first(l) + i, s, keys);
    });
}

void compute_boxes(Structure &s) {
    const int dim = s.dim;
    s.lo.assign(s.nnodes * dim, INFINITY);
    s.hi.assign(s.nnodes * dim, -INFINITY);
    // leaves from their points, inner nodes as the union of their children
    const int64_t lf = Structure::first(s.q);
    for (int64_t v = lf; v < s.nnodes; ++v)
        for (int64_t i = s.begin[v]; i < s.end[v]; ++i)
            for (int a = 0; a < dim; ++a) {
                s.lo[v * dim + a] = std::min(s.lo[v * dim + a], s.pts[i * dim + a]);
                s.hi[v * dim + a] = std::max(s.hi[v * dim + a], s.pts[i * dim + a]);
            }
    for (int64_t v = lf - 1; v >= 0; --v)
        for (int a = 0; a < dim; ++a) {
            s.lo[v * dim + a] = std::min(s.lo[(2 * v + 1) * dim + a], s.lo[(2 * v + 2) * dim + a]);
            s.hi[v * dim + a] = std::max(s.hi[(2 * v + 1) * dim + a], s.hi[(2 * v + 2) * dim + a]);
        }
    double widest = 0.0;
    for (int a = 0; a < dim; ++a) widest = std::max(widest, s.hi[a] - s.lo[a]);
    const double delta = 1e-12 * std::max(1.0, widest);
    for (int64_t v = 0; v < s.nnodes; ++v)
        for (int a = 0; a < dim; ++a)
            if (s.hi[v * dim + a] - s.lo[v * dim + a] == 0.0) {
                s.lo[v * dim + a] -= 0.5 * delta;
                s.hi[v * dim + a] += 0.5 * delta;
            }
}

std::vector<double> diameters(const Structure &s) {
    std::vector<double> diam(size_t(s.nnodes));
    for (int64_t v = 0; v < s.nnodes; ++v) {
        double acc = 0.0;
        for (int a = 0; a < s.dim; ++a) {
            const double e = s.hi[v * s.dim + a] - s.lo[v * s.dim + a];
            acc += e * e;
        }
        diam[v] = std::sqrt(acc);
    }
    return diam;
}

typedef std::vector<std::pair<int32_t, int32_t>> Pairs;

struct Traversal {
    const Structure &s;
    const std::vector<double> &diam;
    std::vector<Pairs> lists;   // per level
    Pairs dense;
    int64_t near_ties = 0;

    Traversal(const Structure &st, const std::vector<double> &d) : s(st), diam(d), lists(st.q + 1) {}

    double gap(int64_t a, int64_t b) const {
        double acc = 0.0;
        for (int x = 0; x < s.dim; ++x) {
            double g = 0.0;
            g = std::max(g, s.lo[a * s.dim + x] - s.hi[b * s.dim + x]);
            g = std::max(g, s.lo[b * s.dim + x] - s.hi[a * s.dim + x]);
            acc += g * g;
        }
        return std::sqrt(acc);
    }

    // Pairs not decided at level `stop` are left in rest.
    void visit(int64_t a, int64_t b, int level, int stop, Pairs *rest) {
        if (level == stop && rest) {
            rest->emplace_back(int32_t(a), int32_t(b));
            return;
        }
        const double size = std::max(diam[a], diam[b]);
        const double far = s.eta * gap(a, b);
        if (far > 0.0 && std::fabs(size - far) < 1e-12 * far) ++near_ties;
        const int64_t f = Structure::first(level);
        if (far > 0.0 && size <= far) {
            lists[level].emplace_back(int32_t(a - f), int32_t(b - f));
        } else if (level == s.q) {
            dense.emplace_back(int32_t(a - f), int32_t(b - f));
        } else {
            for (int i = 1; i <= 2; ++i)
                for (int j = 1; j <= 2; ++j) visit(2 * a + i, 2 * b + j, level + 1, stop, rest);
        }
    }
};

// The pairs of several traversals as block-sparse rows, columns ascending.
Bsr to_bsr(int64_t rows, const std::vector<const Pairs *> &parts) {
    Bsr m;
    m.rowptr.assign(rows + 1, 0);
    for (const Pairs *p : parts)
        for (const auto &x : *p) ++m.rowptr[x.first + 1];
    std::partial_sum(m.rowptr.begin(), m.rowptr.end(), m.rowptr.begin());
    m.colidx.resize(size_t(m.rowptr[rows]));
    std::vector<int32_t> at(m.rowptr.begin(), m.rowptr.end() - 1);
    for (const Pairs *p : parts)
        for (const auto &x : *p) m.colidx[size_t(at[x.first]++)] = x.second;
    for (int64_t r = 0; r < rows; ++r) std::sort(m.colidx.begin() + m.rowptr[r], m.colidx.begin() + m.rowptr[r + 1]);
    return m;
}

}  // namespace

std::string build_structure(const double *points, int64_t n, int dim, int leaf, int cheb_p,
                            double eta, double corr_len, Structure &s) {
    s = Structure();
    s.n = n;
    s.dim = dim;
    s.leaf = leaf;
    s.cheb_p = cheb_p;
    s.eta = eta;
    s.corr_len = corr_len;
    s.rank = 1;
    for (int a = 0; a < dim; ++a) s.rank *= cheb_p;
    while ((int64_t(leaf) << s.q) < n) ++s.q;
    if (s.q > 29) return "tree deeper than 29 levels";
    s.nnodes = (int64_t(2) << s.q) - 1;
    s.lrank.assign(s.q + 1, s.rank);
    s.perm.resize(n);
    std::iota(s.perm.begin(), s.perm.end(), int64_t(0));
    s.begin.assign(s.nnodes, 0);
    s.end.assign(s.nnodes, 0);
    s.end[0] = n;
    split_levels(points, dim, s);
    s.pts.resize(n * dim);
    for (int64_t i = 0; i < n; ++i)
        for (int a = 0; a < dim; ++a) s.pts[i * dim + a] = points[s.perm[i] * dim + a];
    compute_boxes(s);

    // the traversal to the level of 16 nodes here, the pairs below it spread
    // over the host threads (near pairs first to last: about equal work)
    const std::vector<double> diam = diameters(s);
    const int stop = n < 8192 ? s.q + 1 : std::min(s.q, 4);
    std::vector<Traversal> t;
    t.reserve(17);
    t.emplace_back(s, diam);
    Pairs rest;
    t[0].visit(0, 0, 0, stop, &rest);
    const int64_t parts = rest.empty() ? 0 : 16;
    for (int64_t i = 0; i < parts; ++i) t.emplace_back(s, diam);
    parallel_ranges(parts, 1, [&](int64_t p0, int64_t p1) {
        for (int64_t p = p0; p < p1; ++p)   // every 16th pair
            for (size_t i = size_t(p); i < rest.size(); i += 16)
                t[size_t(p) + 1].visit(rest[i].first, rest[i].second, stop, stop, nullptr);
    });
    s.coupling.resize(s.q + 1);
    auto lists = [&](int64_t l0, int64_t l1) {   // level q + 1: the dense blocks
        for (int64_t l = l0; l < l1; ++l) {
            std::vector<const Pairs *> of;
            for (const Traversal &x : t) of.push_back(l > s.q ? &x.dense : &x.lists[size_t(l)]);
            if (l > s.q) s.dense = to_bsr(int64_t(1) << s.q, of);
            else s.coupling[size_t(l)] = to_bsr(int64_t(1) << l, of);
        }
    };
    parallel_ranges(s.q + 2, n < 8192 ? s.q + 2 : 1, lists);
    s.lmin = s.q + 1;
    for (int l = s.q; l >= 0; --l)
        if (s.coupling[l].blocks() > 0) s.lmin = l;
    for (const Traversal &x : t) s.near_ties += x.near_ties;
    return std::string();
}

}  // namespace h2
