// Host part of the nested-dissection coarsest-level solver (see msp_nd.h).
#include "msp_nd.h"

#include <algorithm>
#include <cmath>
#include <future>
#include <memory>
#include <numeric>

#include "msp_host.h"

namespace msp {

namespace {

struct Tree {
    std::vector<int> rows;             // the node's vertices
    std::vector<std::unique_ptr<Tree>> sub;
};
using Forest = std::vector<std::unique_ptr<Tree>>;

constexpr int kSep = -1;          // mark of a separator vertex (never part of a set again)
constexpr int kParallelSet = 700;  // halves of at least this many vertices get a thread

struct Cutter {
    const int *rp, *ci;
    std::vector<int> mark;  // label of the set a vertex belongs to

    // Breadth-first levels of the vertices labelled `from` that start
    // reaches, relabelled `to`; order gets them level after level.
    void bfs(int start, int from, int to, std::vector<int> &order, std::vector<int> &lptr)
    {
        order.clear();
        lptr.assign(1, 0);
        order.push_back(start);
        mark[start] = to;
        for (size_t lo = 0; lo < order.size();) {
            const size_t hi = order.size();
            lptr.push_back((int)hi);
            for (; lo < hi; ++lo) {
                const int u = order[lo];
                for (int k = rp[u]; k < rp[u + 1]; ++k) {
                    const int w = ci[k];
                    if (mark[w] == from) {
                        mark[w] = to;
                        order.push_back(w);
                    }
                }
            }
        }
    }

    // Trees of the set `v` (vertices labelled `lab`, adjacent only to one
    // another and to separators).  Labels lab + 1, lab + 2 are free to use.
    Forest cut(std::vector<int> v, int lab)
    {
        Forest out;
        auto leaf = [&](std::vector<int> r) {
            for (int u : r) mark[u] = kSep;
            std::sort(r.begin(), r.end());
            std::unique_ptr<Tree> t(new Tree);
            t->rows = std::move(r);
            out.push_back(std::move(t));
        };
        if (v.empty()) return out;
        if ((int)v.size() <= kNdLeaf) {
            leaf(std::move(v));
            return out;
        }
        std::vector<int> order, lptr;
        bfs(*std::min_element(v.begin(), v.end()), lab, lab + 1, order, lptr);
        if (order.size() < v.size()) {
            // several components: the large ones on their own, the small ones
            // collected into leaves
            std::vector<int> bin;
            auto take = [&](std::vector<int> &comp) {
                if ((int)comp.size() > kNdLeaf) {
                    for (int u : comp) mark[u] = lab + 2;
                    for (auto &t : cut(comp, lab + 2)) out.push_back(std::move(t));
                    return;
                }
                if (bin.size() + comp.size() > (size_t)kNdLeaf) {
                    leaf(std::move(bin));
                    bin.clear();
                }
                bin.insert(bin.end(), comp.begin(), comp.end());
            };
            take(order);
            for (int u : v)
                if (mark[u] == lab) {
                    bfs(u, lab, lab + 1, order, lptr);
                    take(order);
                }
            if (!bin.empty()) leaf(std::move(bin));
            return out;
        }
        // the smallest level that leaves neither side more than 0.65 of the
        // set separates it.  (The lowest vertex of a set cut out of a mesh in
        // its natural order lies at its rim; starting from the farthest
        // vertex instead gives 3% fewer entries for twice the time.)
        const int n = (int)order.size(), nl = (int)lptr.size() - 1;
        int best = -1;
        for (int q = 1; q + 1 < nl; ++q) {
            const int lo = lptr[q], hi = n - lptr[q + 1], sz = lptr[q + 1] - lptr[q];
            if (std::max(lo, hi) > 0.65 * n) continue;
            if (best < 0 || sz < lptr[best + 1] - lptr[best]) best = q;
        }
        if (best < 0) {
            // no such level: the one that splits most evenly, if there is one
            int bal = n;
            for (int q = 1; q + 1 < nl; ++q) {
                const int m = std::max(lptr[q], n - lptr[q + 1]);
                if (m < bal && m < 0.9 * n) {
                    bal = m;
                    best = q;
                }
            }
        }
        if (best < 0) {
            leaf(std::move(order));
            return out;
        }
        // the level's vertices that touch only one side join it
        std::vector<int> L(order.begin(), order.begin() + lptr[best]);
        std::vector<int> R(order.begin() + lptr[best + 1], order.end());
        std::vector<int> S;
        for (int u : L) mark[u] = lab + 3;
        for (int u : R) mark[u] = lab + 4;
        for (int q = lptr[best]; q < lptr[best + 1]; ++q) {
            const int u = order[q];
            bool r = false;
            for (int k = rp[u]; k < rp[u + 1] && !r; ++k) r = mark[ci[k]] == lab + 4;
            if (r) {
                S.push_back(u);
            } else {
                mark[u] = lab + 3;
                L.push_back(u);
            }
        }
        {
            std::vector<int> T;
            for (int u : S) {
                bool l = false;
                for (int k = rp[u]; k < rp[u + 1] && !l; ++k) l = mark[ci[k]] == lab + 3;
                if (l) {
                    T.push_back(u);
                } else {
                    mark[u] = lab + 4;
                    R.push_back(u);
                }
            }
            S.swap(T);
        }
        for (int u : S) mark[u] = kSep;
        std::sort(S.begin(), S.end());
        Forest fl, fr;
        if ((int)std::min(L.size(), R.size()) >= kParallelSet) {
            // no vertex of one side is adjacent to the other side, so the two
            // touch disjoint marks.  (Deferred where no thread can be had: it then
            // runs in the get below.)
            auto job = std::async(std::launch::async | std::launch::deferred,
                                  [&]() { return cut(std::move(L), lab + 3); });
            fr = cut(std::move(R), lab + 4);
            fl = job.get();
        } else {
            fl = cut(std::move(L), lab + 3);
            fr = cut(std::move(R), lab + 4);
        }
        if (S.empty()) {
            for (auto &t : fl) out.push_back(std::move(t));
            for (auto &t : fr) out.push_back(std::move(t));
            return out;
        }
        std::unique_ptr<Tree> t(new Tree);
        t->rows = std::move(S);
        for (auto &x : fl) t->sub.push_back(std::move(x));
        for (auto &x : fr) t->sub.push_back(std::move(x));
        out.push_back(std::move(t));
        return out;
    }
};

// Postorder numbering of a tree; returns its node index.
int place(const Tree &t, NdPlan &P, std::vector<int> &height)
{
    const int f = (int)P.iperm.size();
    std::vector<int> kids;
    int h = 0;
    for (const auto &x : t.sub) {
        kids.push_back(place(*x, P, height));
        h = std::max(h, height[kids.back()] + 1);
    }
    NdNode q{};
    q.f = f;
    q.s = (int)P.iperm.size();
    q.m = (int)t.rows.size();
    q.parent = -1;
    P.iperm.insert(P.iperm.end(), t.rows.begin(), t.rows.end());
    const int me = (int)P.node.size();
    P.node.push_back(q);
    height.push_back(h);
    for (int k : kids) P.node[k].parent = me;
    return me;
}

}  // namespace

void NdPlan::clear()
{
    n = heights = nlong = cmap_len = 0;
    wtot = qtot = xtot = stot = 0;
    for (std::vector<int> *v :
         {&perm, &iperm, &rows, &rows_ptr, &prod_ptr, &inv_ptr, &first, &first_ptr})
        v->clear();
    node.clear();
    prod.clear();
    inv.clear();
    inv_n.clear();
}

bool nd_dominant(int n, const int *rp, const int *ci, const double *val)
{
    for (int i = 0; i < n; ++i) {
        double d = 0.0, s = 0.0;
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            if (ci[k] == i)
                d = std::fabs(val[k]);
            else
                s += std::fabs(val[k]);
        }
        if (!(d * (1.0 - kNdMargin) > s) || !std::isfinite(d)) return false;
    }
    return true;
}

bool nd_plan(int n, const int *rp, const int *ci, NdPlan &P, bool known_symmetric)
{
    P.clear();
    P.n = n;
    if (n < 1 || n > 32767) return false;
    // with sorted rows, the lower entries of row j come up in order as the rows
    // above it are walked: a pattern that is not symmetric, or lacks a
    // diagonal, declines
    if (!known_symmetric) {
        std::vector<int> cur(rp, rp + n);
        for (int i = 0; i < n; ++i) {
            int k = cur[i];
            if (k >= rp[i + 1] || ci[k] != i) return false;  // its lower entries all matched
            for (++k; k < rp[i + 1]; ++k) {
                const int j = ci[k], m = cur[j]++;
                if (m >= rp[j + 1] || ci[m] != i) return false;
            }
        }
    }
    Cutter C{rp, ci, std::vector<int>(n, 0)};
    std::vector<int> all(n), height;
    std::iota(all.begin(), all.end(), 0);
    Forest forest = C.cut(std::move(all), 0);
    P.iperm.reserve(n);
    for (const auto &t : forest) place(*t, P, height);
    P.perm.resize(n);
    for (int t = 0; t < n; ++t) P.perm[P.iperm[t]] = t;
    const int nn = (int)P.node.size();
    for (int v = 0; v < nn; ++v) {
        NdNode &q = P.node[v];
        if (q.m > kNdMaxNode) return false;
        P.heights = std::max(P.heights, height[v] + 1);
    }
    // chains and offsets (ancestors first: they come later in postorder)
    for (int v = nn - 1; v >= 0; --v) {
        NdNode &q = P.node[v];
        q.len = q.m + (q.parent < 0 ? 0 : P.node[q.parent].len);
        q.c = (q.len + 1) & ~1;
        q.cbase = P.cmap_len;
        P.cmap_len += q.c;
    }
    for (int v = 0; v < nn; ++v) {
        NdNode &q = P.node[v];
        q.qld = (q.s - q.f + 1) & ~1;
        q.mp = (q.m + kNdTile - 1) / kNdTile * kNdTile;
        q.wbase = (long long)P.wtot;
        q.qbase = (long long)P.qtot;
        q.xbase = (long long)P.xtot;
        q.sbase = (long long)P.stot;
        P.wtot += (size_t)q.m * q.c;
        P.qtot += (size_t)q.m * q.qld;
        P.xtot += (size_t)(q.s - q.f) * q.m;
        P.stot += (size_t)q.mp * q.mp;
    }
    // worth it: no more device memory than the two dense triangles of the
    // natural order (W and Y, each n^2 there), and offsets fit 31 bits
    const size_t need = 2 * P.wtot + 3 * P.qtot + P.xtot + 2 * P.stot;
    if (need > 2 * (size_t)n * n + ((size_t)1 << 16)) return false;
    if (P.wtot >= ((size_t)1 << 31) || P.qtot >= ((size_t)1 << 31)) return false;
    // tasks by height
    std::vector<std::vector<int>> at(P.heights);
    for (int v = 0; v < nn; ++v) at[height[v]].push_back(v);
    P.rows_ptr.assign(1, 0);
    P.prod_ptr.assign(1, 0);
    P.inv_ptr.assign(1, 0);
    P.first_ptr.assign(1, 0);
    P.inv_n.resize(P.heights);
    // the descendants of a: the nodes from its subtree's first one up to a
    std::vector<int> firstnode(nn);
    for (int v = 0; v < nn; ++v) firstnode[v] = v;
    for (int v = 0; v < nn; ++v)
        if (P.node[v].parent >= 0)
            firstnode[P.node[v].parent] = std::min(firstnode[P.node[v].parent], firstnode[v]);
    for (int h = 0; h < P.heights; ++h) {
        std::vector<int> &g = at[h];
        std::stable_sort(g.begin(), g.end(),
                         [&](int x, int y) { return P.node[x].mp > P.node[y].mp; });
        for (int a : g) {
            const NdNode &q = P.node[a];
            P.first.push_back(a);
            for (int r = 0; r < q.m; ++r) P.rows.push_back(q.s + r);
            for (int v = firstnode[a]; v < a; ++v)
                for (int i = 0; i < P.node[v].m; i += kNdTile)
                    for (int j = 0; j < q.m; j += kNdTile)
                        P.prod.push_back({v, a, i << 16 | j, P.node[v].len - q.len});
            for (int i = 0; i < q.mp; i += kNdTile)
                for (int j = 0; j < q.mp; j += kNdTile) P.inv.push_back({a, a, i << 16 | j, 0});
        }
        for (int step = 0; !g.empty() && step * kNdTile < P.node[g[0]].mp; ++step) {
            int cnt = 0;
            for (int a : g) {
                const int nb = P.node[a].mp / kNdTile;
                if (nb > step) cnt += nb * nb;
            }
            P.inv_n[h].push_back(cnt);
        }
        P.rows_ptr.push_back((int)P.rows.size());
        P.prod_ptr.push_back((int)P.prod.size());
        P.inv_ptr.push_back((int)P.inv.size());
        P.first_ptr.push_back((int)P.first.size());
    }
    // the solve's order: rows by falling length of their part of Y
    std::vector<int> byl(nn);
    std::iota(byl.begin(), byl.end(), 0);
    std::stable_sort(byl.begin(), byl.end(), [&](int x, int y) {
        return P.node[x].s - P.node[x].f > P.node[y].s - P.node[y].f;
    });
    int o = 0;
    for (int v : byl) {
        NdNode &q = P.node[v];
        q.yord = o;
        o += q.m;
        if (q.s - q.f >= kNdLongRow) P.nlong = o;
    }
    return true;
}

}  // namespace msp
