// Test-only C shim over the nested-dissection plan of the coarsest-level
// solver (msp_nd.cpp), so the CPU suite can carry the plan out without a GPU.
#include <algorithm>
#include <vector>

#include "msp_nd.h"

// The nested-dissection plan of a matrix, carried out step by step on the
// host (each stored index is range checked): x = W (Y f) in natural order.
// Returns 0, 1 if the plan declines the pattern, 2 if the matrix is not
// strictly dominant, -1 if an index of the plan is out of range; *entries
// receives the stored entries of W and Y.
extern "C" int shim_nd_solve(int n, const int *rp, const int *ci, const double *val,
                             const double *f, double *x, long long *entries)
{
    using namespace msp;
    if (!nd_dominant(n, rp, ci, val)) return 2;
    NdPlan P;
    if (!nd_plan(n, rp, ci, P)) return 1;
    *entries = (long long)(P.wtot + P.qtot);
    bool ok = true;
    // the lists that the device builds from the plan
    struct Ent {
        int row, prefix, src, srcT;
    };
    std::vector<int> nodeof(n, -1), cmap(P.cmap_len, -1), seen0(n, 0);
    std::vector<std::vector<Ent>> ent(n);
    std::vector<std::vector<std::pair<int, int>>> self(n);
    struct Row {
        int a, b, c, d;
    };
    std::vector<Row> yrow(n), wrow(n);
    for (int v = 0; v < (int)P.node.size(); ++v) {
        const NdNode &q = P.node[v];
        for (int r = 0; r < q.m; ++r) {
            nodeof[q.s + r] = v;
            ++seen0[q.yord + r];
            yrow[q.yord + r] = {q.s + r, q.f, q.s - q.f, (int)(q.qbase + (long long)r * q.qld)};
            wrow[q.s + r] = {(int)(q.wbase + (long long)r * q.c), q.c, q.cbase, 0};
        }
        int o = 0;
        for (int a = v; a >= 0; a = P.node[a].parent)
            for (int r = 0; r < P.node[a].m; ++r) cmap[q.cbase + o++] = P.node[a].s + r;
        if (o != q.len) ok = false;
        if (q.c > q.len) cmap[q.cbase + q.len] = q.s;
    }
    for (int t = 0; t < n; ++t) {
        if (seen0[t] != 1 || nodeof[t] < 0 || P.perm[P.iperm[t]] != t) ok = false;
        const int i = P.iperm[t];
        const NdNode &q = P.node[nodeof[t]];
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            const int r = P.perm[ci[k]];
            if (r >= q.s && r < q.s + q.m) self[t].push_back({r - q.s, k});
            const int mir = (int)(std::lower_bound(ci + rp[ci[k]], ci + rp[ci[k] + 1], i) - ci);
            if (r < q.s) {
                if (r < q.f) ok = false;  // joins two rows of unrelated nodes
                ent[t].push_back({r, P.node[nodeof[r]].len - q.len, k, mir});
            }
        }
    }
    auto at = [&ok](std::vector<double> &v, long long i) -> double & {
        static double sink;
        if (i < 0 || i >= (long long)v.size()) {
            ok = false;
            sink = 0.0;
            return sink;
        }
        return v[i];
    };
    const double nan = 0.0 / 0.0;  // an entry that is read before it is written shows
    std::vector<double> W(P.wtot, nan), Yt(P.wtot, nan), Y(P.qtot, nan), L(P.qtot), Ut(P.qtot),
        X(P.xtot, nan);
    for (int h = 0; h < P.heights; ++h) {
        for (int q = P.rows_ptr[h]; h > 0 && q < P.rows_ptr[h + 1]; ++q) {  // L(a, S), U(S, a)^T
            const int c = P.rows[q];
            const NdNode &a = P.node[nodeof[c]];
            const long long o = a.qbase + (long long)(c - a.s) * a.qld;
            for (const Ent &t : ent[c]) {
                const NdNode &v = P.node[nodeof[t.row]];
                const long long p = v.wbase + (long long)(t.row - v.s) * v.c;
                if (t.prefix > v.c) ok = false;
                for (int k = 0; k < t.prefix; ++k) {
                    const int col = cmap[v.cbase + k];
                    if (col < a.f || col >= a.s) ok = false;
                    at(L, o + col - a.f) += val[t.src] * at(W, p + k);
                    at(Ut, o + col - a.f) += val[t.srcT] * at(Yt, p + k);
                }
            }
        }
        for (int q = P.prod_ptr[h]; q < P.prod_ptr[h + 1]; ++q) {
            const NdPlan::Tile &t = P.prod[q];
            const NdNode &v = P.node[t.v], &a = P.node[t.a];
            const int i0 = t.ij >> 16, j0 = t.ij & 0xffff;
            for (int r = i0; r < std::min(i0 + kNdTile, v.m); ++r)
                for (int c = j0; c < std::min(j0 + kNdTile, a.m); ++c) {
                    const long long p = v.wbase + (long long)r * v.c;
                    const long long o = a.qbase + (long long)c * a.qld;
                    double s0 = 0.0, s1 = 0.0;
                    for (int k = 0; k < t.k; ++k) {
                        const int col = cmap[v.cbase + k] - a.f;
                        s0 += at(Yt, p + k) * at(L, o + col);
                        s1 += at(W, p + k) * at(Ut, o + col);
                    }
                    if (t.k + c >= v.c) ok = false;
                    at(Yt, p + t.k + c) = -s0;
                    at(Y, o + v.s + r - a.f) = -s0;
                    at(X, a.xbase + (long long)(v.s + r - a.f) * a.m + c) = s1;
                }
        }
        for (int q = P.first_ptr[h]; q < P.first_ptr[h + 1]; ++q) {
            const NdNode &a = P.node[P.first[q]];
            const int m = a.m;
            std::vector<double> S((size_t)m * m, 0.0);
            for (int r = 0; r < m; ++r) {
                const int c = a.s + r;
                for (const Ent &t : ent[c])
                    for (int j = 0; j < m; ++j)
                        S[r * m + j] -=
                            val[t.src] * at(X, a.xbase + (long long)(t.row - a.f) * m + j);
                for (const auto &t : self[c]) at(S, (long long)r * m + t.first) += val[t.second];
            }
            for (int k = 0; k < m; ++k) {  // Gauss-Jordan without interchanges
                const double d = 1.0 / S[k * m + k];
                for (int i = 0; i < m; ++i) {
                    if (i == k) continue;
                    const double g = S[i * m + k] * d;
                    for (int j = 0; j < m; ++j) S[i * m + j] -= j == k ? 0.0 : g * S[k * m + j];
                    S[i * m + k] = -g;
                }
                for (int j = 0; j < m; ++j) S[k * m + j] *= d;
                S[k * m + k] = d;
            }
            for (int r = 0; r < m; ++r)
                for (int j = 0; j < a.c; ++j) {
                    const long long o = a.wbase + (long long)r * a.c + j;
                    if (j < m) {
                        at(W, o) = S[r * m + j];
                        at(Yt, o) = r == j ? 1.0 : 0.0;
                    } else if (j + 1 == a.c) {
                        at(W, o) = 0.0;  // padding (or overwritten by an ancestor)
                    }
                }
            for (int v = 0; v < P.first[q]; ++v) {
                const NdNode &b = P.node[v];
                if (b.s < a.f) continue;
                int k0 = -1;
                for (int k = 0; k < b.c && k0 < 0; ++k)
                    if (cmap[b.cbase + k] == a.s) k0 = k;
                if (k0 < 0) ok = false;
                for (int r = 0; ok && r < b.m; ++r)
                    for (int j = 0; j < m; ++j) {
                        double s = 0.0;
                        for (int k = 0; k < m; ++k)
                            s += at(X, a.xbase + (long long)(b.s + r - a.f) * m + k) * S[k * m + j];
                        at(W, b.wbase + (long long)r * b.c + k0 + j) = -s;
                    }
            }
        }
    }
    std::vector<double> t(n), xp(n), fp(n);
    for (int i = 0; i < n; ++i) fp[P.perm[i]] = f[i];
    std::vector<int> seen(n, 0);
    for (const Row &r : yrow) {
        double s = fp[r.a];
        for (int j = 0; j < r.c; ++j) s += at(Y, (long long)r.d + j) * fp[r.b + j];
        t[r.a] = s;
        ++seen[r.a];
    }
    for (int i = 0; i < n; ++i) {
        const Row &r = wrow[i];
        double s = 0.0;
        for (int j = 0; j < r.b; ++j) s += at(W, (long long)r.a + j) * t[cmap[r.c + j]];
        xp[i] = s;
        if (seen[i] != 1) ok = false;
    }
    for (int i = 0; i < n; ++i) x[i] = xp[P.perm[i]];
    return ok ? 0 : -1;
}
