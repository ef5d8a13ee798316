// Test-only C shim over one row's part of the device matching (msp_match.h), so
// the CPU suite can run the pass under any schedule and limit without a GPU.
#include <algorithm>
#include <vector>

#include "msp_host.h"
#include "msp_match.h"

namespace {
struct Four {
    int x, y, z, w;
};
double entry(const int *rp, const int *ci, const double *val, int i, int j)
{
    for (int k = rp[i]; k < rp[i + 1]; ++k)
        if (ci[k] == j) return val[k];
    return 0.0;
}
}  // namespace

// The pairwise pass of a structurally symmetric matrix in runs of at most
// `looks` counted looks a row, the rows of a run taking turns in ascending (up)
// or descending order; agg: aggregates numbered by their lowest row.  Returns
// the number of runs, or -1 when a run decides nothing.
extern "C" int shim_match(int n, const int *rp, const int *ci, const double *val, int looks,
                          int up, int *agg)
{
    using namespace msp;
    std::vector<double> smax(n, 0.0);
    std::vector<char> elig(n, 0);
    auto strength = [&](int i, int k) {
        return -(val[k] + entry(rp, ci, val, ci[k], i)) / 2.0;
    };
    for (int i = 0; i < n; ++i) {
        bool any = false, coupled = false;
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            if (ci[k] == i) continue;
            const double s = strength(i, k);
            coupled = coupled || val[k] != 0.0;
            if (!any || s > smax[i]) smax[i] = s;
            any = true;
        }
        elig[i] = coupled && smax[i] > 0.0;
    }
    std::vector<int> lst(rp[n]), ncand(n, 0), nin(n, 0), word(n, kFree), partner(n, -1);
    std::vector<Four> rin(n), rcand(n);
    for (int i = 0; i < n; ++i) {
        std::vector<std::pair<double, int>> cand;
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            const int j = ci[k];
            if (j == i || !elig[i] || !elig[j]) continue;
            const double s = strength(i, k);
            if (j < i && s >= 0.25 * smax[j]) lst[rp[i + 1] - ++nin[i]] = j;
            if (j > i && s >= 0.25 * smax[i]) cand.push_back({-s, j});
        }
        std::sort(cand.begin(), cand.end());
        for (auto &c : cand) lst[rp[i] + ncand[i]++] = c.second;
        auto record = [](int m, auto at) {
            if (m > kRec) return Four{kOver, -1, -1, -1};
            return Four{m > 0 ? at(0) : -1, m > 1 ? at(1) : -1, m > 2 ? at(2) : -1,
                        m > 3 ? at(3) : -1};
        };
        rin[i] = record(nin[i], [&](int q) { return lst[rp[i + 1] - 1 - q]; });
        rcand[i] = record(ncand[i], [&](int q) { return lst[rp[i] + q]; });
    }
    const MatchLists<Four> L{rp, lst.data(), ncand.data(), nin.data(), rin.data(), rcand.data()};
    const auto state = [&](int k) { return k < 0 ? kSingle : word[k]; };
    int runs = 0;
    for (int left = n; left > 0;) {
        ++runs;
        const int before = left;
        std::vector<int> open;
        for (int i = 0; i < n; ++i)
            if (word[up ? i : n - 1 - i] == kFree) open.push_back(up ? i : n - 1 - i);
        std::vector<MatchRow<Four>> R(n);
        std::vector<int> waited(n, 0);
        for (int v : open) R[v].start(L, v);
        for (bool busy = true; busy;) {
            busy = false;
            for (int v : open) {
                if (word[v] != kFree || waited[v] >= looks) continue;
                busy = true;
                bool waits;
                const int dec = R[v].look(L, state, waits);
                waited[v] += waits;
                if (dec == kFree) continue;
                if (dec == kHigh) partner[v] = R[v].by;
                word[v] = dec;
                --left;
            }
        }
        if (left == before) return -1;
    }
    int na = 0;
    for (int i = 0; i < n; ++i) agg[i] = word[i] == kHigh ? agg[partner[i]] : na++;
    return runs;
}

// The host chain's pass.
extern "C" int shim_pairwise(int n, const int *rp, const int *ci, const double *val, int *agg)
{
    msp::Csr A;
    A.n = n;
    A.rp.assign(rp, rp + n + 1);
    A.ci.assign(ci, ci + rp[n]);
    A.val.assign(val, val + rp[n]);
    std::vector<int> g;
    const int na = msp::pairwise_pass(A, g);
    std::copy(g.begin(), g.end(), agg);
    return na;
}
