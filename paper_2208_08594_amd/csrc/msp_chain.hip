// Aggregation chain of the AMG setup on the device (Sec. 5 hierarchy, the
// pairwise rule of the host builder): strength and candidate lists per row,
// the pairwise pass with every row waiting for the decisions of lower rows that
// its own needs, the numbering of the aggregates in creation order and the Galerkin product per coarse row.  The
// results equal the host chain bit for bit; msp_chain.h gives the argument.
#include "msp_chain.h"

#include <cstring>

#include <algorithm>
#include <future>
#include <memory>
#include <vector>

#include "msp_match.h"

// every sum and comparison below is a single IEEE operation, as on the host
#pragma clang fp contract(off)

namespace msp {
namespace {

constexpr int kThreads = 256;
static_assert(kScanTile == 4 * kThreads, "four elements per thread of a scan tile");

inline unsigned nblocks(long long n, int per = kThreads)
{
    return (unsigned)std::max<long long>(1, (n + per - 1) / per);
}

__global__ void k_fill_i32(int *p, int v, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Row i of a structurally symmetric M: s_ij = -(m_ij + m_ji)/2 for every
// stored off-diagonal j (m_ji read through the mirror entry), the largest
// s_ij, and eligibility (a stored nonzero off-diagonal value, and a positive
// largest s_ij).  A missing mirror entry sets *asym.
__global__ void k_strength(int n, const int *__restrict__ rp, const int *__restrict__ ci,
                           const double *__restrict__ val, double *__restrict__ s,
                           double *__restrict__ smax, unsigned char *__restrict__ elig,
                           int *__restrict__ asym)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool coupled = false, any = false;
    double mx = 0.0;
    for (int k = rp[i]; k < rp[i + 1]; ++k) {
        const int j = ci[k];
        if (j == i) continue;
        const double aij = val[k];
        int lo = rp[j], hi = rp[j + 1];
        const int end = hi;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (ci[mid] < i)
                lo = mid + 1;
            else
                hi = mid;
        }
        double aji = 0.0;
        if (lo < end && ci[lo] == i)
            aji = val[lo];
        else
            atomicOr(asym, 1);
        if (aij != 0.0) coupled = true;
        const double sij = -(aij + aji) / 2.0;
        s[k] = sij;
        if (!any || sij > mx) mx = sij;
        any = true;
    }
    smax[i] = mx;
    elig[i] = (coupled && any && mx > 0.0) ? 1 : 0;
}

// The two lists of every row i that the matching reads, over the row's own
// slots: its candidates (eligible j > i with s_ij >= 0.25 max_k s_ik, ordered
// by s_ij descending then j ascending) at lst[rp[i] ..), then its in-rows
// (the lower rows j whose candidate it is: s is symmetric, so j < i in row i
// with s_ij >= 0.25 max_k s_jk; any order) behind them.  (Candidates j < i
// never matter: they are placed before i is visited.)  The first kRec entries
// of both lists are also held inline in two records, so that the matching
// loads a whole list at once; kOver in a record's first slot: the list is
// longer.  Unused slots are -1.  The row's state word is cleared.
__global__ void k_lists(int n, const int *__restrict__ rp, const int *__restrict__ ci,
                        const double *__restrict__ s, const double *__restrict__ smax,
                        const unsigned char *__restrict__ elig, int *__restrict__ lst,
                        double *__restrict__ cs, int *__restrict__ ncand, int *__restrict__ nin,
                        int4 *__restrict__ rin, int4 *__restrict__ rcand, int *__restrict__ word)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int m = 0, mi = 0;
    const int b0 = rp[i], b1 = rp[i + 1];
    if (elig[i]) {
        const double thr = 0.25 * smax[i];
        // candidates from the front, in-rows from the back of the row's slots
        for (int k = b0; k < b1; ++k) {
            const int j = ci[k];
            if (j == i || !elig[j]) continue;
            const double sj = s[k];
            if (j < i) {
                if (sj >= 0.25 * smax[j]) lst[b1 - ++mi] = j;
                continue;
            }
            if (!(sj >= thr)) continue;
            int r = m;
            while (r > 0 && (cs[b0 + r - 1] < sj || (cs[b0 + r - 1] == sj && lst[b0 + r - 1] > j))) {
                lst[b0 + r] = lst[b0 + r - 1];
                cs[b0 + r] = cs[b0 + r - 1];
                --r;
            }
            lst[b0 + r] = j;
            cs[b0 + r] = sj;
            ++m;
        }
    }
    int a[kRec] = {-1, -1, -1, -1}, c[kRec] = {-1, -1, -1, -1};
    if (mi > kRec)
        a[0] = kOver;
    else
#pragma unroll
        for (int q = 0; q < kRec; ++q)
            if (q < mi) a[q] = lst[b1 - 1 - q];
    if (m > kRec)
        c[0] = kOver;
    else
#pragma unroll
        for (int q = 0; q < kRec; ++q)
            if (q < m) c[q] = lst[b0 + q];
    rin[i] = make_int4(a[0], a[1], a[2], a[3]);
    rcand[i] = make_int4(c[0], c[1], c[2], c[3]);
    ncand[i] = m;
    nin[i] = mi;
    word[i] = kFree;
}

// The pairwise pass: every row decides for itself, in any order, what the
// ascending pass decides when it visits the row (MatchRow).  The words of the
// work-group's own rows are held in LDS, those of lower work-groups read with
// device-scope loads.  The vote keeps the wavefront's lanes together, so that
// none spins ahead of a lane it waits for.  A row gives up after `looks` looks
// that found an undecided row; rows still undecided then are counted in *left
// and the kernel is run again from their first entries.  Looks that go on along
// a list are not counted (lists end): the lowest undecided row finds every row
// that it asks about decided, so it decides in any run, however long its lists.
// (Work-groups start in order, so a second run is rare.)
// Work-groups of 256 or 512 rows are no faster (128x128x64 cells, all ten
// passes: 8.7 and 8.4 ms, 8.1 with 1024), several rows per thread are slower
// (a lane that starts on its next row stalls the others).
constexpr int kMatchThreads = 1024;
__global__ void __launch_bounds__(kMatchThreads)
k_match(int n, int looks, MatchLists<int4> L, int *word, int *__restrict__ partner,
        int *__restrict__ left)
{
    __shared__ int own[kMatchThreads];
    const int b0 = blockIdx.x * kMatchThreads, v = b0 + threadIdx.x;
    own[threadIdx.x] = v < n ? word[v] : kSingle;
    __syncthreads();
    bool open = own[threadIdx.x] == kFree;
    MatchRow<int4> R;
    if (open) R.start(L, v);
    const auto state = [&](int k) -> int {
        if (k < 0) return kSingle;
        const int o = k - b0;  // (no row above v is read)
        if (o >= 0)
            return __hip_atomic_load(&own[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return __hip_atomic_load(word + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int waited = 0; __any(open && waited < looks);) {
        if (!open || waited >= looks) continue;
        bool waits;
        const int dec = R.look(L, state, waits);
        waited += waits;
        if (dec != kFree) {
            if (dec == kHigh) partner[v] = R.by;
            __hip_atomic_store(&own[threadIdx.x], dec, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(word + v, dec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            open = false;
        }
    }
    const int cnt = __syncthreads_count(open);
    if (threadIdx.x == 0 && cnt) atomicAdd(left, cnt);
}

// ---- exclusive scan -----------------------------------------------------
__device__ inline int block_inclusive(int *sh, int t)
{
    sh[threadIdx.x] = t;
    __syncthreads();
    for (int d = 1; d < kThreads; d <<= 1) {
        const int x = threadIdx.x >= (unsigned)d ? sh[threadIdx.x - d] : 0;
        __syncthreads();
        sh[threadIdx.x] += x;
        __syncthreads();
    }
    return sh[threadIdx.x];
}

// Exclusive scan inside each tile of kScanTile elements, tile totals to
// tile_sum (which k_scan_sums turns into tile offsets): the scan of element i
// is out[i] + tile_sum[i / kScanTile].  LEAD: in holds state words, and a row
// counts one if it opens an aggregate (it is alone or has taken a row).
template <bool LEAD>
__global__ void __launch_bounds__(kThreads)
k_scan_tile(const int *__restrict__ in, int *__restrict__ out, int *__restrict__ tile_sum, int n)
{
    __shared__ int sh[kThreads];
    const long long base = (long long)blockIdx.x * kScanTile + threadIdx.x * 4;
    int v[4], t = 0;
    for (int q = 0; q < 4; ++q) {
        const long long i = base + q;
        v[q] = i < n ? (LEAD ? in[i] != kHigh : in[i]) : 0;
        t += v[q];
    }
    const int incl = block_inclusive(sh, t);
    int run = incl - t;
    for (int q = 0; q < 4; ++q) {
        const long long i = base + q;
        if (i < n) out[i] = run;
        run += v[q];
    }
    if (threadIdx.x == kThreads - 1) tile_sum[blockIdx.x] = incl;
}

__global__ void __launch_bounds__(kThreads)
k_scan_sums(int *__restrict__ tile_sum, int ntiles, int *__restrict__ total)
{
    __shared__ int sh[kThreads];
    __shared__ int carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int c0 = 0; c0 < ntiles; c0 += kThreads) {
        const int i = c0 + threadIdx.x;
        const int t = i < ntiles ? tile_sum[i] : 0;
        const int carry = carry_s;
        const int incl = block_inclusive(sh, t);
        if (i < ntiles) tile_sum[i] = carry + incl - t;
        __syncthreads();
        if (threadIdx.x == kThreads - 1) carry_s = carry + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry_s;
}

// Aggregate numbers in order of their lowest row (= creation order of the
// ascending visit) and the member rows of every aggregate; pos, tile: the
// scan of the rows that open one.
__global__ void k_number(int n, const int *__restrict__ word, const int *__restrict__ partner,
                         const int *__restrict__ pos, const int *__restrict__ tile,
                         int *__restrict__ agg, int *__restrict__ mem0, int *__restrict__ mem1)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int w = word[i];
    if (w == kHigh) {
        const int p = partner[i];
        agg[i] = pos[p] + tile[p / kScanTile];
        return;
    }
    const int I = pos[i] + tile[i / kScanTile];
    agg[i] = I;
    mem0[I] = i;
    mem1[I] = w < 0 ? ~w : -1;
}

// ---- Galerkin product for aggregates of one or two rows -----------------
// Coarse row I gathers the rows mem0[I] < mem1[I] in order, column by column;
// entry (I, agg(j)) is the first term, then plus each later term, in that
// order (the host's (fine row, fine column) order).  The running list,
// sorted by coarse column, lives in the member rows' own slots of wj/wv
// (position t < len0 in row mem0, the rest in row mem1).
__device__ inline int gal_slot(int t, int b0, int len0, int b1)
{
    return t < len0 ? b0 + t : b1 + (t - len0);
}

__global__ void k_gal_rows(int nc, const int *__restrict__ rp, const int *__restrict__ ci,
                           const double *__restrict__ val, const int *__restrict__ agg,
                           const int *__restrict__ mem0, const int *__restrict__ mem1,
                           int *__restrict__ wj, double *__restrict__ wv, int *__restrict__ cnt)
{
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    const int r0 = mem0[I], r1 = mem1[I];
    const int b0 = rp[r0], len0 = rp[r0 + 1] - b0;
    const int b1 = r1 >= 0 ? rp[r1] : 0;
    int m = 0;
    for (int w = 0; w < 2; ++w) {
        const int r = w == 0 ? r0 : r1;
        if (r < 0) break;
        for (int k = rp[r]; k < rp[r + 1]; ++k) {
            const int J = agg[ci[k]];
            const double v = val[k];
            int lo = 0, hi = m;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (wj[gal_slot(mid, b0, len0, b1)] < J)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            if (lo < m && wj[gal_slot(lo, b0, len0, b1)] == J) {
                const int q = gal_slot(lo, b0, len0, b1);
                wv[q] = wv[q] + v;
                continue;
            }
            for (int t = m; t > lo; --t) {
                const int d = gal_slot(t, b0, len0, b1), sidx = gal_slot(t - 1, b0, len0, b1);
                wj[d] = wj[sidx];
                wv[d] = wv[sidx];
            }
            const int q = gal_slot(lo, b0, len0, b1);
            wj[q] = J;
            wv[q] = v;
            ++m;
        }
    }
    cnt[I] = m;
}

// rpc[0..nc) holds the rows' offsets inside their scan tile on entry and the
// row pointers on return.
__global__ void k_gal_fill(int nc, const int *__restrict__ rp, const int *__restrict__ mem0,
                           const int *__restrict__ mem1, const int *__restrict__ wj,
                           const double *__restrict__ wv, const int *__restrict__ cnt,
                           const int *__restrict__ tile, int *__restrict__ rpc,
                           int *__restrict__ cic, double *__restrict__ valc)
{
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I >= nc) return;
    const int r0 = mem0[I], r1 = mem1[I];
    const int b0 = rp[r0], len0 = rp[r0 + 1] - b0;
    const int b1 = r1 >= 0 ? rp[r1] : 0;
    const int o = rpc[I] + tile[I / kScanTile], m = cnt[I];
    rpc[I] = o;
    for (int t = 0; t < m; ++t) {
        const int q = gal_slot(t, b0, len0, b1);
        cic[o + t] = wj[q];
        valc[o + t] = wv[q];
    }
}

__global__ void k_compose(int n, const int *__restrict__ a1, const int *__restrict__ a2,
                          int *__restrict__ agg)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) agg[i] = a2[a1[i]];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct DevLevel {
    int n = 0;
    int *rp = nullptr, *ci = nullptr;
    double *val = nullptr;
};

struct Chain {
    hipStream_t st = nullptr;
    HipFail hip_fail = nullptr;
    int *pinned = nullptr;
    int looks = kMatchLooks;
    hipEvent_t ev_lvl = nullptr;  // a new level is on the device
    // work arrays, sized for level 0 (no later matrix is larger)
    double *s = nullptr, *cs = nullptr, *smax = nullptr;
    int *lst = nullptr, *ncand = nullptr, *nin = nullptr, *partner = nullptr, *word = nullptr;
    int4 *rin = nullptr, *rcand = nullptr;  // per-row records of the two lists
    int *pos = nullptr, *cnt = nullptr, *tiles = nullptr, *ctr = nullptr;
    int *a1 = nullptr, *a2 = nullptr, *aggf = nullptr, *mem0 = nullptr, *mem1 = nullptr;
    unsigned char *elig = nullptr;
    DevLevel set[3];  // M1 and two alternating coarse levels

    void ck(hipError_t e) const
    {
        if (e != hipSuccess) {
            (void)hipGetLastError();
            hip_fail(e);
        }
    }
    void launched() const { ck(hipGetLastError()); }
    int read_int(const int *d, int slot)
    {
        ck(hipMemcpyAsync(pinned + slot, d, sizeof(int), hipMemcpyDeviceToHost, st));
        ck(hipStreamSynchronize(st));
        return pinned[slot];
    }
    void fill(int *p, int v, int n)
    {
        if (n <= 0) return;
        k_fill_i32<<<nblocks(n), kThreads, 0, st>>>(p, v, n);
        launched();
    }
    // tile-wise exclusive scan of in[0..n) (see k_scan_tile), the total to *total
    template <bool LEAD>
    void scan(const int *in, int *out, int *total, int n)
    {
        const int ntiles = (int)std::max<long long>(1, ((long long)n + kScanTile - 1) / kScanTile);
        k_scan_tile<LEAD><<<ntiles, kThreads, 0, st>>>(in, out, tiles, n);
        launched();
        k_scan_sums<<<1, kThreads, 0, st>>>(tiles, ntiles, total);
        launched();
    }
    void strength(const DevLevel &L)
    {
        k_strength<<<nblocks(L.n), kThreads, 0, st>>>(L.n, L.rp, L.ci, L.val, s, smax, elig,
                                                      ctr + 2);
        launched();
    }
    // One pairwise pass on L (strength already computed when have_s); agg
    // into `agg`, members into mem0/mem1; returns the aggregate count.
    int pass(const DevLevel &L, bool have_s, int *agg)
    {
        const int n = L.n;
        if (!have_s) strength(L);
        k_lists<<<nblocks(n), kThreads, 0, st>>>(n, L.rp, L.ci, s, smax, elig, lst, cs, ncand, nin,
                                                 rin, rcand, word);
        launched();
        // every run of the matching decides at least the lowest undecided row
        for (long long run = 0;; ++run) {
            if (run > (long long)n + 1) hip_fail(hipErrorUnknown);
            fill(ctr + 1, 0, 1);
            k_match<<<nblocks(n, kMatchThreads), kMatchThreads, 0, st>>>(
                n, looks, MatchLists<int4>{L.rp, lst, ncand, nin, rin, rcand}, word, partner,
                ctr + 1);
            launched();
            scan<true>(word, pos, ctr, n);
            k_number<<<nblocks(n), kThreads, 0, st>>>(n, word, partner, pos, tiles, agg, mem0, mem1);
            launched();
            ck(hipMemcpyAsync(pinned, ctr, 2 * sizeof(int), hipMemcpyDeviceToHost, st));
            ck(hipStreamSynchronize(st));
            if (pinned[1] == 0) return pinned[0];
        }
    }
    // C = P^T L P for the pass just numbered (aggregates of one or two rows),
    // queued without a wait (nnz(C) is C.rp[nc] on the device).  The list
    // arrays serve as the row lists.
    void galerkin(const DevLevel &L, const int *agg, int nc, DevLevel &C)
    {
        C.n = nc;
        k_gal_rows<<<nblocks(nc), kThreads, 0, st>>>(nc, L.rp, L.ci, L.val, agg, mem0, mem1, lst,
                                                     s, cnt);
        launched();
        scan<false>(cnt, C.rp, C.rp + nc, nc);
        k_gal_fill<<<nblocks(nc), kThreads, 0, st>>>(nc, L.rp, mem0, mem1, lst, s, cnt, tiles, C.rp,
                                                     C.ci, C.val);
        launched();
    }
    void to_device(const Csr &H, DevLevel &C)
    {
        C.n = H.n;
        ck(hipMemcpyAsync(C.rp, H.rp.data(), sizeof(int) * (H.n + 1), hipMemcpyHostToDevice, st));
        if (H.nnz()) {
            ck(hipMemcpyAsync(C.ci, H.ci.data(), sizeof(int) * H.nnz(), hipMemcpyHostToDevice, st));
            ck(hipMemcpyAsync(C.val, H.val.data(), sizeof(double) * H.nnz(),
                              hipMemcpyHostToDevice, st));
        }
        ck(hipStreamSynchronize(st));
    }
};

struct EventGuard {
    hipEvent_t *ev;
    ~EventGuard()
    {
        if (*ev) (void)hipEventDestroy(*ev);
    }
};

// Sets every work array of X to its offset in one allocation at `base`,
// each sized for level 0 (no later matrix is larger) and 256-byte aligned;
// with base == nullptr it only measures.  Returns the bytes used.
size_t place(Chain &X, char *base, int n0, long long nnz0)
{
    const long long n1 = (long long)n0 + 1, ntiles = n0 / kScanTile + 2;
    size_t off = 0;
    auto take = [&](long long count, size_t sz) -> void * {
        void *r = base ? (void *)(base + off) : nullptr;
        off += (((size_t)std::max<long long>(count, 1) * sz) + 255) & ~(size_t)255;
        return r;
    };
    X.s = (double *)take(nnz0, sizeof(double));
    X.cs = (double *)take(nnz0, sizeof(double));
    X.smax = (double *)take(n0, sizeof(double));
    X.lst = (int *)take(nnz0, sizeof(int));
    X.ncand = (int *)take(n0, sizeof(int));
    X.nin = (int *)take(n0, sizeof(int));
    X.word = (int *)take(n0, sizeof(int));
    X.partner = (int *)take(n0, sizeof(int));
    X.a1 = (int *)take(n0, sizeof(int));
    X.a2 = (int *)take(n0, sizeof(int));
    X.aggf = (int *)take(n0, sizeof(int));
    X.mem0 = (int *)take(n1, sizeof(int));
    X.mem1 = (int *)take(n1, sizeof(int));
    X.pos = (int *)take(n1, sizeof(int));
    X.cnt = (int *)take(n1, sizeof(int));
    X.tiles = (int *)take(ntiles, sizeof(int));
    X.ctr = (int *)take(4, sizeof(int));
    X.elig = (unsigned char *)take(n0, 1);
    X.rin = (int4 *)take(n0, sizeof(int4));
    X.rcand = (int4 *)take(n0, sizeof(int4));
    for (int k = 0; k < 3; ++k) {
        X.set[k].rp = (int *)take(n1, sizeof(int));
        X.set[k].ci = (int *)take(nnz0, sizeof(int));
        X.set[k].val = (double *)take(nnz0, sizeof(double));
    }
    return off;
}

}  // namespace

int scan_tiles(int n)
{
    return (int)std::max<long long>(1, ((long long)n + kScanTile - 1) / kScanTile);
}

hipError_t launch_tile_scan(const int *in, int *out, int *tiles, int *total, int n, hipStream_t st)
{
    k_scan_tile<false><<<scan_tiles(n), kThreads, 0, st>>>(in, out, tiles, n);
    k_scan_sums<<<1, kThreads, 0, st>>>(tiles, scan_tiles(n), total);
    return hipGetLastError();
}

size_t device_chain_bytes(int n0, long long nnz0)
{
    Chain X;
    return place(X, nullptr, n0, nnz0);
}

int device_hierarchy(Csr &A0, const int *rp0, const int *ci0, const double *val0,
                     int max_coarse, int max_levels, int max_dense, Hierarchy &H,
                     const LevelCallback &on_smoothed, const std::function<void()> &level0_values,
                     hipStream_t st, hipStream_t copy_st,
                     const DeviceAlloc &alloc, HipFail hip_fail, int *pinned,
                     const PinnedBuffer &staging, const int **last_rp, const int **last_ci,
                     const double **last_val, int looks)
{
    const auto report = [&](const int *rp, const int *ci, const double *val) {
        if (last_rp) *last_rp = rp;
        if (last_ci) *last_ci = ci;
        if (last_val) *last_val = val;
    };
    const int n0 = A0.n;
    const long long nnz0 = A0.nnz();
    if (n0 <= max_coarse || max_levels <= 1) {
        H = Hierarchy();
        H.A.push_back(std::move(A0));
        level0_values();  // level 0 is the coarsest: the caller inverts it next
        report(rp0, ci0, val0);
        return H.A.back().n > max_dense ? -9 : 0;
    }
    Chain X;
    X.st = st;
    X.hip_fail = hip_fail;
    X.pinned = pinned;
    X.looks = looks;
    EventGuard guard{&X.ev_lvl};
    X.ck(hipEventCreateWithFlags(&X.ev_lvl, hipEventDisableTiming));
    // one allocation for every work array
    char *base = (char *)alloc(place(X, nullptr, n0, nnz0));
    place(X, base, n0, nnz0);
    // level 0: strength first, which also tells whether the pattern is
    // structurally symmetric
    DevLevel cur;
    cur.n = n0;
    cur.rp = const_cast<int *>(rp0);
    cur.ci = const_cast<int *>(ci0);
    cur.val = const_cast<double *>(val0);
    X.fill(X.ctr + 2, 0, 1);
    X.strength(cur);
    if (X.read_int(X.ctr + 2, 0) != 0) return 1;

    H = Hierarchy();
    H.A.push_back(std::move(A0));
    // The host copy of each new level (and of the aggregation map that made
    // it) runs on a copy thread while the device goes on with the next level;
    // that thread also starts the level's host work (on_smoothed).  A level
    // is joined before its device buffers can be reused: the previous level's
    // copy before this level's aggregation map is composed (aggf is shared,
    // the level buffers alternate), and every copy before the host reads it.
    // `pending` ends when the copy thread is done; `copied` as soon as its
    // device reads are (with staging, the host copies out of the page-locked
    // buffer may still run: they write only through pointers taken before)
    std::future<void> pending, copied;
    const auto join = [&pending, &copied]() {
        if (copied.valid()) copied.get();
        if (pending.valid()) pending.get();
    };
    // (a failure of the copy thread before its device reads ended comes
    // through `copied`)
    const auto join_device = [&copied]() {
        if (copied.valid()) copied.get();
    };
    bool have_s = true;
    bool main_calls = true;  // level l's on_smoothed is due on this thread
    int next = 1;  // set[0] holds M1; levels alternate between set[1] and set[2]
    for (int l = 0;; ++l) {
        const int nl = H.A[l].n;
        const bool last = nl <= max_coarse || l == max_levels - 1 ||
                          (l > 0 && (double)nl > 0.9 * (double)H.A[l - 1].n);
        if (last) break;
        if (main_calls && on_smoothed) {
            if (l > 0) join();
            const Csr &hc = H.A[l];
            on_smoothed(l, hc.n, hc.rp.data(), hc.ci.data());
        }
        const int nc1 = X.pass(cur, have_s, X.a1);
        have_s = false;
        DevLevel &M1 = X.set[0];
        X.galerkin(cur, X.a1, nc1, M1);
        const int nc2 = X.pass(M1, false, X.a2);
        DevLevel &C = X.set[next];
        X.galerkin(M1, X.a2, nc2, C);
        join_device();
        k_compose<<<nblocks(cur.n), kThreads, 0, st>>>(cur.n, X.a1, X.a2, X.aggf);
        X.launched();
        X.ck(hipEventRecord(X.ev_lvl, st));
        {
            // sized (and cleared) by the copy thread, off this thread's path
            Csr Cn;
            Cn.n = nc2;
            H.agg.emplace_back();
            H.A.push_back(std::move(Cn));
        }
        const bool stalled = (double)nc2 > 0.9 * (double)cur.n;
        // level l+1 is smoothed unless it is the last one (a stalled level
        // may still change below, so its host work starts on this thread)
        const bool next_smoothed =
            !stalled && !(nc2 <= max_coarse || l + 1 == max_levels - 1);
        {
            Csr &hn = H.A[l + 1];
            std::vector<int> &hagg = H.agg[l];
            const int nf = cur.n;
            const DevLevel Cd = C;
            const int *aggf = X.aggf;
            const hipEvent_t ready = X.ev_lvl;
            const int lnext = l + 1;
            const bool call = next_smoothed && on_smoothed;
            const PinnedBuffer *stg = staging ? &staging : nullptr;
            auto dev_done = std::make_shared<std::promise<void>>();
            copied = dev_done->get_future();
            pending = std::async(std::launch::async, [&hn, &hagg, nf, Cd, aggf, ready, copy_st,
                                                      hip_fail, call, lnext, &on_smoothed, stg,
                                                      dev_done]() {
                bool signalled = false;
                try {
                    hn.rp.resize(Cd.n + 1);
                    auto ck = [hip_fail](hipError_t e) {
                        if (e != hipSuccess) {
                            (void)hipGetLastError();
                            hip_fail(e);
                        }
                    };
                    ck(hipStreamWaitEvent(copy_st, ready, 0));
                    ck(hipMemcpyAsync(hn.rp.data(), Cd.rp, sizeof(int) * (Cd.n + 1),
                                      hipMemcpyDeviceToHost, copy_st));
                    ck(hipStreamSynchronize(copy_st));
                    const long long nnzc = hn.rp[Cd.n];
                    // page-locked staging: [ci | val | agg], one DMA each
                    char *sb = stg ? (char *)(*stg)(lnext, sizeof(int) * (size_t)nnzc +
                                                               sizeof(double) * (size_t)nnzc +
                                                               sizeof(int) * (size_t)nf)
                                   : nullptr;
                    if (!sb) {
                        hagg.resize(nf);
                        hn.ci.resize(nnzc);
                        hn.val.resize(nnzc);
                    }
                    int *sci = sb ? (int *)sb : hn.ci.data();
                    double *sval =
                        sb ? (double *)(sb + sizeof(int) * (size_t)nnzc) : hn.val.data();
                    int *sagg = sb ? (int *)(sb + (sizeof(int) + sizeof(double)) * (size_t)nnzc)
                                   : hagg.data();
                    // the pattern first: the level's host work (its groups) needs
                    // only that, and starts while the rest is copied
                    if (nnzc)
                        ck(hipMemcpyAsync(sci, Cd.ci, sizeof(int) * nnzc, hipMemcpyDeviceToHost,
                                          copy_st));
                    ck(hipStreamSynchronize(copy_st));
                    if (call) on_smoothed(lnext, hn.n, hn.rp.data(), sci);
                    if (nnzc)
                        ck(hipMemcpyAsync(sval, Cd.val, sizeof(double) * nnzc,
                                          hipMemcpyDeviceToHost, copy_st));
                    ck(hipMemcpyAsync(sagg, aggf, sizeof(int) * nf, hipMemcpyDeviceToHost,
                                      copy_st));
                    // the host arrays are sized (their pages cleared) behind the
                    // copies, after the level's host work has started: 43 MB on
                    // 306,000 rows, 4 ms.  H grows on the main thread once the
                    // device reads are done: the destinations are taken here
                    // (moving a vector keeps its storage)
                    if (sb) {
                        hn.ci.resize(nnzc);
                        hn.val.resize(nnzc);
                        hagg.resize(nf);
                    }
                    int *dci = hn.ci.data(), *dagg = hagg.data();
                    double *dval = hn.val.data();
                    if (sb) std::memcpy(dci, sci, sizeof(int) * (size_t)nnzc);
                    ck(hipStreamSynchronize(copy_st));
                    signalled = true;
                    dev_done->set_value();
                    if (sb) {
                        std::memcpy(dval, sval, sizeof(double) * (size_t)nnzc);
                        std::memcpy(dagg, sagg, sizeof(int) * (size_t)nf);
                    }
                } catch (...) {
                    if (signalled) throw;
                    (void)hipStreamSynchronize(copy_st);
                    (void)hipGetLastError();
                    dev_done->set_exception(std::current_exception());
                }
            });
        }
        main_calls = !next_smoothed;
        if (stalled) {
            // stalled: absorb singletons, then one Galerkin product on A_l
            join();
            if (l == 0) level0_values();
            const int nc3 = absorb_singletons(H.A[l], H.agg[l], nc2);
            if (nc3 < nc2) {
                H.A[l + 1] = msp::galerkin(H.A[l], H.agg[l], nc3);
                X.to_device(H.A[l + 1], C);
            }
        }
        cur = C;
        next = 3 - next;
    }
    join();
    report(cur.rp, cur.ci, cur.val);
    return H.A.back().n > max_dense ? -9 : 0;
}

}  // namespace msp
