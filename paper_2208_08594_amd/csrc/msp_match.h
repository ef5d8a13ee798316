// One row's part in the pairwise pass of the device aggregation chain: the
// walk over the state words of lower rows that its decision needs.  Plain code
// for the matching kernel and for the CPU tests.
//
// Row v
//  - is taken (kHigh) if some in-row has taken it;
//  - otherwise, once all its in-rows are decided, takes the first candidate
//    that no lower row has taken: a candidate j is known to be taken when one
//    of j's in-rows below v has taken it, and known to be free when all of
//    them are decided and none has; while neither is known, v waits;
//  - stays alone when every candidate is taken.
// A decision reads only state words of lower rows, each written once, so
// stale reads only delay it and the result does not depend on the schedule.
#pragma once

// (a row is held in registers: nothing below may take its members' addresses)
#ifdef __HIPCC__
#define MSP_BOTH __host__ __device__ inline __attribute__((always_inline))
#else
#define MSP_BOTH inline
#endif

namespace msp {

// state word of a row in the matching: undecided, alone, taken by a lower
// row, or ~j: it has taken row j
constexpr int kFree = 0, kSingle = 1, kHigh = 2;

// The lists of every row i: its candidates at lst[rp[i] ..), its in-rows from
// the back of the row's slots; the first kRec of both also inline in records
// (unused entries -1; kOver in the first: the list is longer).
constexpr int kRec = 4;
constexpr int kOver = -2;
template <class Rec>  // four ints x, y, z, w
struct MatchLists {
    const int *rp, *lst, *ncand, *nin;
    const Rec *rin, *rcand;
};

template <class Rec>
struct MatchRow {
    int v;
    // what v waits for: the in-rows below v of `target` (v itself, then its
    // candidates in order), up to four entries at a time
    int target, pos, cq, nc;
    int by;  // the row that has taken v
    Rec a, cand, rec0;

    MSP_BOTH void start(const MatchLists<Rec> &L, int row)
    {
        v = target = row;
        cq = -1;
        by = -1;
        cand = L.rcand[v];
        nc = L.ncand[v];
        rec0 = L.rin[v];
        begin(L, rec0);
        if (cand.x >= 0) rec0 = L.rin[cand.x];  // (read ahead)
    }
    // One look at the entries that are left.  Returns the row's decision, or
    // kFree while it has none; `waits` then tells whether some entry is
    // undecided (otherwise the next look goes on from here).
    template <class State>  // state word of a row, kSingle for -1
    MSP_BOTH int look(const MatchLists<Rec> &L, const State &state, bool &waits)
    {
        const int w0 = state(a.x), w1 = state(a.y), w2 = state(a.z), w3 = state(a.w);
        int taker = -1;  // the row that has taken the target
        if (w0 == ~target) taker = a.x;
        if (w1 == ~target) taker = a.y;
        if (w2 == ~target) taker = a.z;
        if (w3 == ~target) taker = a.w;
        if (w0 != kFree) a.x = -1;
        if (w1 != kFree) a.y = -1;
        if (w2 != kFree) a.z = -1;
        if (w3 != kFree) a.w = -1;
        waits = false;
        if (taker < 0) {
            waits = left();
            if (waits) return kFree;
            if (pos >= 0) {
                next(L);
                if (left()) return kFree;
            }
        }
        if (cq < 0 && taker >= 0) {
            by = taker;
            return kHigh;
        }
        if (cq >= 0 && taker < 0) return ~target;  // no lower row took this candidate
        if (++cq == nc) return kSingle;
        target = cand.x == kOver ? L.lst[L.rp[v] + cq]
                 : cq == 0       ? cand.x
                 : cq == 1       ? cand.y
                 : cq == 2       ? cand.z
                                 : cand.w;
        if (!(cq == 0 && cand.x != kOver)) rec0 = L.rin[target];
        begin(L, rec0);
        return kFree;
    }

private:
    MSP_BOTH bool left() const { return (a.x & a.y & a.z & a.w) != -1; }
    // the next entries, from number pos on, of a list longer than a record
    MSP_BOTH void next(const MatchLists<Rec> &L)
    {
        int r[kRec] = {-1, -1, -1, -1};
        const int e = L.rp[target + 1], m = L.nin[target];
#pragma unroll
        for (int u = 0; u < kRec; ++u)
            while (pos < m && r[u] < 0) {
                const int k = L.lst[e - 1 - pos++];
                if (k < v) r[u] = k;
            }
        a.x = r[0];
        a.y = r[1];
        a.z = r[2];
        a.w = r[3];
    }
    MSP_BOTH void begin(const MatchLists<Rec> &L, const Rec rec)
    {
        pos = -1;
        a = rec;
        if (rec.x == kOver) {
            pos = 0;
            next(L);
        } else {
            if (a.x >= v) a.x = -1;
            if (a.y >= v) a.y = -1;
            if (a.z >= v) a.z = -1;
            if (a.w >= v) a.w = -1;
        }
    }
};

}  // namespace msp
