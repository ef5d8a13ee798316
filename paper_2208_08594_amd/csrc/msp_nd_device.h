// Device side of the nested-dissection coarsest-level solver: launchers (see
// msp_nd.h for the method and the plan).
#pragma once

#include <hip/hip_runtime.h>

#include "msp_nd.h"

namespace msp {

// Device pointers of a factorisation: copies of the plan's lists, the matrix
// in natural CSR order, lists built here, and the work and result arrays.
struct NdDev {
    const NdNode *node;
    const int *rows, *first;
    const int4 *prod, *inv;
    const int *rp, *ci;
    const double *val;
    const int *iperm;
    int *perm, *nodeof, *cmap;  // built: n, n, cmap_len
    int4 *yrow, *wrow;          // built: n each, see NdSolve
    // built, nnz each: the stored entries of a permuted row t = perm[i] towards
    // descendants of its node at ent[rp[i] ..): {permuted row, chain entries of
    // that row below t's node, CSR index of (i, .), CSR index of (., i)}; those
    // inside the node from the end of the row's slots backwards at self:
    // {column relative to the node, CSR index}; ecnt[t]: {how many of each}
    int4 *ent;
    int2 *self, *ecnt;
    double *W, *Yt;      // packed rows (wtot each)
    double *Y, *L, *Ut;  // qtot each
    double *X;           // xtot
    double *S0, *S1;     // stot each
    double *Dk;          // 2 tiles per node
};
// Computes W and Y (d.W and d.Y), queued on st.
hipError_t launch_nd_factor(const NdPlan &P, const NdDev &d, hipStream_t st);

// What the solve reads (kept with the preconditioner): the rows of Y by falling
// length, {row, first column, length, offset}, and per row of W {offset,
// entries, offset of their columns in cmap, 0}.
struct NdSolve {
    int n = 0, nlong = 0;
    const int4 *yrow = nullptr, *wrow = nullptr;
    const int *cmap = nullptr;
    const double *W = nullptr, *Y = nullptr;
};
// x = A^-1 f = W (Y f), vectors in permuted order (map != nullptr: entry r goes
// to x[map[r]]); t: FP64 work vector of n.
template <typename T>
hipError_t launch_nd_solve(const NdSolve &s, const T *f, double *t, T *x, const int *map,
                           hipStream_t st);

}  // namespace msp
