// Nested-dissection direct solve of the coarsest AMG level.
//
// The coarsest matrix A (structurally symmetric, every row strictly
// diagonally dominant) is permuted so that its unknowns form a tree of nodes
// (leaves, and separators above the parts they separate): an entry of A joins
// two rows only if one's node is an ancestor of the other's, or they share a
// node.  With A = L U at node granularity (L unit block lower triangular, U
// with the Schur complements on its diagonal), the inverse factors Y = L^-1
// and W = U^-1 then have entries only between a row and its node's
// descendants (Y) or ancestors (W), and
//   x = W (Y f)
// is two products with all rows in parallel that read a fraction of the n^2
// values of the natural order.  A strictly diagonally dominant matrix has
// bounded element growth without interchanges in every symmetric order, so
// nothing is pivoted here; other matrices keep the natural-order block LU
// with pivoting inside its blocks (dense_inverse).
//
// Why: the natural order's solver is bound by a chain of n / 128 pivot blocks
// (about 170 us each), its solve by reading n^2 values.  Here the chain is one
// launch per 64-row block step of the largest node of each height, and W and
// Y hold 0.16 to 0.22 n^2 values.  Measured on 64x64x32 cells, b = 4 (9,713
// coarsest rows: 76 pivot blocks and 755 MB before; 33 block steps and 160 MB
// now): setup 19.8 -> 10.9 ms, FGMRES solve 4.5 -> 3.2 ms; eight 20^3 systems
// (8,000 coarsest rows each) solved together 44.9 -> 8.4 ms (the natural
// order's compute-unit masked streams, one hardware queue each, are no longer
// created).  Only the tree and the task lists are made on the host: the lists
// per row and per entry (2.5 MB there) follow from them on the device, and the
// matrix is taken where the aggregation chain left it.  With that, gathered
// rows and a shorter pivot chain the Newton step on these cells went from 12.0
// to 10.7 ms, and on 24x24x24 cells, b = 5 (3,662 coarsest rows) from 4.4 to
// 3.9 ms.
#pragma once

#include <cstddef>
#include <vector>

namespace msp {

constexpr int kNdLeaf = 128;     // parts of at most this many rows are not cut further
constexpr int kNdMaxNode = 1024; // larger nodes: the graph does not separate
constexpr int kNdTile = 64;      // tile of the node products and of the node inverses
// a row is taken as strictly dominant if |a_ii| (1 - kNdMargin) > sum |a_ij|
constexpr double kNdMargin = 1e-5;

// Node of the tree as the kernels see it.  Rows [s, s + m) in permuted order;
// its descendants are the rows [f, s).  chain = the node's own rows and all
// its ancestors' rows, lowest first (len of them; c: len rounded up to even);
// a row of W (and of Y^T while Y is computed) is stored as its c chain entries
// at wbase + (row - s) c, their columns at cmap + cbase.  Chain entries of the
// node below its ancestor a: len - a.len.
struct NdNode {
    int s, m, f, c;
    int len, cbase, qld, mp;  // qld: s - f rounded up to even; mp: m rounded up to tiles
    int parent, yord;         // yord: place of the node's rows among the rows by length of Y
    long long wbase;          // packed rows of W and of Y^T
    long long qbase;          // m x qld: the node's rows of Y (and of L and U^T)
    long long xbase;          // (s - f) x m: A_SS^-1 A(S, node), S the descendants
    long long sbase;          // mp x mp: the node's Schur complement / its inverse
};

// What depends on the pattern only (device arrays are copies of these): order,
// tree and the task lists of each height.
struct NdPlan {
    int n = 0, heights = 0;
    std::vector<int> perm, iperm;  // natural -> permuted, permuted -> natural
    std::vector<NdNode> node;      // postorder: descendants before their ancestors
    // task lists; height h takes [ptr[h], ptr[h+1])
    struct Tile {
        int v, a, ij, k;  // nodes, tile origin (i << 16 | j), chain entries of v below a
    };
    std::vector<int> rows, rows_ptr;      // rows of the nodes
    std::vector<Tile> prod;               // tiles of the descendants' rows x node columns
    std::vector<int> prod_ptr;
    std::vector<Tile> inv;                // tiles of the node inverses, largest nodes first
    std::vector<int> inv_ptr;
    std::vector<int> first, first_ptr;    // nodes, largest first
    std::vector<std::vector<int>> inv_n;  // per height and block step: tiles that take part
    int nlong = 0;                        // rows with at least kNdLongRow entries of Y
    int cmap_len = 0;
    size_t wtot = 0, qtot = 0, xtot = 0, stot = 0;  // doubles
    // Empties the lists and keeps their storage for the next plan.
    void clear();
};
constexpr int kNdLongRow = 1024;

// Builds the plan of a pattern (rp, ci: sorted rows).  False if the pattern
// is not structurally symmetric with a full diagonal, or its graph does not
// separate well enough: the natural-order solver then reads less or needs
// less memory.  known_symmetric: the pattern is known to be structurally
// symmetric and its diagonal full (it is not looked at again).
bool nd_plan(int n, const int *rp, const int *ci, NdPlan &P, bool known_symmetric = false);
// True if every row is strictly diagonally dominant by kNdMargin.
bool nd_dominant(int n, const int *rp, const int *ci, const double *val);

}  // namespace msp
