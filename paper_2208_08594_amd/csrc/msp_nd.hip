// Kernels of the nested-dissection coarsest-level solver (see msp_nd.h), for
// gfx950: the inverse factors of all nodes of one height of the tree per
// launch, FP64 matrix cores for the dense products and the node inverses.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "msp_lanes.h"
#include "msp_nd_device.h"

namespace msp {

namespace {

constexpr int kThreads = 256;
constexpr int kT = kNdTile;
constexpr int kKC = 16;  // k-chunk of the node products
typedef double dbl4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// lists that follow from the tree: per node, its rows' node numbers, the
// columns of its chain and the solve's row descriptors (one work-group a node)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_nd_nodes(NdDev d)
{
    const int v = blockIdx.x;
    const NdNode q = d.node[v];
    for (int r = threadIdx.x; r < q.m; r += kThreads) {
        const int row = q.s + r;
        d.nodeof[row] = v;
        d.perm[d.iperm[row]] = row;
        d.yrow[q.yord + r] = make_int4(row, q.f, q.s - q.f, (int)(q.qbase + (long long)r * q.qld));
        d.wrow[row] = make_int4((int)(q.wbase + (long long)r * q.c), q.c, q.cbase, 0);
    }
    int o = 0;
    for (int a = v; a >= 0;) {
        const NdNode p = d.node[a];
        for (int r = threadIdx.x; r < p.m; r += kThreads) d.cmap[q.cbase + o + r] = p.s + r;
        o += p.m;
        a = p.parent;
    }
    if (threadIdx.x == 0 && q.c > q.len) d.cmap[q.cbase + q.len] = q.s;  // padding, value zero
}

// the entry lists of every row (one thread a row; rows are short and sorted)
__global__ __launch_bounds__(kThreads) void k_nd_entries(int n, NdDev d)
{
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= n) return;
    const int i = d.iperm[t], b0 = d.rp[i], b1 = d.rp[i + 1];
    const NdNode q = d.node[d.nodeof[t]];
    int ne = 0, ns = 0;
    for (int k = b0; k < b1; ++k) {
        const int j = d.ci[k], r = d.perm[j];
        if (r >= q.s + q.m) continue;  // an ancestor's row, which lists the pair
        if (r >= q.s) {
            d.self[b1 - ++ns] = make_int2(r - q.s, k);
            continue;
        }
        int lo = d.rp[j], hi = d.rp[j + 1];  // the mirror entry (the pattern is symmetric)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (d.ci[mid] < i)
                lo = mid + 1;
            else
                hi = mid;
        }
        d.ent[b0 + ne++] = make_int4(r, d.node[d.nodeof[r]].len - q.len, k, lo);
    }
    d.ecnt[t] = make_int2(ne, ns);
}

// ---------------------------------------------------------------------------
// rows of L(a, S) and U(S, a)^T of the nodes a of one height, S the
// descendants of a: L(a, S) = A(a, S) W(S, S), U(S, a) = Y(S, S) A(S, a).  A
// stored entry towards row r adds a multiple of r's packed row of W (of Y^T),
// which holds the columns of the nodes w on r's chain: those with r in w's
// subtree.  One work-group per row, side and kRowCols columns; each thread
// gathers its columns' terms over the row's entries.
// ---------------------------------------------------------------------------
constexpr int kRowCols = 4 * kThreads;
constexpr int kRowEnts = 64;  // entries staged at a time
__global__ __launch_bounds__(kThreads) void k_nd_rows(NdDev d, const int *__restrict__ rows)
{
    __shared__ int er[kRowEnts], el[kRowEnts];
    __shared__ long long eo[kRowEnts];
    __shared__ double ev[kRowEnts];
    const int c = rows[blockIdx.x];
    const NdNode a = d.node[d.nodeof[c]];
    const int len = a.s - a.f, j0 = (blockIdx.y >> 1) * kRowCols;
    if (j0 >= len) return;
    const bool low = (blockIdx.y & 1) == 0;
    const double *P = low ? d.W : d.Yt;
    double *out = (low ? d.L : d.Ut) + a.qbase + (long long)(c - a.s) * a.qld;
    const int e0 = d.rp[d.iperm[c]], ne = d.ecnt[c].x;
    double acc[4];
    int wf[4], we[4], wl[4], wo[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int j = j0 + u * kThreads + threadIdx.x;
        acc[u] = 0.0;
        wf[u] = 0x7fffffff;  // no row is in this "subtree"
        we[u] = wl[u] = wo[u] = 0;
        if (j < len) {
            const NdNode w = d.node[d.nodeof[a.f + j]];
            wf[u] = w.f;
            we[u] = w.s + w.m;
            wl[u] = w.len;
            wo[u] = a.f + j - w.s;
        }
    }
    for (int k0 = 0; k0 < ne; k0 += kRowEnts) {
        const int m = min(kRowEnts, ne - k0);
        __syncthreads();
        if ((int)threadIdx.x < m) {
            const int4 t = d.ent[e0 + k0 + threadIdx.x];
            const NdNode q = d.node[d.nodeof[t.x]];
            er[threadIdx.x] = t.x;
            el[threadIdx.x] = q.len;
            eo[threadIdx.x] = q.wbase + (long long)(t.x - q.s) * q.c;
            ev[threadIdx.x] = d.val[low ? t.z : t.w];
        }
        __syncthreads();
        for (int k = 0; k < m; ++k) {
            const int r = er[k];
            const double *p = P + eo[k] + el[k];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r >= wf[u] && r < we[u]) acc[u] += ev[k] * p[wo[u] - wl[u]];
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int j = j0 + u * kThreads + threadIdx.x;
        if (j < len) out[j] = acc[u];
    }
}

// 64 x 64 product tile C = sum_k A(i, k) B(j, k) on 4 waves (32 x 32 each),
// both operands through LDS in k-chunks of 16, double buffered.  fa(i, k),
// fb(j, k, x) return the operands (0 beyond K); KMAJ: fb is read with j along
// the lanes instead of k.  x = ix(k) is fb's index of k, read a chunk ahead.
// Lane layout of the FP64 MFMA: A[i][k] in lane i + 16k, B[k][j] in lane
// j + 16k, D[i][j] in lane j + 16(i%4), element i/4.
struct NdLds {
    double A[2][kT][kKC + 1], B[2][kT][kKC + 1];
};
template <bool KMAJ, typename FA, typename FB, typename IX>
__device__ inline void nd_product(int K, const FA &fa, const FB &fb, const IX &ix,
                                  dbl4 (&acc)[2][2], NdLds &s)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32, li = lane & 15, lk = lane >> 4;
    const int ak = tid & 15, ai = tid >> 4;
    const int bk = KMAJ ? tid >> 6 : ak, bj = KMAJ ? tid & 63 : ai;
    double ra[2][4], rb[2][4];
    int x = KMAJ ? 0 : ix(ak);
    const auto fetch = [&](double (&A)[4], double (&Bv)[4], int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) A[u] = fa(ai + 16 * u, k0 + ak);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            Bv[u] = KMAJ ? fb(bj, k0 + bk + 4 * u, 0) : fb(bj + 16 * u, k0 + bk, x);
        if (!KMAJ) x = ix(k0 + kKC + ak);
    };
    const auto stash = [&](const double (&A)[4], const double (&Bv)[4], int buf) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s.A[buf][ai + 16 * u][ak] = A[u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (KMAJ)
                s.B[buf][bj][bk + 4 * u] = Bv[u];
            else
                s.B[buf][bj + 16 * u][bk] = Bv[u];
        }
    };
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
    const int nch = (K + kKC - 1) / kKC;
    // chunk ch from LDS buffer BUF = ch mod 2, chunk ch + 1 in the other
    // register set, chunk ch + 2 on its way into this one
    const auto chunk = [&](auto BUF, int ch) {
        constexpr int buf = decltype(BUF)::value;
        if (ch + 2 < nch) fetch(ra[buf], rb[buf], (ch + 2) * kKC);
#pragma unroll
        for (int kk = 0; kk < kKC; kk += 4) {
            double av[2], bv[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) av[a] = s.A[buf][wr + 16 * a + li][kk + lk];
#pragma unroll
            for (int b = 0; b < 2; ++b) bv[b] = s.B[buf][wc + 16 * b + li][kk + lk];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
        }
        if (ch + 1 < nch) stash(ra[buf ^ 1], rb[buf ^ 1], buf ^ 1);
        __syncthreads();
    };
    fetch(ra[0], rb[0], 0);
    if (nch > 1) fetch(ra[1], rb[1], kKC);
    stash(ra[0], rb[0], 0);
    __syncthreads();
    for (int ch = 0; ch < nch; ch += 2) {
        chunk(std::integral_constant<int, 0>(), ch);
        if (ch + 1 < nch) chunk(std::integral_constant<int, 1>(), ch + 1);
    }
}

// ---------------------------------------------------------------------------
// rows of a descendant v, columns of the node a (K = chain entries of v below
// a): side 0, Y(a, v)^T = -Y^T(v, below) L(a, below)^T, stored packed and, for
// the solve, as rows of Y; side 1, X(v, a) = W(v, below) U(below, a), where
// X = A_SS^-1 A(S, a).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_nd_prod(NdDev d, const int4 *__restrict__ tiles)
{
    __shared__ NdLds s;
    const int4 t = tiles[blockIdx.x];
    const bool low = blockIdx.y == 0;
    const NdNode v = d.node[t.x], a = d.node[t.y];
    const int i0 = t.z >> 16, j0 = t.z & 0xffff, K = t.w;
    double *P = (low ? d.Yt : d.W) + v.wbase;
    const double *Q = (low ? d.L : d.Ut) + a.qbase;
    const int *cm = d.cmap + v.cbase;
    const auto fa = [&](int i, int k) {
        return k < K && i0 + i < v.m ? P[(long long)(i0 + i) * v.c + k] : 0.0;
    };
    const auto ix = [&](int k) { return k < K ? cm[k] - a.f : 0; };
    const auto fb = [&](int j, int k, int x) {
        return k < K && j0 + j < a.m ? Q[(long long)(j0 + j) * a.qld + x] : 0.0;
    };
    dbl4 acc[2][2];
    nd_product<false>(K, fa, fb, ix, acc, s);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r0 = i0 + (wave >> 1) * 32 + (lane >> 4), c0 = j0 + (wave & 1) * 32 + (lane & 15);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + 16 * x + 4 * q, c = c0 + 16 * y;
                if (r >= v.m || c >= a.m) continue;
                if (low) {
                    const double w = -acc[x][y][q];
                    P[(long long)r * v.c + K + c] = w;
                    d.Y[a.qbase + (long long)c * a.qld + v.s + r - a.f] = w;
                } else {
                    d.X[a.xbase + (long long)(v.s + r - a.f) * a.m + c] = acc[x][y][q];
                }
            }
}

// ---------------------------------------------------------------------------
// Schur complement S_a = A(a, a) - A(a, S) X, padded to tiles with the
// identity.  One work-group per padded row (row0 = the node's first padded
// row in the grid's list of nodes).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_nd_schur(NdDev d, const int *__restrict__ nodes)
{
    const NdNode a = d.node[nodes[blockIdx.x]];
    for (int r = blockIdx.y; r < a.mp; r += gridDim.y) {
        double *out = d.S0 + a.sbase + (long long)r * a.mp;
        int e0 = 0, e1 = 0, ne = 0, ns = 0;
        if (r < a.m) {
            const int i = d.iperm[a.s + r];
            const int2 cnt = d.ecnt[a.s + r];
            e0 = d.rp[i];
            e1 = d.rp[i + 1];
            ne = cnt.x;
            ns = cnt.y;
        }
        for (int j = threadIdx.x; j < a.mp; j += kThreads) {
            double acc = (r >= a.m && r == j) ? 1.0 : 0.0;
            if (r < a.m && j < a.m)
                for (int e = 0; e < ne; ++e) {
                    const int4 t = d.ent[e0 + e];
                    acc -= d.val[t.z] * d.X[a.xbase + (long long)(t.x - a.f) * a.m + j];
                }
            out[j] = acc;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < ns; e += kThreads) {
            const int2 t = d.self[e1 - 1 - e];
            out[t.x] += d.val[t.y];
        }
    }
}

// ---------------------------------------------------------------------------
// Inverse of a 64 x 64 block held in LDS (leading dimension kLd), in place,
// by Gauss-Jordan elimination without interchanges in four panels of 16: wave
// 0 inverts the panel's diagonal block in registers (row li, columns 4 lk ..
// 4 lk + 3 per lane), then wave w forms the row panel's column tile w and
// updates the other rows of that tile on the matrix cores.
// ---------------------------------------------------------------------------
constexpr int kLdA = 68, kLdB = 80;  // LDS leading dimensions: row-wise / column-wise reads

// entry of lane t of every row of 16 lanes, to all lanes of that row
template <int T>
__device__ inline double row_bcast(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + T, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + T, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ inline double lane_value(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Steps T .. 15 of the in-place Gauss-Jordan inverse of a 16 x 16 block, row
// li, columns 4 lk .. 4 lk + 3 in x.  A step's chain is the pivot's
// reciprocal, one product and one multiply-add.
template <int T>
__device__ inline void nd_gj16(double (&x)[4], int li, int lk)
{
    if constexpr (T < 16) {
        // (two Newton steps on the hardware's estimate save 1 us of 15.5 a block of
        // 64 rows, but are a unit in the last place off for a few mantissas just
        // below a power of two, which decoupled diagonals of nearly 1 do take)
        const double rp = 1.0 / lane_value(x[T & 3], ((T >> 2) << 4) | T);
        const double f = __shfl(x[T & 3], ((T >> 2) << 4) | li, 64);  // column T, this row
        double pr[4];  // row T, this lane's columns
#pragma unroll
        for (int q = 0; q < 4; ++q) pr[q] = row_bcast<T>(x[q]);
        const double fr = f * rp;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool colt = lk == (T >> 2) && q == (T & 3);
            const double up = colt ? -fr : x[q] - fr * pr[q];
            const double pv = colt ? rp : pr[q] * rp;
            x[q] = li == T ? pv : up;
        }
        nd_gj16<T + 1>(x, li, lk);
    }
}

// Inverse of a pivot block in LDS, its first `rows` rows in use: the padding is
// the identity and couples to nothing, so blocks of 16 rows beyond them are left
// out (14 us for 64 rows, about 3 us less for each block).
__device__ inline void nd_invert64(double (*__restrict__ M)[kLdA], int rows)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int p = 0; 16 * p < min(rows, kT); ++p) {
        const int P0 = 16 * p;
        if (wave == 0) {
            double x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = M[P0 + li][P0 + 4 * lk + q];
            nd_gj16<0>(x, li, lk);
#pragma unroll
            for (int q = 0; q < 4; ++q) M[P0 + li][P0 + 4 * lk + q] = x[q];
        }
        __syncthreads();
        // wave w, column tile w: R = D M(p, w), M(i, w) -= M(i, p) R for
        // i != p; the wave of the panel's own tile forms -M(i, p) D instead
        double bp[4], ad[4];
        dbl4 R{0.0, 0.0, 0.0, 0.0}, C[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            bp[k] = M[P0 + 4 * k + lk][16 * wave + li];
            ad[k] = M[P0 + li][P0 + 4 * k + lk];
        }
        if (wave != p) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                R = __builtin_amdgcn_mfma_f64_16x16x4f64(ad[k], bp[k], R, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) bp[k] = R[k];  // element k is row 4k + lk: a B operand
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i == p) {
                C[i] = R;
                continue;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                C[i][r] = wave == p ? 0.0 : M[16 * i + lk + 4 * r][16 * wave + li];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                C[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(-M[16 * i + li][P0 + 4 * k + lk], bp[k],
                                                           C[i], 0, 0, 0);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i == p && wave == p) continue;  // the inverted diagonal block stays
#pragma unroll
            for (int r = 0; r < 4; ++r) M[16 * i + lk + 4 * r][16 * wave + li] = C[i][r];
        }
        __syncthreads();
    }
}

// A 64 x 64 tile between global memory (leading dimension ld, 16-byte aligned
// rows) and LDS: all loads of a thread go out before the first store.
template <int LD>
__device__ inline void nd_tile_in(const double *__restrict__ S, int ld, double (*__restrict__ M)[LD])
{
    double2 v[8];
    const int r = threadIdx.x >> 5, c = 2 * (threadIdx.x & 31);
#pragma unroll
    for (int u = 0; u < 8; ++u)
        v[u] = *reinterpret_cast<const double2 *>(S + (long long)(r + 8 * u) * ld + c);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        M[r + 8 * u][c] = v[u].x;
        M[r + 8 * u][c + 1] = v[u].y;
    }
}
template <int LD>
__device__ inline void nd_tile_out(const double (*__restrict__ M)[LD], double *__restrict__ S, int ld)
{
    const int r = threadIdx.x >> 5, c = 2 * (threadIdx.x & 31);
#pragma unroll
    for (int u = 0; u < 8; ++u)
        *reinterpret_cast<double2 *>(S + (long long)(r + 8 * u) * ld + c) =
            make_double2(M[r + 8 * u][c], M[r + 8 * u][c + 1]);
}

// First pivot block of every node: D = S(0, 0)^-1 into the node's slot of Dk.
__global__ __launch_bounds__(kThreads) void k_nd_first(NdDev d, const int *__restrict__ nodes)
{
    __shared__ double M[kT][kLdA];
    const int id = nodes[blockIdx.x];
    const NdNode a = d.node[id];
    nd_tile_in(d.S0 + a.sbase, a.mp, M);
    __syncthreads();
    nd_invert64(M, a.m);
    nd_tile_out(M, d.Dk + (long long)id * 2 * kT * kT, kT);
}

// Block step k of the node inverses (blocked Gauss-Jordan without
// interchanges), S -> the other buffer, one 64 x 64 tile (i, j) per
// work-group, D the inverse of pivot block k:
//   (k, k): D;  (k, j): D S_kj;  (i, k): -S_ik D;  else S_ij - S_ik (D S_kj).
// Each tile forms D S_kj itself, so a step is one launch; the work-group of
// tile (k+1, k+1) then inverts that tile for the next step.
__global__ __launch_bounds__(kThreads) void k_nd_step(NdDev d, const int4 *__restrict__ tiles, int k)
{
    __shared__ double Am[kT][kLdA], Dm[kT][kLdA], Bm[kT][kLdB];
    const int4 t = tiles[blockIdx.x];
    const NdNode a = d.node[t.x];
    const int i0 = t.z >> 16, j0 = t.z & 0xffff, k0 = k * kT, tid = threadIdx.x;
    const double *S = (k & 1 ? d.S1 : d.S0) + a.sbase;
    double *O = (k & 1 ? d.S0 : d.S1) + a.sbase;
    const double *D = d.Dk + ((long long)t.x * 2 + (k & 1)) * kT * kT;
    const bool rk = i0 == k0, ck = j0 == k0;
    nd_tile_in(D, kT, Dm);
    if (!rk) nd_tile_in(S + (long long)i0 * a.mp + k0, a.mp, Am);
    if (ck)
        nd_tile_in(D, kT, Bm);
    else
        nd_tile_in(S + (long long)k0 * a.mp + j0, a.mp, Bm);
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    dbl4 acc[2][2];
    // product of a row-wise with a column-wise operand, this wave's 32 x 32
    const auto mul = [&](const double (*X)[kLdA], double sgn) {
#pragma unroll 4
        for (int kk = 0; kk < kT; kk += 4) {
            double av[2], bv[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) av[x] = sgn * X[wr + 16 * x + li][kk + lk];
#pragma unroll
            for (int y = 0; y < 2; ++y) bv[y] = Bm[kk + lk][wc + 16 * y + li];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv[y], acc[x][y], 0, 0, 0);
        }
    };
    const auto load = [&](auto &&f) {  // acc = f(row, column)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[x][y][q] = f(wr + 16 * x + lk + 4 * q, wc + 16 * y + li);
    };
    const auto store = [&](auto &&f) {  // f(row, column, acc)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    f(wr + 16 * x + lk + 4 * q, wc + 16 * y + li, (double)acc[x][y][q]);
    };
    if (!ck) {  // T = D S_kj
        load([](int, int) { return 0.0; });
        mul(Dm, 1.0);
        __syncthreads();
        store([&](int r, int c, double v) { Bm[r][c] = v; });
        __syncthreads();
    }
    if (rk) {
        nd_tile_out(Bm, O + (long long)i0 * a.mp + j0, a.mp);
        return;
    }
    load([&](int r, int c) { return ck ? 0.0 : S[(long long)(i0 + r) * a.mp + j0 + c]; });
    mul(Am, -1.0);
    store([&](int r, int c, double v) { O[(long long)(i0 + r) * a.mp + j0 + c] = v; });
    if (i0 == k0 + kT && j0 == k0 + kT) {  // the next pivot block
        __syncthreads();  // every wave has read Am
        store([&](int r, int c, double v) { Am[r][c] = v; });
        __syncthreads();
        nd_invert64(Am, a.m - i0);
        nd_tile_out(Am, d.Dk + ((long long)t.x * 2 + ((k + 1) & 1)) * kT * kT, kT);
    }
}

// W(v, a) = -X(v, a) S_a^-1 for the descendants' rows (ntile tiles); the
// work-groups after them take one row each of the nodes themselves: S_a^-1
// into its packed row of W, the identity into that of Y^T.
__global__ __launch_bounds__(kThreads) void k_nd_scale(NdDev d, const int4 *__restrict__ tiles,
                                                       int ntile, const int *__restrict__ rows)
{
    __shared__ NdLds s;
    const int b = blockIdx.x;
    if (b >= ntile) {
        const int c = rows[b - ntile];
        const NdNode a = d.node[d.nodeof[c]];
        const int r = c - a.s;
        const double *Sv = ((a.mp / kT) & 1 ? d.S1 : d.S0) + a.sbase + (long long)r * a.mp;
        double *w = d.W + a.wbase + (long long)r * a.c, *y = d.Yt + a.wbase + (long long)r * a.c;
        for (int j = threadIdx.x; j < a.m; j += kThreads) {
            w[j] = Sv[j];
            y[j] = r == j ? 1.0 : 0.0;
        }
        return;
    }
    const int4 t = tiles[b];
    const NdNode v = d.node[t.x], a = d.node[t.y];
    const int i0 = t.z >> 16, j0 = t.z & 0xffff;
    const double *X = d.X + a.xbase + (long long)(v.s - a.f) * a.m;
    const double *Sv = ((a.mp / kT) & 1 ? d.S1 : d.S0) + a.sbase;
    const auto fa = [&](int i, int k) {
        return k < a.m && i0 + i < v.m ? X[(long long)(i0 + i) * a.m + k] : 0.0;
    };
    const auto fb = [&](int j, int k, int) {
        return k < a.m && j0 + j < a.m ? Sv[(long long)k * a.mp + j0 + j] : 0.0;
    };
    dbl4 acc[2][2];
    nd_product<true>(a.m, fa, fb, [](int) { return 0; }, acc, s);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r0 = i0 + (wave >> 1) * 32 + (lane >> 4), c0 = j0 + (wave & 1) * 32 + (lane & 15);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + 16 * x + 4 * q, c = c0 + 16 * y;
                if (r < v.m && c < a.m)
                    d.W[v.wbase + (long long)r * v.c + t.w + c] = -acc[x][y][q];
            }
}

// ---------------------------------------------------------------------------
// solve x = W (Y f), FP64 arithmetic: t = f + Y(., descendants) f, then
// x = W t.  Rows of Y by falling length: the nlong longest take a work-group
// each (four waves share the row), the rest a wavefront each.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kThreads) void k_nd_lower(int n, int nlong,
                                                       const int4 *__restrict__ rows,
                                                       const double *__restrict__ Y,
                                                       const T *__restrict__ f,
                                                       double *__restrict__ t)
{
    __shared__ double red[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, b = blockIdx.x;
    const bool wide = b < nlong;  // uniform over the work-group
    const int q = wide ? b : nlong + (b - nlong) * 4 + wave;
    if (q >= n) return;  // (only in a work-group of single-wave rows)
    const int4 d = rows[q];
    const double *y = Y + d.w;
    const T *fv = f + d.y;
    const int step = wide ? 512 : 128;
    double acc = 0.0;
#pragma unroll 4
    for (int j = 2 * lane + (wide ? 128 * wave : 0); j + 1 < d.z; j += step) {
        const double2 v = *reinterpret_cast<const double2 *>(y + j);
        acc += v.x * (double)fv[j] + v.y * (double)fv[j + 1];
    }
    if ((d.z & 1) && lane == 0 && (!wide || wave == 0)) acc += y[d.z - 1] * (double)fv[d.z - 1];
    acc = wave_sum(acc);
    if (wide) {
        if (lane == 0) red[wave] = acc;
        __syncthreads();
        if (threadIdx.x == 0)
            t[d.x] = (double)f[d.x] + ((red[0] + red[1]) + (red[2] + red[3]));
    } else if (lane == 0) {
        t[d.x] = (double)f[d.x] + acc;
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_nd_upper(int n, const int4 *__restrict__ rows,
                                                       const int *__restrict__ cmap,
                                                       const double *__restrict__ W,
                                                       const double *__restrict__ t,
                                                       T *__restrict__ x,
                                                       const int *__restrict__ map)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= n) return;
    const int4 d = rows[row];
    const double *w = W + d.x;
    const int *cm = cmap + d.z;
    double acc = 0.0;
#pragma unroll 4
    for (int j = 2 * lane; j < d.y; j += 128) {
        const double2 v = *reinterpret_cast<const double2 *>(w + j);
        acc += v.x * t[cm[j]] + v.y * t[cm[j + 1]];
    }
    acc = wave_sum(acc);
    if (lane == 0) x[map ? map[row] : row] = (T)acc;
}

__global__ __launch_bounds__(kThreads) void k_nd_zero(long long n, double *__restrict__ x)
{
    for (long long q = (long long)blockIdx.x * kThreads + threadIdx.x; q < n;
         q += (long long)gridDim.x * kThreads)
        x[q] = 0.0;
}

}  // namespace

hipError_t launch_nd_factor(const NdPlan &P, const NdDev &d, hipStream_t st)
{
    k_nd_nodes<<<(unsigned)P.node.size(), kThreads, 0, st>>>(d);
    k_nd_entries<<<(P.n + kThreads - 1) / kThreads, kThreads, 0, st>>>(P.n, d);
    k_nd_zero<<<1024, kThreads, 0, st>>>((long long)P.wtot, d.W);  // the rows' padding entries
    for (int h = 0; h < P.heights; ++h) {
        const int nodes = P.first_ptr[h + 1] - P.first_ptr[h];
        const int nprod = P.prod_ptr[h + 1] - P.prod_ptr[h];
        const int nrows = P.rows_ptr[h + 1] - P.rows_ptr[h];
        const int *first = d.first + P.first_ptr[h], *rows = d.rows + P.rows_ptr[h];
        const int4 *prod = d.prod + P.prod_ptr[h], *inv = d.inv + P.inv_ptr[h];
        if (nodes == 0) continue;
        const int mp = P.node[P.first[P.first_ptr[h]]].mp;  // the largest
        if (nprod > 0) {
            int len = 0;
            for (int q = P.first_ptr[h]; q < P.first_ptr[h + 1]; ++q)
                len = std::max(len, P.node[P.first[q]].s - P.node[P.first[q]].f);
            k_nd_rows<<<dim3(nrows, 2 * ((len + kRowCols - 1) / kRowCols)), kThreads, 0, st>>>(d,
                                                                                            rows);
            k_nd_prod<<<dim3(nprod, 2), kThreads, 0, st>>>(d, prod);
        }
        k_nd_schur<<<dim3(nodes, mp), kThreads, 0, st>>>(d, first);
        k_nd_first<<<nodes, kThreads, 0, st>>>(d, first);
        for (size_t k = 0; k < P.inv_n[h].size(); ++k)
            k_nd_step<<<P.inv_n[h][k], kThreads, 0, st>>>(d, inv, (int)k);
        k_nd_scale<<<nprod + nrows, kThreads, 0, st>>>(d, prod, nprod, rows);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_nd_solve(const NdSolve &s, const T *f, double *t, T *x, const int *map,
                           hipStream_t st)
{
    k_nd_lower<T><<<s.nlong + (s.n - s.nlong + 3) / 4, kThreads, 0, st>>>(s.n, s.nlong, s.yrow, s.Y,
                                                                         f, t);
    k_nd_upper<T><<<(s.n + 3) / 4, kThreads, 0, st>>>(s.n, s.wrow, s.cmap, s.W, t, x, map);
    return hipGetLastError();
}
template hipError_t launch_nd_solve<float>(const NdSolve &, const float *, double *, float *,
                                           const int *, hipStream_t);
template hipError_t launch_nd_solve<double>(const NdSolve &, const double *, double *, double *,
                                            const int *, hipStream_t);

}  // namespace msp
