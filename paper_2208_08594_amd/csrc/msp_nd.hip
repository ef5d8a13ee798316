// Kernels of the nested-dissection coarsest-level solver (see msp_nd.h), for
// gfx950: the inverse factors of all nodes of one height of the tree per
// launch, FP64 matrix cores for the dense products and the node inverses.
#include <hip/hip_runtime.h>

#include "msp_nd_device.h"

namespace msp {

namespace {

constexpr int kThreads = 256;
constexpr int kT = kNdTile;
constexpr int kKC = 16;  // k-chunk of the node products
typedef double dbl4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// rows of L(a, S) and U(S, a)^T of the nodes a of one height, S the
// descendants of a: L(a, S) = A(a, S) W(S, S), U(S, a) = Y(S, S) A(S, a).
// Each stored entry adds a multiple of one packed row of W (of Y^T), whose
// columns below a are distinct.  One work-group per row and side.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_nd_rows(NdDev d, const int *__restrict__ rows)
{
    const int c = rows[blockIdx.x];
    const bool low = blockIdx.y == 0;
    const NdNode a = d.node[d.nodeof[c]];
    const int len = a.s - a.f;
    double *out = (low ? d.L : d.Ut) + a.qbase + (long long)(c - a.s) * a.qld;
    const double *P = low ? d.W : d.Yt;
    for (int j = threadIdx.x; j < len; j += kThreads) out[j] = 0.0;
    for (int e = d.ent_ptr[c]; e < d.ent_ptr[c + 1]; ++e) {
        __syncthreads();  // the writes of the previous entry are complete
        const int4 t = d.ent[e];
        const double v = d.val[low ? t.z : t.w];
        const NdNode q = d.node[d.nodeof[t.x]];
        const double *p = P + q.wbase + (long long)(t.x - q.s) * q.c;
        const int *cm = d.cmap + q.cbase;
        for (int k = threadIdx.x; k < t.y; k += kThreads) out[cm[k] - a.f] += v * p[k];
    }
}

// 64 x 64 product tile C = sum_k A(i, k) B(j, k) on 4 waves (32 x 32 each),
// both operands through LDS in k-chunks of 16, double buffered.  fa(i, k),
// fb(j, k) return the operands (0 beyond K); KMAJ: fb is read with j along
// the lanes instead of k.  Lane layout of the FP64 MFMA: A[i][k] in lane
// i + 16k, B[k][j] in lane j + 16k, D[i][j] in lane j + 16(i%4), element i/4.
struct NdLds {
    double A[2][kT][kKC + 1], B[2][kT][kKC + 1];
};
template <bool KMAJ, typename FA, typename FB>
__device__ inline void nd_product(int K, const FA &fa, const FB &fb, dbl4 (&acc)[2][2], NdLds &s)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32, li = lane & 15, lk = lane >> 4;
    const int ak = tid & 15, ai = tid >> 4;
    const int bk = KMAJ ? tid >> 6 : ak, bj = KMAJ ? tid & 63 : ai;
    double ra[4], rb[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) ra[u] = fa(ai + 16 * u, k0 + ak);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            rb[u] = KMAJ ? fb(bj, k0 + bk + 4 * u) : fb(bj + 16 * u, k0 + bk);
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 4; ++u) s.A[buf][ai + 16 * u][ak] = ra[u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (KMAJ)
                s.B[buf][bj][bk + 4 * u] = rb[u];
            else
                s.B[buf][bj + 16 * u][bk] = rb[u];
        }
    };
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
    const int nch = (K + kKC - 1) / kKC;
    fetch(0);
    stash(0);
    __syncthreads();
    for (int ch = 0; ch < nch; ++ch) {
        const int buf = ch & 1;
        if (ch + 1 < nch) fetch((ch + 1) * kKC);
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
        if (ch + 1 < nch) stash(buf ^ 1);
        __syncthreads();
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
    const auto fb = [&](int j, int k) {
        return k < K && j0 + j < a.m ? Q[(long long)(j0 + j) * a.qld + cm[k] - a.f] : 0.0;
    };
    dbl4 acc[2][2];
    nd_product<false>(K, fa, fb, acc, s);
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
        const int c = a.s + r;
        for (int j = threadIdx.x; j < a.mp; j += kThreads) {
            double acc = (r >= a.m && r == j) ? 1.0 : 0.0;
            if (r < a.m && j < a.m)
                for (int e = d.ent_ptr[c]; e < d.ent_ptr[c + 1]; ++e) {
                    const int4 t = d.ent[e];
                    acc -= d.val[t.z] * d.X[a.xbase + (long long)(t.x - a.f) * a.m + j];
                }
            out[j] = acc;
        }
        __syncthreads();
        if (r < a.m)
            for (int e = d.self_ptr[c] + threadIdx.x; e < d.self_ptr[c + 1]; e += kThreads) {
                const int2 t = d.self[e];
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

__device__ inline void nd_invert64(double (*__restrict__ M)[kLdA])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int p = 0; p < 4; ++p) {
        const int P0 = 16 * p;
        if (wave == 0) {
            double x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = M[P0 + li][P0 + 4 * lk + q];
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                // row t (this lane's columns), column t (this lane's row), pivot
                double pr[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) pr[q] = __shfl(x[q], (lane & 48) | t, 64);
                const double f = __shfl(x[t & 3], ((t >> 2) << 4) | li, 64);
                const double rp = 1.0 / __shfl(x[t & 3], ((t >> 2) << 4) | t, 64);
                const double fr = f * rp;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool colt = 4 * lk + q == t;
                    const double up = colt ? -fr : x[q] - fr * pr[q];
                    const double pv = colt ? rp : pr[q] * rp;
                    x[q] = li == t ? pv : up;
                }
            }
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

// First pivot block of every node: D = S(0, 0)^-1 into the node's slot of Dk.
__global__ __launch_bounds__(kThreads) void k_nd_first(NdDev d, const int *__restrict__ nodes)
{
    __shared__ double M[kT][kLdA];
    const int id = nodes[blockIdx.x];
    const NdNode a = d.node[id];
    const double *S = d.S0 + a.sbase;
    for (int q = threadIdx.x; q < kT * kT; q += kThreads)
        M[q >> 6][q & 63] = S[(long long)(q >> 6) * a.mp + (q & 63)];
    __syncthreads();
    nd_invert64(M);
    double *D = d.Dk + (long long)id * 2 * kT * kT;
    for (int q = threadIdx.x; q < kT * kT; q += kThreads) D[q] = M[q >> 6][q & 63];
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
    for (int q = tid; q < kT * kT; q += kThreads) {
        const int r = q >> 6, c = q & 63;
        const double dv = D[q];
        Dm[r][c] = dv;
        if (!rk) Am[r][c] = S[(long long)(i0 + r) * a.mp + k0 + c];
        Bm[r][c] = ck ? dv : S[(long long)(k0 + r) * a.mp + j0 + c];
    }
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    dbl4 acc[2][2];
    // product of a row-wise with a column-wise operand, this wave's 32 x 32
    const auto mul = [&](const double (*X)[kLdA], double sgn) {
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
        for (int q = tid; q < kT * kT; q += kThreads)
            O[(long long)(i0 + (q >> 6)) * a.mp + j0 + (q & 63)] = Bm[q >> 6][q & 63];
        return;
    }
    load([&](int r, int c) { return ck ? 0.0 : S[(long long)(i0 + r) * a.mp + j0 + c]; });
    mul(Am, -1.0);
    store([&](int r, int c, double v) { O[(long long)(i0 + r) * a.mp + j0 + c] = v; });
    if (i0 == k0 + kT && j0 == k0 + kT) {  // the next pivot block
        __syncthreads();  // every wave has read Am
        store([&](int r, int c, double v) { Am[r][c] = v; });
        __syncthreads();
        nd_invert64(Am);
        double *N = d.Dk + ((long long)t.x * 2 + ((k + 1) & 1)) * kT * kT;
        for (int q = tid; q < kT * kT; q += kThreads) N[q] = Am[q >> 6][q & 63];
    }
}

// W(v, a) = -X(v, a) S_a^-1 for the descendants' rows; a tile with v == a
// copies the inverse itself into the node's rows of W (and the identity into
// those of Y^T).
__global__ __launch_bounds__(kThreads) void k_nd_scale(NdDev d, const int4 *__restrict__ tiles)
{
    __shared__ NdLds s;
    const int4 t = tiles[blockIdx.x];
    const NdNode v = d.node[t.x], a = d.node[t.y];
    const int i0 = t.z >> 16, j0 = t.z & 0xffff;
    const double *X = d.X + a.xbase + (long long)(v.s - a.f) * a.m;
    const double *Sv = ((a.mp / kT) & 1 ? d.S1 : d.S0) + a.sbase;
    const auto fa = [&](int i, int k) {
        return k < a.m && i0 + i < v.m ? X[(long long)(i0 + i) * a.m + k] : 0.0;
    };
    const auto fb = [&](int j, int k) {
        return k < a.m && j0 + j < a.m ? Sv[(long long)k * a.mp + j0 + j] : 0.0;
    };
    dbl4 acc[2][2];
    nd_product<true>(a.m, fa, fb, acc, s);
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

// The nodes' own entries: S_a^-1 into the packed rows of W, the identity into
// those of Y^T, zero into the padding entry of every row.
__global__ __launch_bounds__(kThreads) void k_nd_own(NdDev d, const int *__restrict__ nodes)
{
    const NdNode a = d.node[nodes[blockIdx.x]];
    const double *Sv = ((a.mp / kT) & 1 ? d.S1 : d.S0) + a.sbase;
    for (int r = blockIdx.y; r < a.m; r += gridDim.y) {
        double *w = d.W + a.wbase + (long long)r * a.c, *y = d.Yt + a.wbase + (long long)r * a.c;
        for (int j = threadIdx.x; j < a.m; j += kThreads) {
            w[j] = Sv[(long long)r * a.mp + j];
            y[j] = r == j ? 1.0 : 0.0;
        }
    }
}

// ---------------------------------------------------------------------------
// solve x = W (Y f), FP64 arithmetic: t = f + Y(., descendants) f, then
// x = W t.  Rows of Y by falling length: the nlong longest take a work-group
// each (four waves share the row), the rest a wavefront each.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double nd_wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

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
    acc = nd_wave_sum(acc);
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
    acc = nd_wave_sum(acc);
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
    k_nd_zero<<<1024, kThreads, 0, st>>>((long long)P.wtot, d.W);  // the rows' padding entries
    for (int h = 0; h < P.heights; ++h) {
        const int nodes = P.first_ptr[h + 1] - P.first_ptr[h];
        const int nprod = P.prod_ptr[h + 1] - P.prod_ptr[h];
        const int nrows = P.rows_ptr[h + 1] - P.rows_ptr[h];
        const int *first = d.first + P.first_ptr[h];
        const int4 *prod = d.prod + P.prod_ptr[h], *inv = d.inv + P.inv_ptr[h];
        if (nodes == 0) continue;
        const int mp = P.node[P.first[P.first_ptr[h]]].mp;  // the largest
        if (nprod > 0) {
            k_nd_rows<<<dim3(nrows, 2), kThreads, 0, st>>>(d, d.rows + P.rows_ptr[h]);
            k_nd_prod<<<dim3(nprod, 2), kThreads, 0, st>>>(d, prod);
        }
        k_nd_schur<<<dim3(nodes, mp), kThreads, 0, st>>>(d, first);
        k_nd_first<<<nodes, kThreads, 0, st>>>(d, first);
        for (size_t k = 0; k < P.inv_n[h].size(); ++k)
            k_nd_step<<<P.inv_n[h][k], kThreads, 0, st>>>(d, inv, (int)k);
        k_nd_own<<<dim3(nodes, mp), kThreads, 0, st>>>(d, first);
        if (nprod > 0) k_nd_scale<<<nprod, kThreads, 0, st>>>(d, prod);
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
