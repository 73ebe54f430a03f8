// Kernels of the outer iteration that evaluate the problem's coefficients: the
// residual of a gridded u~ and the second stage of PDD.
#include <algorithm>

#include "path_walk.hpp"

namespace pdd {
namespace {

// Residual r = f - ((1/2) sigma^2 Lap u + b.grad u + c u) of a gridded u at
// its points, b, c, f from the problem (FP64), the derivatives of u by
// second-order differences (central inside; three-point one-sided first and
// four-point one-sided second derivatives at the ends of each axis).
template <class S>
__device__ __forceinline__ double fd_first(const S *__restrict__ u, uint64_t p, uint64_t s, int a, int n, double dx)
{
    if (a == 0) return (-3.0 * (double)u[p] + 4.0 * (double)u[p + s] - (double)u[p + 2 * s]) / (2.0 * dx);
    if (a == n - 1) return (3.0 * (double)u[p] - 4.0 * (double)u[p - s] + (double)u[p - 2 * s]) / (2.0 * dx);
    return ((double)u[p + s] - (double)u[p - s]) / (2.0 * dx);
}

template <class S>
__device__ __forceinline__ double fd_second(const S *__restrict__ u, uint64_t p, uint64_t s, int a, int n, double dx)
{
    if (a == 0)
        return (2.0 * (double)u[p] - 5.0 * (double)u[p + s] + 4.0 * (double)u[p + 2 * s] - (double)u[p + 3 * s]) /
               (dx * dx);
    if (a == n - 1)
        return (2.0 * (double)u[p] - 5.0 * (double)u[p - s] + 4.0 * (double)u[p - 2 * s] - (double)u[p - 3 * s]) /
               (dx * dx);
    return ((double)u[p + s] - 2.0 * (double)u[p] + (double)u[p - s]) / (dx * dx);
}

template <class S, int D>
__global__ void __launch_bounds__(256) grid_residual_kernel(const DevProblem<double> P, const S *__restrict__ u,
                                                            int n0, int n1, int n2, double lo0, double lo1,
                                                            double lo2, double dx0, double dx1, double dx2,
                                                            double half_s2, S *__restrict__ r)
{
    __shared__ double s_cf[kMaxDense];
    for (int q = threadIdx.x; q < kMaxDense; q += blockDim.x) s_cf[q] = P.fdense[q];
    __syncthreads();
    const uint64_t m01 = (uint64_t)n0 * n1;
    const uint64_t total = m01 * (D == 3 ? (uint64_t)n2 : 1);
    const int nn[3] = {n0, n1, n2};
    MathOf<double> mt;
    mt.init();
    const double lo[3] = {lo0, lo1, lo2}, dx[3] = {dx0, dx1, dx2};
    const uint64_t st[3] = {1, (uint64_t)n0, m01};
    for (uint64_t p = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; p < total;
         p += (uint64_t)gridDim.x * blockDim.x) {
        const int idx[3] = {(int)(p % n0), (int)((p / n0) % n1), D == 3 ? (int)(p / m01) : 0};
        double x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) x[d] = lo[d] + (double)idx[d] * dx[d];
        double b[D], c, f = 0.0;
        coefficients<double, D, true>(mt, P, x, b, c, f, true, s_cf, P.tab);
        double lap = 0.0, adv = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lap += fd_second<S>(u, p, st[d], idx[d], nn[d], dx[d]);
            adv += b[d] * fd_first<S>(u, p, st[d], idx[d], nn[d], dx[d]);
        }
        r[p] = (S)(f - (half_s2 * lap + adv + c * (double)u[p]));
    }
}

// Second stage (the subdomain-BVP step of Alg. A:IterPDD) on a 2D box cut by
// axis-parallel interfaces. Grid coordinates are lo + span i / (n - 1), as
// everywhere the grids are sampled.
__device__ __forceinline__ double stage2_coord(double lo, double span, int n, int i)
{
    return lo + span * (double)i / (double)(n - 1);
}

// g at every point of the box's edges.
__global__ void __launch_bounds__(256) stage2_boundary_kernel(const DevProblem<double> P, const Stage2Grid g)
{
    const int n0 = g.n0, n1 = g.n1;
    const int total = 2 * n0 + 2 * (n1 - 2);
    MathOf<double> mt;
    mt.init();
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < total; q += gridDim.x * blockDim.x) {
        int i, j;
        if (q < n0) {
            i = q, j = 0;
        } else if (q < 2 * n0) {
            i = q - n0, j = n1 - 1;
        } else {
            const int r = q - 2 * n0;
            i = (r & 1) ? n0 - 1 : 0;
            j = 1 + (r >> 1);
        }
        const double x[2] = {stage2_coord(g.lo0, g.span0, n0, i), stage2_coord(g.lo1, g.span1, n1, j)};
        g.u[(size_t)j * n0 + i] = boundary_value<double, 2, true>(mt, P, x, P.tab);
    }
}

__device__ __forceinline__ double multiquadric(const double *t, const double *lam, int m, double eps, double x)
{
    double acc = 0.0;
    for (int q = 0; q < m; ++q) {
        const double e = eps * (x - t[q]);
        acc += lam[q] * sqrt(1.0 + e * e);
    }
    return acc;
}

// One workgroup row per line (blockIdx.y); the points of the line strictly
// between the box's edges.
__global__ void __launch_bounds__(256) stage2_lines_kernel(const Stage2Grid g, const Stage2Line *lines, int32_t n_lines,
                                                           const double *t, const double *lam)
{
    const Stage2Line L = lines[blockIdx.y];
    const int ne = L.d == 0 ? g.n1 : g.n0;  // points along the line
    for (int p = 1 + blockIdx.x * blockDim.x + threadIdx.x; p < ne - 1; p += gridDim.x * blockDim.x) {
        const double tp = L.d == 0 ? stage2_coord(g.lo1, g.span1, g.n1, p) : stage2_coord(g.lo0, g.span0, g.n0, p);
        // a line of the other axis through this point
        int cross = -1;
        for (int q = 0; q < n_lines; ++q)
            if (lines[q].d != L.d && lines[q].k == p) cross = q;
        if (cross >= 0 && L.d == 1) continue;  // the crossing axis-0 line writes the point
        double v = multiquadric(t + L.at, lam + L.at, L.m, L.eps, tp);
        if (cross >= 0) {
            const Stage2Line C = lines[cross];
            const double tc = stage2_coord(g.lo0, g.span0, g.n0, L.k);
            v = 0.5 * (v + multiquadric(t + C.at, lam + C.at, C.m, C.eps, tc));
        }
        const size_t at = L.d == 0 ? (size_t)p * g.n0 + L.k : (size_t)L.k * g.n0 + p;
        g.u[at] = v;
    }
}

// Grid point of unknown r of a subdomain.
__device__ __forceinline__ void stage2_point(const SubBox &b, uint64_t r, int &i, int &j)
{
    const int s = (int)(r / (uint64_t)b.w), f = (int)(r % (uint64_t)b.w);
    if (b.fast_x) {
        i = b.i0 + 1 + f;
        j = b.j0 + 1 + s;
    } else {
        i = b.i0 + 1 + s;
        j = b.j0 + 1 + f;
    }
}

// Stencil of every unknown: (1/2) sigma^2 Lap v + b.grad v + c v = f by
// second-order differences; neighbours on the subdomain's boundary move to
// the right side with their grid values. Slots: 0 slow-1, 1 fast-1,
// 2 centre, 3 fast+1, 4 slow+1, 5 right side; aux: f, and the boundary
// neighbours' part of the right side (the same products, summed from zero).
__global__ void __launch_bounds__(256) stage2_stencil_kernel(const DevProblem<double> P, const Stage2Grid g,
                                                             const SubBox *boxes, double *stencil, double *aux)
{
    __shared__ double s_cf[kMaxDense];
    for (int q = threadIdx.x; q < kMaxDense; q += blockDim.x) s_cf[q] = P.fdense[q];
    __syncthreads();
    const SubBox b = boxes[blockIdx.y];
    MathOf<double> mt;
    mt.init();
    const uint64_t n = (uint64_t)b.w * (uint64_t)b.L;
    const double cx = g.half_s2 / (g.dx0 * g.dx0), cy = g.half_s2 / (g.dx1 * g.dx1);
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        int i, j;
        stage2_point(b, r, i, j);
        const double x[2] = {stage2_coord(g.lo0, g.span0, g.n0, i), stage2_coord(g.lo1, g.span1, g.n1, j)};
        double bb[2], c, f = 0.0;
        coefficients<double, 2, true>(mt, P, x, bb, c, f, true, s_cf, P.tab);
        const double aW = cx - bb[0] / (2.0 * g.dx0), aE = cx + bb[0] / (2.0 * g.dx0);
        const double aS = cy - bb[1] / (2.0 * g.dx1), aN = cy + bb[1] / (2.0 * g.dx1);
        double out[6] = {0.0, 0.0, -2.0 * cx - 2.0 * cy + c, 0.0, 0.0, f};
        double yb = 0.0;
        // neighbours: west, east, south, north with their band slots
        const int ni[4] = {i - 1, i + 1, i, i};
        const int nj[4] = {j, j, j - 1, j + 1};
        const double a[4] = {aW, aE, aS, aN};
        const int slot[4] = {b.fast_x ? 1 : 0, b.fast_x ? 3 : 4, b.fast_x ? 0 : 1, b.fast_x ? 4 : 3};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool inside = ni[q] > b.i0 && ni[q] < b.i1 && nj[q] > b.j0 && nj[q] < b.j1;
            if (inside) {
                out[slot[q]] = a[q];
            } else {
                const double t = a[q] * g.u[(size_t)nj[q] * g.n0 + ni[q]];
                out[5] -= t;
                yb -= t;
            }
        }
        double *o = stencil + (b.first + r) * 6;
#pragma unroll
        for (int q = 0; q < 6; ++q) o[q] = out[q];
        aux[(b.first + r) * 2] = f;
        aux[(b.first + r) * 2 + 1] = yb;
    }
}

// Entry e (column r - w + e) of unknown r's row of a subdomain's band matrix.
__device__ __forceinline__ double stage2_entry(const double *st, int w, int e)
{
    double v = 0.0;
    if (e == 0) v += st[0];
    if (e == w - 1) v += st[1];
    if (e == w) v += st[2];
    if (e == w + 1) v += st[3];
    if (e == 2 * w) v += st[4];
    return v;
}

// A lane's double, read by every lane (wave-uniform result).
__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Banded LU without pivoting (the stencil matrices are diagonally dominant
// once h is small enough for the drift) of one subdomain per workgroup: the
// rows of the active window (the pivot row and the w rows below it) stay in
// LDS in a ring of w + 1 slots; a retired pivot row goes to `factor` (its w + 1
// upper entries; stride kStage2MaxBand + 2, the last slot left for the
// eliminated right side), the multipliers l(k + 1 + t, k) of pivot k to
// lmul[k w + t], and the row w + 1 below it takes its slot. The factors depend
// on the operator, the grid and the subdomains only, not on the data on the
// interfaces, so a context keeps them for the next call with the same ones.
constexpr int kStage2LuThreads = 1024;

__global__ void __launch_bounds__(kStage2LuThreads) stage2_lu_kernel(const SubBox *boxes, const double *stencil,
                                                                     double *factor, double *lmul)
{
    constexpr int MW = kStage2MaxBand;
    constexpr int ROW = 2 * MW + 1;
    constexpr int FS = MW + 2;  // factor stride
    constexpr int CH = 64;      // back-substitution chunk
    __shared__ double A[(MW + 1) * ROW];
    __shared__ double lcol[MW];
    __shared__ double S[CH * 6];  // stencils of the rows that the next CH pivots bring into the window
    const SubBox bx = boxes[blockIdx.x];
    const int w = bx.w, R = w + 1;
    const uint64_t n = (uint64_t)w * (uint64_t)bx.L;
    const double *st = stencil + bx.first * 6;
    double *U = factor + bx.first * FS;
    double *Lm = lmul + bx.first * MW;
    const int tid = threadIdx.x;
    for (int idx = tid; idx < R * (2 * w + 1); idx += blockDim.x) {
        const int rr = idx / (2 * w + 1), e = idx % (2 * w + 1);
        A[rr * ROW + e] = (uint64_t)rr < n ? stage2_entry(st + (size_t)rr * 6, w, e) : 0.0;
    }
    // this thread's (row, column) offsets of the w x w update, the same at
    // every pivot: pair m is update idx = tid + T m (T threads), row offset
    // idx / w and column offset idx % w (no division inside the pivot loop)
    constexpr int T = kStage2LuThreads;
    constexpr int kPairs = MW * MW / T;
    static_assert(MW * MW % T == 0, "whole pairs per thread");
    int prr[kPairs], pcc[kPairs];
#pragma unroll
    for (int m = 0; m < kPairs; ++m) {
        const int idx = tid + T * m;
        prr[m] = idx < w * w ? idx / w : -1;
        pcc[m] = idx < w * w ? idx % w : 0;
    }
    int sk = 0;  // slot of pivot row k: k mod R
    for (uint64_t k = 0; k < n; ++k) {
        __syncthreads();
        if (k % CH == 0) {  // rows k + R .. k + R + CH - 1, entering at pivots k .. k + CH - 1
            for (int idx = tid; idx < CH * 6; idx += blockDim.x) {
                const uint64_t q = (k + R) * 6 + idx;
                S[idx] = q < n * 6 ? st[q] : 0.0;
            }
            __syncthreads();
        }
        if (tid < w) {
            const uint64_t r = k + 1 + tid;
            double l = 0.0;
            if (r < n) {
                int sr = sk + 1 + tid;
                if (sr >= R) sr -= R;
                l = A[sr * ROW + (w - 1 - tid)] / A[sk * ROW + w];  // column k of row r: offset k - r + w
            }
            lcol[tid] = l;
            Lm[k * w + tid] = l;
        }
        __syncthreads();
        const uint64_t left = n - 1 - k;  // unknowns after k: rows and columns k + 1 + o exist for o < left
        // all reads first, then the stores: each pair writes its own entry, and
        // the pivot row and multipliers are not written in this phase
        int at[kPairs];
        double upd[kPairs];
#pragma unroll
        for (int m = 0; m < kPairs; ++m) {
            const int rr = prr[m], cc = pcc[m];
            at[m] = -1;
            if (rr >= 0 && (uint64_t)rr < left && (uint64_t)cc < left) {
                int sr = sk + 1 + rr;
                if (sr >= R) sr -= R;
                at[m] = sr * ROW + (cc - rr + w);
                upd[m] = A[at[m]] - lcol[rr] * A[sk * ROW + (cc + 1 + w)];
            }
        }
#pragma unroll
        for (int m = 0; m < kPairs; ++m)
            if (at[m] >= 0) A[at[m]] = upd[m];
        __syncthreads();
        // retire row k (its columns k .. k + w) and load row k + R into its slot
        const uint64_t nr = k + R;
        const double *sn = S + (k % CH) * 6;  // row nr's stencil
        for (int e = tid; e < 2 * w + 1; e += blockDim.x) {
            if (e >= w) U[k * FS + (e - w)] = A[sk * ROW + e];
            A[sk * ROW + e] = nr < n ? stage2_entry(sn, w, e) : 0.0;
        }
        if (++sk == R) sk = 0;
    }
}

// Forward elimination of the right sides (column 5 of the stencils) with the
// stored multipliers, then back substitution, one subdomain per workgroup,
// both in wave 0 with the pending rows in registers: row r's value lives in
// lane r mod w (n = w L, so the w rows of a window fill the lanes). Forward,
// pivot k: its value y_k (final) is broadcast from lane k mod w, that lane
// takes row k + w, and every lane subtracts l(r, k) y_k from its row r in
// k + 1 .. k + w: the products and differences of eliminating the right side
// alongside the factorization, in its order. y_k goes to the right-side slot
// of factor row k. Back, from k = n - 1 down: x_k = (its value) / u(k, k) is
// broadcast, written to u, its lane takes row k - w's y, and every row j in
// k - w .. k - 1 subtracts u(j, k) x_k. Multipliers, entering right sides and
// U rows are staged through LDS in chunks.
constexpr int kStage2SubstThreads = 256;

// dst[i] = src[i] for i < count (count <= PER x the block's threads): each
// thread issues its PER global loads before any LDS store, so that they are
// in flight together rather than one after another.
template <int PER>
__device__ __forceinline__ void stage_chunk(double *dst, const double *src, int count, int tid)
{
    double t[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid + u * kStage2SubstThreads;
        t[u] = i < count ? gload(src + i) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid + u * kStage2SubstThreads;
        if (i < count) dst[i] = t[u];
    }
}

__global__ void __launch_bounds__(kStage2SubstThreads) stage2_subst_kernel(const Stage2Grid g, const SubBox *boxes,
                                                                           const double *stencil, double *factor,
                                                                           const double *lmul)
{
    constexpr int MW = kStage2MaxBand;
    constexpr int FS = MW + 2;  // factor stride
    constexpr int CH = 64;      // pivots (rows) per chunk
    constexpr int PF = 8;       // steps whose operands are read ahead
    __shared__ double Lc[CH * MW];          // forward: multipliers of the chunk's pivots
    __shared__ double Bc[CH];               // forward: right sides entering the window
    __shared__ double Uc[(CH + MW) * FS];   // back: U rows lo - w .. hi - 1
    const SubBox bx = boxes[blockIdx.x];
    const int w = bx.w;
    const uint64_t n = (uint64_t)w * (uint64_t)bx.L;
    const double *st = stencil + bx.first * 6;
    double *U = factor + bx.first * FS;
    const double *Lm = lmul + bx.first * MW;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    double v = tid < 64 && lane < w ? st[(size_t)lane * 6 + 5] : 0.0;  // rows 0 .. w - 1
    int s = 0;  // lane of pivot k: k mod w
    for (uint64_t k0 = 0; k0 < n; k0 += CH) {
        const int m = n - k0 < (uint64_t)CH ? (int)(n - k0) : CH;
        __syncthreads();
        stage_chunk<CH * MW / kStage2SubstThreads>(Lc, Lm + k0 * w, m * w, tid);
        for (int idx = tid; idx < m; idx += blockDim.x) {
            const uint64_t q = k0 + idx + w;  // the row entering the window at pivot k0 + idx
            Bc[idx] = q < n ? st[q * 6 + 5] : 0.0;
        }
        __syncthreads();
        if (tid < 64) {
            double ybuf = 0.0;  // lane i keeps y of pivot k0 + i
            for (int i0 = 0; i0 < m; i0 += PF) {
                // this lane's multipliers and the entering right sides of the
                // next PF pivots, read ahead of the dependent chain
                double lv[PF], bv[PF];
                int su = s;
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    int d = lane - su - 1;  // this lane's row at pivot k0 + i0 + u: k + 1 + d
                    if (d < 0) d += w;
                    const bool ok = i0 + u < m && lane < w && k0 + i0 + u + 1 + d < n;
                    lv[u] = ok ? Lc[(i0 + u) * w + d] : 0.0;
                    bv[u] = i0 + u < m ? Bc[i0 + u] : 0.0;
                    if (++su == w) su = 0;
                }
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    if (i0 + u >= m) break;
                    const double yk = readlane_f64(v, s);
                    ybuf = lane == i0 + u ? yk : ybuf;
                    v = lane == s ? bv[u] : v;
                    const double nv = v - lv[u] * yk;
                    v = lv[u] != 0.0 ? nv : v;  // rows in pivot k's reach (a zero multiplier changes nothing)
                    if (++s == w) s = 0;
                }
            }
            if (lane < m) U[(k0 + lane) * FS + MW + 1] = ybuf;
        }
    }
    // back substitution; rows n - w .. n - 1 fill lanes 0 .. w - 1
    s = w - 1;  // lane of row n - 1
    for (uint64_t hi = n; hi > 0;) {
        const uint64_t lo = hi > CH ? hi - CH : 0;
        const uint64_t base = lo > (uint64_t)w ? lo - w : 0;  // rows base .. hi - 1 staged
        __syncthreads();
        stage_chunk<((CH + MW) * FS + kStage2SubstThreads - 1) / kStage2SubstThreads>(Uc, U + base * FS,
                                                                                      (int)(hi - base) * FS, tid);
        __syncthreads();
        if (tid < 64) {
            if (hi == n) v = lane < w ? Uc[(n - w + lane - base) * FS + MW + 1] : 0.0;
            const int cnt = (int)(hi - lo);
            double xbuf = 0.0;  // lane i keeps x of row hi - 1 - i
            for (int i0 = 0; i0 < cnt; i0 += PF) {
                // rows hi - 1 - i0 - u: the divisor's reciprocal, this lane's
                // entry of the row it updates and the right side entering the
                // window
                double rv[PF], uv[PF], yv[PF];
                int su = s;
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    const uint64_t k = hi - 1 - (uint64_t)(i0 + u);
                    const bool in = i0 + u < cnt;
                    int d = su - 1 - lane;  // this lane's row: k - 1 - d
                    if (d < 0) d += w;
                    rv[u] = 1.0 / (in ? Uc[(k - base) * FS] : 1.0);
                    uv[u] = in && lane < w && k >= (uint64_t)(d + 1) ? Uc[(k - 1 - d - base) * FS + (d + 1)] : 0.0;
                    yv[u] = in && k >= (uint64_t)w ? Uc[(k - w - base) * FS + MW + 1] : 0.0;
                    if (--su < 0) su = w - 1;
                }
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    if (i0 + u >= cnt) break;
                    const double xk = readlane_f64(v, s) * rv[u];
                    xbuf = lane == i0 + u ? xk : xbuf;
                    v = lane == s ? yv[u] : v;
                    const double nv = v - uv[u] * xk;
                    v = uv[u] != 0.0 ? nv : v;
                    if (--s < 0) s = w - 1;
                }
            }
            if (lane < cnt) {
                int i, j;
                stage2_point(bx, hi - 1 - (uint64_t)lane, i, j);
                g.u[(size_t)j * g.n0 + i] = xbuf;
            }
        }
        hi = lo;
    }
}

// Response columns of the subdomains (one workgroup per subdomain and four
// columns, a wave per column): the solution for a unit right side at each
// row next to the box's boundary, and for the source f with zero boundary
// values, by the substitution of stage2_subst_kernel with the stored factors
// (the chunks of multipliers and U rows staged once for the four waves). The
// forward pass leaves y in the column, the backward pass overwrites it with
// the solution.
constexpr int kStage2RespWaves = kStage2SubstThreads / 64;
__global__ void __launch_bounds__(kStage2SubstThreads) stage2_resp_kernel(const SubBox *boxes, const double *aux,
                                                                          const double *factor, const double *lmul,
                                                                          const Stage2Resp *tab, const uint32_t *rb,
                                                                          double *resp)
{
    constexpr int MW = kStage2MaxBand;
    constexpr int FS = MW + 2;
    constexpr int CH = 64;
    constexpr int PF = 8;
    constexpr int NW = kStage2RespWaves;
    __shared__ double Lc[CH * MW];
    __shared__ double Bc[NW][CH];
    __shared__ double Uc[(CH + MW) * FS];
    __shared__ double Yc[NW][CH + MW];
    const SubBox bx = boxes[blockIdx.x];
    const Stage2Resp rt = tab[blockIdx.x];
    const int w = bx.w;
    const uint64_t n = (uint64_t)w * (uint64_t)bx.L;
    const double *U = factor + bx.first * FS;
    const double *Lm = lmul + bx.first * MW;
    const double *fa = aux + bx.first * 2;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int col = (int)blockIdx.y * NW + wv;
    const bool act = col <= rt.nb;
    const bool src = col == rt.nb;  // the source column
    const uint64_t rc = act && !src ? rb[rt.rb_at + col] : ~0ull;
    double *out = resp + rt.out_at + (uint64_t)(act ? col : 0) * n;
    auto rhs = [&](uint64_t q) { return src ? fa[q * 2] : (q == rc ? 1.0 : 0.0); };
    double v = act && lane < w ? rhs((uint64_t)lane) : 0.0;
    int s = 0;
    for (uint64_t k0 = 0; k0 < n; k0 += CH) {
        const int m = n - k0 < (uint64_t)CH ? (int)(n - k0) : CH;
        __syncthreads();
        stage_chunk<CH * MW / kStage2SubstThreads>(Lc, Lm + k0 * w, m * w, tid);
        for (int idx = lane; idx < m; idx += 64) {
            const uint64_t q = k0 + idx + w;
            Bc[wv][idx] = act && q < n ? rhs(q) : 0.0;
        }
        __syncthreads();
        if (act) {
            double ybuf = 0.0;
            for (int i0 = 0; i0 < m; i0 += PF) {
                double lv[PF], bv[PF];
                int su = s;
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    int d = lane - su - 1;
                    if (d < 0) d += w;
                    const bool ok = i0 + u < m && lane < w && k0 + i0 + u + 1 + d < n;
                    lv[u] = ok ? Lc[(i0 + u) * w + d] : 0.0;
                    bv[u] = i0 + u < m ? Bc[wv][i0 + u] : 0.0;
                    if (++su == w) su = 0;
                }
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    if (i0 + u >= m) break;
                    const double yk = readlane_f64(v, s);
                    ybuf = lane == i0 + u ? yk : ybuf;
                    v = lane == s ? bv[u] : v;
                    const double nv = v - lv[u] * yk;
                    v = lv[u] != 0.0 ? nv : v;
                    if (++s == w) s = 0;
                }
            }
            if (lane < m) out[k0 + lane] = ybuf;
        }
    }
    s = w - 1;
    for (uint64_t hi = n; hi > 0;) {
        const uint64_t lo = hi > CH ? hi - CH : 0;
        const uint64_t base = lo > (uint64_t)w ? lo - w : 0;
        __syncthreads();
        stage_chunk<((CH + MW) * FS + kStage2SubstThreads - 1) / kStage2SubstThreads>(Uc, U + base * FS,
                                                                                      (int)(hi - base) * FS, tid);
        for (int idx = lane; idx < (int)(hi - base); idx += 64) Yc[wv][idx] = act ? gload(out + base + idx) : 0.0;
        __syncthreads();
        if (act) {
            if (hi == n) v = lane < w ? Yc[wv][n - w + lane - base] : 0.0;
            const int cnt = (int)(hi - lo);
            double xbuf = 0.0;
            for (int i0 = 0; i0 < cnt; i0 += PF) {
                double rv[PF], uv[PF], yv[PF];
                int su = s;
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    const uint64_t k = hi - 1 - (uint64_t)(i0 + u);
                    const bool in = i0 + u < cnt;
                    int d = su - 1 - lane;
                    if (d < 0) d += w;
                    rv[u] = 1.0 / (in ? Uc[(k - base) * FS] : 1.0);
                    uv[u] = in && lane < w && k >= (uint64_t)(d + 1) ? Uc[(k - 1 - d - base) * FS + (d + 1)] : 0.0;
                    yv[u] = in && k >= (uint64_t)w ? Yc[wv][k - w - base] : 0.0;
                    if (--su < 0) su = w - 1;
                }
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    if (i0 + u >= cnt) break;
                    const double xk = readlane_f64(v, s) * rv[u];
                    xbuf = lane == i0 + u ? xk : xbuf;
                    v = lane == s ? yv[u] : v;
                    const double nv = v - uv[u] * xk;
                    v = uv[u] != 0.0 ? nv : v;
                    if (--s < 0) s = w - 1;
                }
            }
            if (lane < cnt) out[hi - 1 - lane] = xbuf;
        }
        hi = lo;
    }
}

// Interior values from the response columns: u = (f's column) + sum over the
// rows next to the boundary of (that row's column) x (its boundary part of
// the right side), in row order; one thread per unknown.
__global__ void __launch_bounds__(256) stage2_apply_kernel(const Stage2Grid g, const SubBox *boxes, const double *aux,
                                                           const Stage2Resp *tab, const uint32_t *rb,
                                                           const double *resp)
{
    __shared__ double yb[kStage2MaxBoundaryRows];
    const SubBox bx = boxes[blockIdx.y];
    const Stage2Resp rt = tab[blockIdx.y];
    const uint64_t n = (uint64_t)bx.w * (uint64_t)bx.L;
    for (int c = threadIdx.x; c < rt.nb; c += blockDim.x) yb[c] = aux[(bx.first + rb[rt.rb_at + c]) * 2 + 1];
    __syncthreads();
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const double *col = resp + rt.out_at + r;
        double acc = col[(uint64_t)rt.nb * n];
        for (int c = 0; c < rt.nb; ++c) acc = fma(col[(uint64_t)c * n], yb[c], acc);
        int i, j;
        stage2_point(bx, r, i, j);
        g.u[(size_t)j * g.n0 + i] = acc;
    }
}

}  // namespace

hipError_t launch_grid_residual(const DevProblem<double> &P, double sigma, const pdd_grid *g, void *r, hipStream_t s)
{
    const int D = g->dim;
    const int n2 = D == 3 ? g->n[2] : 1;
    const uint64_t total = (uint64_t)g->n[0] * g->n[1] * n2;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((total + 255) / 256, 16384);
    double dx[3] = {0, 0, 0};
    for (int d = 0; d < D; ++d) dx[d] = (g->hi[d] - g->lo[d]) / (g->n[d] - 1);
    const double h2 = 0.5 * sigma * sigma;
    if (g->dtype == PDD_DTYPE_F32) {
        const float *u = static_cast<const float *>(g->data);
        float *out = static_cast<float *>(r);
        if (D == 2)
            hipLaunchKernelGGL((grid_residual_kernel<float, 2>), dim3(blocks), dim3(256), 0, s, P, u, g->n[0], g->n[1],
                               n2, g->lo[0], g->lo[1], 0.0, dx[0], dx[1], 0.0, h2, out);
        else
            hipLaunchKernelGGL((grid_residual_kernel<float, 3>), dim3(blocks), dim3(256), 0, s, P, u, g->n[0], g->n[1],
                               n2, g->lo[0], g->lo[1], g->lo[2], dx[0], dx[1], dx[2], h2, out);
    } else {
        const double *u = static_cast<const double *>(g->data);
        double *out = static_cast<double *>(r);
        if (D == 2)
            hipLaunchKernelGGL((grid_residual_kernel<double, 2>), dim3(blocks), dim3(256), 0, s, P, u, g->n[0],
                               g->n[1], n2, g->lo[0], g->lo[1], 0.0, dx[0], dx[1], 0.0, h2, out);
        else
            hipLaunchKernelGGL((grid_residual_kernel<double, 3>), dim3(blocks), dim3(256), 0, s, P, u, g->n[0],
                               g->n[1], n2, g->lo[0], g->lo[1], g->lo[2], dx[0], dx[1], dx[2], h2, out);
    }
    return hipGetLastError();
}

hipError_t launch_stage2_boundary(const DevProblem<double> &P, const Stage2Grid &g, hipStream_t s)
{
    const int total = 2 * g.n0 + 2 * (g.n1 - 2);
    hipLaunchKernelGGL(stage2_boundary_kernel, dim3((total + 255) / 256), dim3(256), 0, s, P, g);
    return hipGetLastError();
}

hipError_t launch_stage2_lines(const Stage2Grid &g, const Stage2Line *lines, int32_t n_lines, const double *t,
                               const double *lam, hipStream_t s)
{
    if (n_lines == 0) return hipSuccess;
    const int len = g.n0 > g.n1 ? g.n0 : g.n1;
    hipLaunchKernelGGL(stage2_lines_kernel, dim3((len + 255) / 256, n_lines), dim3(256), 0, s, g, lines, n_lines, t,
                       lam);
    return hipGetLastError();
}

hipError_t launch_stage2_solve(const DevProblem<double> &P, const Stage2Grid &g, const SubBox *boxes,
                               int32_t n_boxes, uint32_t max_unknowns, double *stencil, double *aux, double *factor,
                               double *lmul, const Stage2Plan &plan, hipStream_t s)
{
    if (n_boxes == 0) return hipSuccess;
    hipLaunchKernelGGL(stage2_stencil_kernel, dim3((max_unknowns + 255) / 256, n_boxes), dim3(256), 0, s, P, g,
                       boxes, stencil, aux);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!plan.factored) {
        hipLaunchKernelGGL(stage2_lu_kernel, dim3(n_boxes), dim3(kStage2LuThreads), 0, s, boxes, stencil, factor,
                           lmul);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (!plan.resp) {
        hipLaunchKernelGGL(stage2_subst_kernel, dim3(n_boxes), dim3(kStage2SubstThreads), 0, s, g, boxes, stencil,
                           factor, lmul);
        return hipGetLastError();
    }
    if (!plan.resp_ready) {
        const uint32_t groups = (uint32_t)(plan.max_cols + kStage2RespWaves - 1) / kStage2RespWaves;
        hipLaunchKernelGGL(stage2_resp_kernel, dim3(n_boxes, groups), dim3(kStage2SubstThreads), 0, s, boxes, aux,
                           factor, lmul, plan.resp_tab, plan.rb, plan.resp);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((max_unknowns + 255) / 256, 1024);
    hipLaunchKernelGGL(stage2_apply_kernel, dim3(blocks, n_boxes), dim3(256), 0, s, g, boxes, aux, plan.resp_tab,
                       plan.rb, plan.resp);
    return hipGetLastError();
}

}  // namespace pdd
