// Kernels of the outer iteration that evaluate the problem's coefficients: the
// residual of a gridded u~ and the second stage of PDD.
#include <algorithm>
#include <type_traits>

#include "path_walk.hpp"

namespace pdd {
namespace {

// First and second derivative along one axis at point p, whose index there is
// a of n (stride st): central inside, one-sided at the two ends.
template <class S, class I>
__device__ __forceinline__ void fd(const S *__restrict__ u, I p, double u0, I st, int a, int n, double dx, double &first,
                                   double &second)
{
    const bool low = a == 0, high = a == n - 1;
    // the point before and the point after, or at an end the next two inwards
    const double v1 = (double)u[low ? p + st : p - st];
    const double v2 = (double)u[low ? p + 2 * st : high ? p - 2 * st : p + st];
    double n1 = v2 - v1, n2 = v2 - 2.0 * u0 + v1;
    if (low || high) {
        const double v3 = (double)u[low ? p + 3 * st : p - 3 * st];
        n1 = low ? -3.0 * u0 + 4.0 * v1 - v2 : 3.0 * u0 - 4.0 * v1 + v2;
        n2 = 2.0 * u0 - 5.0 * v1 + 4.0 * v2 - v3;
    }
    first = n1 / (2.0 * dx);
    second = n2 / (dx * dx);
}

// Residual r = f - ((1/2) sigma^2 Lap u + b.grad u + c u) of a gridded u at
// its points, b, c, f from the problem (FP64), the derivatives of u by
// second-order differences (central inside; three-point one-sided first and
// four-point one-sided second derivatives at the ends of each axis).
// I: the type that holds a point's number (a division by a 64-bit grid size
// costs more than the derivatives). TAB: the problem has tabulated coefficients
// or trig arguments that need the library's reduction. Bound by the source's
// FP64 functions. 513^2 FP64 points 8.3 us, 5.4 us with 32-bit numbers, all
// loads first and the analytic form; 2049^2 61 and 41 us (67 MB: 14 us at the
// rate of a copy); 129^3 FP32 131 and 87 us.
template <class S, int D, class I, bool TAB>
__global__ void __launch_bounds__(256) grid_residual_kernel(const DevProblem<double> P, const S *__restrict__ u,
                                                            int n0, int n1, int n2, double lo0, double lo1,
                                                            double lo2, double dx0, double dx1, double dx2,
                                                            double half_s2, S *__restrict__ r)
{
    __shared__ double s_cf[kMaxDense];
    for (int q = threadIdx.x; q < kMaxDense; q += blockDim.x) s_cf[q] = P.fdense[q];
    __syncthreads();
    const I m01 = (I)n0 * n1, total = m01 * (D == 3 ? n2 : 1);
    const int nn[3] = {n0, n1, n2};
    MathOf<double> mt;
    mt.init();
    const double lo[3] = {lo0, lo1, lo2}, dx[3] = {dx0, dx1, dx2};
    const I st[3] = {1, (I)n0, m01};
    for (I p = blockIdx.x * (I)blockDim.x + threadIdx.x; p < total; p += (I)gridDim.x * blockDim.x) {
        const I jk = p / n0;
        const int k = D == 3 ? (int)(jk / n1) : 0;
        const int idx[3] = {(int)(p - jk * n0), D == 3 ? (int)(jk - (I)k * n1) : (int)jk, k};
        const double u0 = (double)u[p];
        double x[D], first[D], second[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            x[d] = lo[d] + (double)idx[d] * dx[d];
            fd<S, I>(u, p, u0, st[d], idx[d], nn[d], dx[d], first[d], second[d]);
        }
        double b[D], c, f = 0.0;
        coefficients<double, D, TAB>(mt, P, x, b, c, f, true, s_cf, TAB ? P.tab : 0u);
        double lap = 0.0, adv = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            lap += second[d];
            adv += b[d] * first[d];
        }
        r[p] = (S)(f - (half_s2 * lap + adv + c * u0));
    }
}

template <class S, int D, bool TAB>
hipError_t launch_residual(const DevProblem<double> &P, double sigma, const pdd_grid *g, void *r, hipStream_t s)
{
    const int n2 = D == 3 ? g->n[2] : 1;
    const uint64_t total = (uint64_t)g->n[0] * g->n[1] * n2;
    // four workgroups per CU: what a wave loads before its first point (the
    // problem, the functions' coefficients) is shared by more points (2049^2
    // points 49 us with a workgroup per 256 points, 41 us so)
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((total + 255) / 256, 1024);
    double dx[3] = {0, 0, 0};
    for (int d = 0; d < D; ++d) dx[d] = (g->hi[d] - g->lo[d]) / (g->n[d] - 1);
    // (2^31: a thread's next point still fits in 32 bits)
    const auto kernel = total < (1ull << 31) ? grid_residual_kernel<S, D, uint32_t, TAB>
                                               : grid_residual_kernel<S, D, uint64_t, TAB>;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, P, static_cast<const S *>(g->data), g->n[0], g->n[1], n2,
                       g->lo[0], g->lo[1], D == 3 ? g->lo[2] : 0.0, dx[0], dx[1], dx[2], 0.5 * sigma * sigma,
                       static_cast<S *>(r));
    return hipGetLastError();
}

// Second stage (the subdomain-BVP step of Alg. A:IterPDD) on a 2D box cut by
// axis-parallel interfaces. Grid coordinates are lo + span i / (n - 1), as
// everywhere the grids are sampled.
__device__ __forceinline__ double stage2_coord(double lo, double span, int n, int i)
{
    return lo + span * (double)i / (double)(n - 1);
}

// g at point q of the box's edges.
__device__ __forceinline__ void stage2_edge_point(const DevProblem<double> &P, const Stage2Grid &g, const MathOf<double> &mt,
                                                  int q)
{
    const int n0 = g.n0, n1 = g.n1;
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

__device__ __forceinline__ double multiquadric(const double *t, const double *lam, int m, double eps, double x)
{
    double acc = 0.0;
    for (int q = 0; q < m; ++q) {
        const double e = eps * (x - t[q]);
        acc += lam[q] * sqrt(1.0 + e * e);
    }
    return acc;
}

// A lane's double, read by every lane (wave-uniform result).
__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The largest of v over the wave (NaN apart), by way of the rows of 16 lanes.
__device__ __forceinline__ double wave_max(double v)
{
    const auto step = [&v](auto ctrl) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)(b >> 32);
        const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, decltype(ctrl)::value, 0xf, 0xf, false);
        const uint32_t h = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, decltype(ctrl)::value, 0xf, 0xf, false);
        v = fmax(v, __builtin_bit_cast(double, (uint64_t)h << 32 | l));
    };
    step(std::integral_constant<int, 0x111>{});  // from 1, 2, 4 and 8 lanes before
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    step(std::integral_constant<int, 0x142>{});  // the last lane of a row to the next row
    step(std::integral_constant<int, 0x143>{});  // lane 31 to the upper half
    return readlane_f64(v, 63);
}

// Multiquadric weights of one line, one workgroup each: Phi lam = z by Gaussian
// elimination with partial pivoting, Phi and, as its last column, z in LDS up to
// kStage2MaxLdsNodes data points (149 KB), else in device memory; false if it is
// singular. The elimination's operations on each element, and its pivots, are
// those of the textbook loop. Bound by its chain of pivots, three barriers and a
// division each; up to kWeightsOneWave points (strips have some eight) ONE wave
// goes through them without barriers. 14 lines of 114 points: a second stage of
// 257^2 points with kept factors took 2.1 ms with the systems solved on the host
// and takes 0.35 ms.
constexpr int kWeightsThreads = 1024, kWeightsOneWave = 16;
template <bool ONE>
__device__ __forceinline__ void weights_sync()
{
    if constexpr (ONE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}
template <bool ONE>
__device__ __forceinline__ bool solve_weights(double *M, double *z, double first, double last, const double *t,
                                              double eps, int m)
{
    constexpr int kThreads = ONE ? 64 : kWeightsThreads;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // rows and columns of a thread in the matrix
    const int row = ONE ? lane >> 3 : wave, col = ONE ? lane & 7 : lane;
    constexpr int kRows = ONE ? 8 : kThreads / 64, kCols = ONE ? 8 : 64;
    const size_t ld = m + 1;
    for (int r = row; r < m; r += kRows)
        for (int c = col; c <= m; c += kCols) {
            const double ee = eps * (t[r] - (c < m ? t[c] : 0.0));
            M[r * ld + c] = c < m ? sqrt(1.0 + ee * ee) : r == 0 ? first : r == m - 1 ? last : z[r];
        }
    weights_sync<ONE>();
    for (int c = 0; c < m; ++c) {
        // the largest |entry| of the column from the diagonal on, the first of
        // equals; every wave finds it for itself
        double best = -1.0;
        for (int r = c + lane; r < m; r += 64) best = fmax(best, fabs(M[r * ld + c]));
        best = wave_max(best);
        int p = c;
        for (int r0 = c; r0 < m; r0 += 64) {
            const int r = r0 + lane;
            const uint64_t hit = __ballot(r < m && fabs(M[(r < m ? r : c) * ld + c]) == best);
            if (hit) {
                p = r0 + __builtin_ctzll(hit);
                break;
            }
        }
        const double pivot = M[p * ld + c];
        weights_sync<ONE>();
        if (pivot == 0.0) return false;  // every wave alike
        // rows c and p change places; their multipliers take the entries of
        // column c below the diagonal (row p's is of the row that came there)
        if (threadIdx.x < kThreads / 2) {
            for (int cc = c + 1 + threadIdx.x; cc <= m; cc += kThreads / 2) {
                const double v = M[p * ld + cc];
                M[p * ld + cc] = M[c * ld + cc];
                M[c * ld + cc] = v;
            }
        } else {
            for (int r = c + threadIdx.x - kThreads / 2; r < m; r += kThreads / 2) {
                if (r == c && p != c) continue;
                const double v = M[(r == p ? c : r) * ld + c];
                if (r == p) M[c * ld + c] = pivot;
                if (r > c) M[r * ld + c] = v / pivot;
            }
        }
        weights_sync<ONE>();
        for (int cc = c + 1 + col; cc <= m; cc += kCols) {
            const double top = M[c * ld + cc];
            for (int r = c + 1 + row; r < m; r += kRows) M[r * ld + cc] -= M[r * ld + c] * top;
        }
        weights_sync<ONE>();
    }
    for (int r = m - 1; r >= 0; --r) {
        if (wave * 64 > r) {
            weights_sync<ONE>();
            continue;
        }
        const double x = M[r * ld + m] / M[r * ld + r];
        if (threadIdx.x == 0) z[r] = x;
        for (int rr = threadIdx.x; rr < r; rr += kThreads) M[rr * ld + m] -= M[rr * ld + r] * x;
        weights_sync<ONE>();
    }
    return true;
}
// One workgroup per line (its weights, then its values between the box's edges
// into g.lines), the ones after them for the box's edges, and for the tables'
// way to the device. Lines and their data are read where the host put them: a copy
// ahead of the kernel cost a call with kept factors 5 us.
__global__ void __launch_bounds__(kWeightsThreads) stage2_edges_kernel(const DevProblem<double> P, const Stage2Grid g,
                                                                       const Stage2Edges a)
{
    __shared__ double s_M[kStage2MaxLdsNodes * (kStage2MaxLdsNodes + 1)];
    __shared__ double s_t[kStage2MaxLdsNodes], s_z[kStage2MaxLdsNodes], ends[2];
    __shared__ bool solved;
    const int tid = threadIdx.x, edge_blocks = (2 * (g.n0 + g.n1 - 2) + kWeightsThreads - 1) / kWeightsThreads;
    if ((int)blockIdx.x >= a.n_lines + edge_blocks) {  // whole workgroup, as below
        const uint64_t blocks = gridDim.x - a.n_lines - edge_blocks;
        for (uint64_t w = (blockIdx.x - a.n_lines - edge_blocks) * (uint64_t)kWeightsThreads + tid; w < a.table_words;
             w += blocks * kWeightsThreads)
            a.table[w] = a.host_table[w];
        return;
    }
    MathOf<double> mt;
    mt.init();
    if ((int)blockIdx.x >= a.n_lines) {
        const int q = ((int)blockIdx.x - a.n_lines) * kWeightsThreads + tid;
        if (q < 2 * (g.n0 + g.n1 - 2)) stage2_edge_point(P, g, mt, q);
        return;
    }
    const Stage2Line L = a.host_lines[blockIdx.x];
    const bool in_lds = L.m <= kStage2MaxLdsNodes;
    double *t = in_lds ? s_t : a.t + L.at, *z = in_lds ? s_z : a.lam + L.at;
    for (int q = tid; q < L.m; q += kWeightsThreads) {
        t[q] = a.host_t[L.at + q];
        z[q] = a.host_z[L.at + q];
    }
    if (tid < 2) {
        const int e = tid ? (L.d == 0 ? g.n1 : g.n0) - 1 : 0;  // along the line
        const int i = L.d == 0 ? L.k : e, j = L.d == 0 ? e : L.k;
        const double x[2] = {stage2_coord(g.lo0, g.span0, g.n0, i), stage2_coord(g.lo1, g.span1, g.n1, j)};
        ends[tid] = boundary_value<double, 2, true>(mt, P, x, P.tab);
    }
    __syncthreads();
    if (L.m <= kWeightsOneWave) {
        if (tid < 64) {
            const bool ok = solve_weights<true>(s_M, s_z, ends[0], ends[1], s_t, L.eps, L.m);
            if (tid == 0) solved = ok;
        }
    } else {
        const bool ok = in_lds ? solve_weights<false>(s_M, s_z, ends[0], ends[1], s_t, L.eps, L.m)
                               : solve_weights<false>(a.matrices + L.matrix, z, ends[0], ends[1], t, L.eps, L.m);
        if (tid == 0) solved = ok;
    }
    __syncthreads();
    if (tid == 0) {
        g.line_failed[blockIdx.x] = solved ? 0 : 1;
        if (!solved) a.host_marks[blockIdx.x] = 1;
    }
    if (!solved) return;
    const int ne = L.d == 0 ? g.n1 : g.n0;  // points along the line
    double *out = g.lines + (size_t)blockIdx.x * g.line_stride;
    for (int p = 1 + tid; p < ne - 1; p += kWeightsThreads) {
        const double tp = L.d == 0 ? stage2_coord(g.lo1, g.span1, g.n1, p) : stage2_coord(g.lo0, g.span0, g.n0, p);
        out[p] = in_lds ? multiquadric(s_t, s_z, L.m, L.eps, tp) : multiquadric(t, z, L.m, L.eps, tp);
    }
}

// Line q's points into u, by one workgroup (one where an axis-0 and an axis-1 line
// cross by the axis-0 line).
__device__ __forceinline__ void stage2_line_to_grid(const Stage2Grid &g, const Stage2Line *lines, int32_t n_lines, int q)
{
    const Stage2Line L = lines[q];
    const int ne = L.d == 0 ? g.n1 : g.n0;
    for (int p = 1 + threadIdx.x; p < ne - 1; p += blockDim.x) {
        int cross = -1;  // a line of the other axis through this point
        for (int c = 0; c < n_lines; ++c)
            if (lines[c].d != L.d && lines[c].k == p) cross = c;
        if (cross >= 0 && L.d == 1) continue;
        double v = g.lines[(size_t)q * g.line_stride + p];
        if (cross >= 0) v = 0.5 * (v + g.lines[(size_t)cross * g.line_stride + L.k]);
        g.u[L.d == 0 ? (size_t)p * g.n0 + L.k : (size_t)L.k * g.n0 + p] = v;
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
// 2 centre, 3 fast+1, 4 slow+1, 5 right side, which also goes to rhs; with
// `parts`, f and the boundary values' part go there instead, two values per
// unknown. *not_dominant (if given) is set where a neighbour's coefficient is
// negative or c positive. The last workgroup of every row writes interface lines
// into u.
__global__ void __launch_bounds__(256) stage2_stencil_kernel(const DevProblem<double> P, const Stage2Grid g,
                                                             const SubBox *boxes, const Stage2Line *lines,
                                                             int32_t n_lines, double *stencil, double *rhs, bool parts,
                                                             int32_t *not_dominant)
{
    __shared__ double s_cf[kMaxDense];
    if (blockIdx.x == gridDim.x - 1) {  // whole workgroup
        int32_t failed = 0;
        for (int q = 0; q < n_lines; ++q) failed |= g.line_failed[q];
        if (blockIdx.y == 0 && threadIdx.x == 0) *g.failed = failed;
        for (int q = blockIdx.y; q < n_lines && !failed; q += gridDim.y) stage2_line_to_grid(g, lines, n_lines, q);
        return;
    }
    for (int q = threadIdx.x; q < kMaxDense; q += blockDim.x) s_cf[q] = P.fdense[q];
    __syncthreads();
    const SubBox b = boxes[blockIdx.y];
    MathOf<double> mt;
    mt.init();
    const uint64_t n = (uint64_t)b.w * (uint64_t)b.L;
    const double cx = g.half_s2 / (g.dx0 * g.dx0), cy = g.half_s2 / (g.dx1 * g.dx1);
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (gridDim.x - 1) * (uint64_t)blockDim.x) {
        int i, j;
        stage2_point(b, r, i, j);
        const double x[2] = {stage2_coord(g.lo0, g.span0, g.n0, i), stage2_coord(g.lo1, g.span1, g.n1, j)};
        double bb[2], c, f = 0.0;
        coefficients<double, 2, true>(mt, P, x, bb, c, f, true, s_cf, P.tab);
        const double aW = cx - bb[0] / (2.0 * g.dx0), aE = cx + bb[0] / (2.0 * g.dx0);
        const double aS = cy - bb[1] / (2.0 * g.dx1), aN = cy + bb[1] / (2.0 * g.dx1);
        double out[6] = {0.0, 0.0, -2.0 * cx - 2.0 * cy + c, 0.0, 0.0, f};
        double yb = 0.0;
        if (not_dominant && !(aW >= 0.0 && aE >= 0.0 && aS >= 0.0 && aN >= 0.0 && c <= 0.0)) *not_dominant = 1;
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
                const double t = a[q] * (b.side[q] < 0 ? g.u[(size_t)nj[q] * g.n0 + ni[q]]
                                                       : g.lines[b.side[q] * (size_t)g.line_stride + (q < 2 ? j : i)]);
                out[5] -= t;
                yb -= t;
            }
        }
        double *o = stencil + (b.first + r) * 6;
#pragma unroll
        for (int q = 0; q < 6; ++q) o[q] = out[q];
        if (parts) {
            rhs[(b.first + r) * 2] = f;
            rhs[(b.first + r) * 2 + 1] = yb;
        } else {
            rhs[b.first + r] = out[5];
        }
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
    if (*g.failed) return;
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
    if (*g.failed) return;
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

// Block cyclic reduction of the subdomains. In the order r = s w + f a
// subdomain's matrix is block tridiagonal: L block rows of w x w blocks D
// (tridiagonal), and diagonal blocks A (to row s - 1) and C (to row s + 1).
// With block rows numbered 1 .. L, level l (t = 2^l) eliminates the odd
// multiples i of t,
//   x_i = D_i^-1 f_i - P_i x_{i-t} - Q_i x_{i+t},  P = D^-1 A, Q = D^-1 C,
// from the even ones, which become a block tridiagonal system again:
//   D_i -= A_i Q_{i-t} + C_i P_{i+t},  A_i <- -A_i P_{i-t},  C_i <- -C_i Q_{i+t},
//   f_i -= M_i f_{i-t} + N_i f_{i+t},  M_i = A_i D_{i-t}^-1,  N_i = C_i D_{i+t}^-1,
// until one block row is left. No pivoting, as in the banded LU; but the
// inverses of the D and the products with them are formed, and these grow where
// the matrix is far from diagonally dominant: strips of 63 x 63 unknowns with
// |b| dx / sigma^2 = 2e3 come out 1e-8 from exact (the LU 3e-12), with 2e5 0.1
// (3e-8); c = 83.5 on a strip of 1/4 x 1, near its first eigenvalue, 9e-12
// (4e-13). So this is for matrices of the kind -(M-matrix) with row sums that
// are not positive, of which every D is again one and |P| and |Q| row sums add
// up to at most 1: |b_d| dx_d <= sigma^2 and c <= 0 at every unknown. The other
// ones are factored by the banded LU. The LU's chain of w L dependent
// pivots, one workgroup a subdomain, becomes 1 + log2 L levels whose rows are
// independent. Four strips of 63 x 255 unknowns: 39.9 ms with the LU and the
// solutions for unit boundary values that it was kept as, 0.50 ms now; with
// the factors kept 0.26 and 0.12 ms. What bounds a level is the inversion
// (24 us: 64 dependent pivots) and the products on the FP64 matrix cores
// (9 us; 37 us where the rows are several per CU). Blocks are padded by the
// identity to WP (a multiple of 16, the same for a run of subdomains) and kept by
// column: D (D^-1 once eliminated), P, Q of every row (D's rounding in P's place
// before), and M, N and the new A,
// C of every (row, level); level 0, whose A and C are diagonal, has no P, Q, M
// and N (stored all the same they took 32 us of 0.48 ms).
template <int WP>
struct CrBox {
    static constexpr int kBlock = WP * WP;
    SubBox b;
    Stage2Cr c;
    __device__ __forceinline__ CrBox(const SubBox *boxes, const Stage2Cr *tab, int q) : b(boxes[q]), c(tab[q]) {}
    // D (or D^-1), P, Q of block row i (from 1)
    __device__ __forceinline__ double *row(double *cr, int i) const { return cr + c.at + (size_t)(i - 1) * 3 * kBlock; }
    // M, N, A, C of the m-th even multiple (from 1) of level l
    __device__ __forceinline__ double *pair(double *cr, int l, int m) const
    {
        int before = 0;
        for (int q = 0; q < l; ++q) before += b.L >> (q + 1);
        return cr + c.mn + (size_t)(before + m - 1) * 4 * kBlock;
    }
    // stencil slot q of unknown f of block row i
    __device__ __forceinline__ double slot(const double *stencil, int i, int f, int q) const
    {
        return f < b.w ? stencil[(b.first + (uint64_t)(i - 1) * b.w + f) * 6 + q] : 0.0;
    }
    __device__ __forceinline__ double centre(const double *stencil, int i, int r, int k) const
    {
        if (r >= b.w || k >= b.w) return r == k ? 1.0 : 0.0;
        return r == k ? slot(stencil, i, r, 2) : r == k + 1 ? slot(stencil, i, r, 1)
               : r + 1 == k ? slot(stencil, i, r, 3) : 0.0;
    }
};

constexpr int kCrThreads = 1024;
constexpr int kCrWaves = kCrThreads / 64;
typedef double Acc4 __attribute__((ext_vector_type(4)));

// A block (by column) to registers, and from there to LDS.
template <int WP>
struct CrCopy {
    static constexpr int kPer = (WP * WP + kCrThreads - 1) / kCrThreads;
    double t[kPer];
    __device__ __forceinline__ void fetch(const double *src)
    {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = threadIdx.x + u * kCrThreads;
            t[u] = e < WP * WP ? gload(src + e) : 0.0;
        }
    }
    __device__ __forceinline__ void put(double *dst) const
    {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = threadIdx.x + u * kCrThreads;
            if (e < WP * WP) dst[(e / WP) * (WP + 1) + e % WP] = t[u];
        }
    }
};
template <int WP>
__device__ __forceinline__ void cr_stage(double *dst, const double *src)
{
    CrCopy<WP> c;
    c.fetch(src);
    c.put(dst);
}

// 16 x 16 tile (ti, tj) of acc + sign X Y on the matrix cores, X and Y in LDS.
// The tile is formed transposed, so that a lane's four values are of columns
// 16 tj + 4 v + lane / 16 and of row 16 ti + lane % 16: stores run along rows.
template <int WP>
__device__ __forceinline__ Acc4 cr_tile(const double *X, const double *Y, int ti, int tj, double sign, Acc4 acc)
{
    const int lane = threadIdx.x & 63, low = lane & 15, high = lane >> 4;
    const double *x = X + high * (WP + 1) + ti * 16 + low, *y = Y + (tj * 16 + low) * (WP + 1) + high;
#pragma unroll
    for (int k = 0; k < WP; k += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sign * y[k], x[k * (WP + 1)], acc, 0, 0, 0);
    return acc;
}
template <int WP>
__device__ __forceinline__ double *cr_element(double *block, int ti, int tj, int v)
{
    const int lane = threadIdx.x & 63;
    return block + (tj * 16 + 4 * v + (lane >> 4)) * WP + ti * 16 + (lane & 15);
}

// a + b, and what its rounding left out.
__device__ __forceinline__ double cr_add(double a, double b, double &lost)
{
    const double s = a + b, c = s - a;
    lost = (a - (s - c)) + (b - c);
    return s;
}

// What rounds a value v, |v| <= most, to a multiple of 2^-22 of the next power
// of two above `most`: (v + u) - u for this u.
__device__ __forceinline__ double cr_rounder(double most)
{
    return __builtin_ldexp(1.5, __builtin_amdgcn_frexp_exp(most) + 30);
}

// 16 x 16 tile of acc - (D + S) X, D, S (D's rounding) and X in LDS, nearly as if
// summed exactly: with D + S = D1 + D2 and X = X1 + X2 (D1, X1 of 23 bits each
// against the largest values) every partial sum of acc - D1 X1 is exact, acc
// being that of I, and the rest is 2^-22 of it.
template <int WP>
__device__ __forceinline__ Acc4 cr_residual_tile(const double *D, const double *S, const double *X, int ti, int tj,
                                                 double ud, double ux, Acc4 acc)
{
    const int lane = threadIdx.x & 63, low = lane & 15, high = lane >> 4;
    const double *d = D + high * (WP + 1) + ti * 16 + low, *x = X + (tj * 16 + low) * (WP + 1) + high;
    const double *l = S + (d - D);
#pragma unroll 4
    for (int k = 0; k < WP; k += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-((x[k] + ux) - ux), (d[k * (WP + 1)] + ud) - ud, acc, 0, 0, 0);
#pragma unroll 2
    for (int k = 0; k < WP; k += 4) {
        const double d1 = (d[k * (WP + 1)] + ud) - ud, d2 = (d[k * (WP + 1)] - d1) + l[k * (WP + 1)];
        const double x1 = (x[k] + ux) - ux, x2 = x[k] - x1;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-x2, d1, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-x1, d2, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-x2, d2, acc, 0, 0, 0);
    }
    return acc;
}

// D^-1, P and Q (D^-1 alone at the FIRST level) of the odd multiples of
// 2^level, one workgroup each. D is inverted in registers: lane r of wave q
// holds columns 4 q .. 4 q + 3 of row r. The pivots of a wave's columns are its
// own work, without a barrier (row k comes from lane k); their multipliers then
// go to the other waves through LDS: one barrier per four pivots. (32 us a
// level with one per pivot, 27 us with eight waves of eight columns, 24 us so.)
// Rows are left unscaled until the end. At the lower levels one Newton step,
// X + X (I - D X), then takes out the elimination's rounding: the rows of a
// level have (nearly) the same D where the coefficients vary little, so its
// errors do not average out over them, and without the step the solution was 3
// to 8 times as far from exact as the banded LU's. Level 1's inverse counts
// most; there I - D X is summed as if exactly. What the update left out in
// rounding D is kept in the place of P until then. (Errors against the banded
// LU's, strips of 63 x 255 unknowns, c varying and c = 0 throughout: 3.7 and 7.4
// without, 0.7 and 2.1 with the steps alone, 0.6 and 1.2 so; steps at fewer
// levels 0.8 to 1.3, exact sums at all of them no better. A new operator on
// 257^2 points takes 0.50 ms, 0.44 without, 0.57 with exact sums at all levels.)
constexpr int kCrNewtonLevels = 4;
template <int WP, bool FIRST>
__global__ void __launch_bounds__(kCrThreads) stage2_cr_eliminate_kernel(const SubBox *boxes, const Stage2Cr *tab,
                                                                         const double *stencil, double *cr, int level)
{
    constexpr int kLds = WP * (WP + 1);
    __shared__ double X[kLds], R[kLds];  // R: D, then I - D X
    __shared__ double A[FIRST ? 1 : kLds], C[FIRST ? 1 : kLds];
    constexpr int kCols = 64 / kCrWaves;
    __shared__ double mult[2][kCols][64], inverse[64];
    const CrBox<WP> bx(boxes, tab, blockIdx.y);
    const int t = 1 << level, i = t * (2 * (int)blockIdx.x + 1), L = bx.b.L;
    if (i > L) return;  // whole workgroup
    const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
    double *row = bx.row(cr, i);
    constexpr int nb = WP * WP;
    double a[kCols];
#pragma unroll
    for (int e = 0; e < kCols; ++e) {
        const int k = q * kCols + e;
        if (FIRST)
            a[e] = bx.centre(stencil, i, r, k);
        else
            a[e] = r < WP && k < WP ? gload(row + k * WP + r) : (r == k ? 1.0 : 0.0);
        if (!FIRST && r < WP && k < WP) R[k * (WP + 1) + r] = a[e];
    }
    CrCopy<WP> to_a;
    if (!FIRST) {  // the last update's; D's rounding is in A's place meanwhile
        const double *ac = bx.pair(cr, level - 1, i >> level) + 2 * nb;
        to_a.fetch(ac);
        cr_stage<WP>(C, ac + nb);
        if (level < kCrNewtonLevels)
            cr_stage<WP>(A, row + nb);
        else
            to_a.put(A);
    }
    for (int k0 = 0, b = 0; k0 < WP; k0 += kCols, b ^= 1) {
        if (q * kCols == k0) {
            // column kk at a[0]: each pivot moves the columns one place on
#pragma unroll 1
            for (int kk = 0; kk < kCols; ++kk) {
                const int k = k0 + kk;
                const double pivot = readlane_f64(a[0], k);
                double inv = __builtin_amdgcn_rcp(pivot);
                inv = madd(inv, madd(-pivot, inv, 1.0), inv);
                inv = madd(inv, madd(-pivot, inv, 1.0), inv);
                const double m = r == k ? 0.0 : a[0] * inv;
#pragma unroll
                for (int e = 1; e < kCols; ++e) a[e - 1] = madd(-m, readlane_f64(a[e], k), a[e]);
                a[kCols - 1] = r == k ? 1.0 : -m;
                mult[b][kk][r] = m;
                if (r == k) inverse[k] = inv;
            }
        }
        __syncthreads();
        if (q * kCols != k0) {
#pragma unroll 2
            for (int kk = 0; kk < kCols; ++kk) {
                const double m = mult[b][kk][r];
#pragma unroll
                for (int e = 0; e < kCols; ++e) a[e] = madd(-m, readlane_f64(a[e], k0 + kk), a[e]);
            }
        }
    }
    const double scale = r < WP ? inverse[r] : 1.0;
#pragma unroll
    for (int e = 0; e < kCols; ++e) {
        const int k = q * kCols + e;
        a[e] *= scale;
        if (r < WP && k < WP) X[k * (WP + 1) + r] = a[e];
    }
    __syncthreads();
    double *D = row, *P = row + nb, *Q = row + 2 * nb;
    const int nt = WP / 16, ti = q / nt, tj = q % nt;
    const bool mine = q < nt * nt;  // a tile a wave
    Acc4 acc{0, 0, 0, 0};
    if (FIRST || level < kCrNewtonLevels) {
        const int tile = (tj * 16 + (r >> 4)) * (WP + 1) + ti * 16 + (r & 15);  // acc[v]: 4 v columns on
        if (FIRST) {
            if (r < WP) {
                const double lower = r ? bx.centre(stencil, i, r, r - 1) : 0.0, centre = bx.centre(stencil, i, r, r);
                const double upper = r + 1 < WP ? bx.centre(stencil, i, r, r + 1) : 0.0;
#pragma unroll
                for (int e = 0; e < kCols; ++e) {
                    const int k = q * kCols + e;
                    if (k >= WP) continue;
                    const double *x = X + k * (WP + 1);
                    double v = madd(-centre, a[e], r == k ? 1.0 : 0.0);
                    v = madd(-lower, x[r ? r - 1 : 0], v);
                    R[k * (WP + 1) + r] = madd(-upper, x[r + 1 < WP ? r + 1 : r], v);
                }
            }
        } else {
            if (mine) {
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = ti * 16 + (r & 15) == tj * 16 + 4 * v + (r >> 4) ? 1.0 : 0.0;
                if (level == 1) {
                    // (the largest entries of a diagonally dominant D and of its
                    // inverse are on their diagonals)
                    const int at = r < WP ? r * (WP + 2) : 0;
                    const double ud = cr_rounder(wave_max(fabs(R[at]))), ux = cr_rounder(wave_max(fabs(X[at])));
                    acc = cr_residual_tile<WP>(R, A, X, ti, tj, ud, ux, acc);
                } else {
                    acc = cr_tile<WP>(A, X, ti, tj, -1.0, cr_tile<WP>(R, X, ti, tj, -1.0, acc));
                }
            }
            __syncthreads();
            if (mine)
#pragma unroll
                for (int v = 0; v < 4; ++v) R[tile + 4 * v * (WP + 1)] = acc[v];
            to_a.put(A);
        }
        __syncthreads();
        if (mine) {
            acc = cr_tile<WP>(X, R, ti, tj, 1.0, Acc4{0, 0, 0, 0});
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc[v] += X[tile + 4 * v * (WP + 1)];
                gstore(cr_element<WP>(D, ti, tj, v), acc[v]);
            }
        }
        if (FIRST) return;
        __syncthreads();
        if (mine)
#pragma unroll
            for (int v = 0; v < 4; ++v) X[tile + 4 * v * (WP + 1)] = acc[v];
        __syncthreads();
    } else {
#pragma unroll
        for (int e = 0; e < kCols; ++e) {
            const int k = q * kCols + e;
            if (r < WP && k < WP) gstore(D + k * WP + r, a[e]);
        }
    }
    for (int n = q; n < 2 * nt * nt; n += kCrWaves) {
        const bool second = n >= nt * nt;
        const int m = second ? n - nt * nt : n;
        acc = cr_tile<WP>(X, second ? C : A, m / nt, m % nt, 1.0, Acc4{0, 0, 0, 0});
#pragma unroll
        for (int v = 0; v < 4; ++v) gstore(cr_element<WP>(second ? Q : P, m / nt, m % nt, v), acc[v]);
    }
}

// The even multiples of 2 after level 0, whose A and C are diagonal: all from
// the neighbours' D^-1, element by element.
template <int WP>
__global__ void __launch_bounds__(kCrThreads) stage2_cr_first_update_kernel(const SubBox *boxes, const Stage2Cr *tab,
                                                                            const double *stencil, double *cr)
{
    __shared__ double al[WP], cl[WP], ai[WP], ci[WP], au[WP], cu[WP];
    const CrBox<WP> bx(boxes, tab, blockIdx.y);
    const int i = 2 * ((int)blockIdx.x + 1);
    if (i > bx.b.L) return;  // whole workgroup
    const bool has_upper = i + 1 <= bx.b.L;
    if (threadIdx.x < WP) {
        const int r = threadIdx.x;
        al[r] = bx.slot(stencil, i - 1, r, 0), cl[r] = bx.slot(stencil, i - 1, r, 4);
        ai[r] = bx.slot(stencil, i, r, 0), ci[r] = bx.slot(stencil, i, r, 4);
        au[r] = has_upper ? bx.slot(stencil, i + 1, r, 0) : 0.0, cu[r] = has_upper ? bx.slot(stencil, i + 1, r, 4) : 0.0;
    }
    __syncthreads();
    constexpr int nb = WP * WP;
    const double *lower = bx.row(cr, i - 1), *upper = bx.row(cr, has_upper ? i + 1 : i - 1);
    double *D = bx.row(cr, i), *ac = bx.pair(cr, 0, (int)blockIdx.x + 1) + 2 * nb;
    for (int e = threadIdx.x; e < nb; e += kCrThreads) {
        const int r = e % WP, k = e / WP;
        const double va = ai[r] * gload(lower + e), vc = has_upper ? ci[r] * gload(upper + e) : 0.0;
        double lost;
        gstore(D + e, cr_add(bx.centre(stencil, i, r, k), -madd(va, cl[k], vc * au[k]), lost));
        gstore(D + nb + e, lost);
        gstore(ac + e, -(va * al[k]));
        gstore(ac + nb + e, -(vc * cu[k]));
    }
}

// The even multiples of 2^level, level > 0, after their neighbours'
// elimination: M and N (part 0), the new A and C (1) and D (2), a workgroup
// each, two products.
template <int WP>
__global__ void __launch_bounds__(kCrThreads) stage2_cr_update_kernel(const SubBox *boxes, const Stage2Cr *tab,
                                                                      double *cr, int level)
{
    __shared__ double X[2][WP * (WP + 1)], Y[2][WP * (WP + 1)];
    const CrBox<WP> bx(boxes, tab, blockIdx.y);
    const int t = 1 << level, i = 2 * t * ((int)blockIdx.x + 1), L = bx.b.L;
    if (i > L) return;  // whole workgroup
    const int part = blockIdx.z;
    constexpr int nb = WP * WP;
    double *D = bx.row(cr, i), *out = bx.pair(cr, level, (int)blockIdx.x + 1) + (part == 1 ? 2 * nb : 0);
    const bool has_upper = i + t <= L;
    const double *lower = bx.row(cr, i - t), *upper = bx.row(cr, has_upper ? i + t : i - t);
    // A times `a` of the lower row, C times `c` of the upper one
    const double *a = lower + (size_t)(part == 0 ? 0 : part == 1 ? 1 : 2) * nb;
    const double *c = upper + (size_t)(part == 0 ? 0 : part == 1 ? 2 : 1) * nb;
    const double sign = part == 0 ? 1.0 : -1.0;
    const int q = threadIdx.x >> 6, nt = WP / 16, tiles = nt * nt;
    const double *ac = bx.pair(cr, level - 1, i >> level) + 2 * nb;
    cr_stage<WP>(X[0], ac);
    cr_stage<WP>(Y[0], a);
    if (has_upper) {
        cr_stage<WP>(X[1], ac + nb);
        cr_stage<WP>(Y[1], c);
    }
    __syncthreads();
    for (int m = q; m < tiles; m += kCrWaves) {
        const int ti = m / nt, tj = m % nt;
        // (A Q + C P is summed up before it is taken from D, whose rounding
        // would otherwise go into every term)
        Acc4 acc = cr_tile<WP>(X[0], Y[0], ti, tj, sign, Acc4{0, 0, 0, 0});
        if (part != 2) {
#pragma unroll
            for (int v = 0; v < 4; ++v) gstore(cr_element<WP>(out, ti, tj, v), acc[v]);
            acc = Acc4{0, 0, 0, 0};
        }
        if (has_upper) acc = cr_tile<WP>(X[1], Y[1], ti, tj, sign, acc);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double *at = cr_element<WP>(part == 2 ? D : out + nb, ti, tj, v);
            if (part == 2) {
                double lost;
                gstore(at, cr_add(gload(at), acc[v], lost));
                gstore(at + nb, gload(at + nb) + lost);
            } else {
                gstore(at, acc[v]);
            }
        }
    }
}

// A row's substitution: 4 x kRow threads, thread r of quarter q takes the
// columns of quarter q of each block it needs.
template <int WP>
struct CrSolve {
    static constexpr int kRow = WP == 48 ? 64 : WP, kThreads = 4 * kRow, kPart = WP / 4;
    double x[3][kRow], part[4][kRow];

    // Quarter q of row r of a block (by column), and its product with x.
    struct Piece {
        double v[kPart];
    };
    __device__ static __forceinline__ Piece load(const double *B, int r, int q, bool there)
    {
        Piece p;
#pragma unroll
        for (int k = 0; k < kPart; ++k) p.v[k] = there && r < WP ? gload(B + (q * kPart + k) * WP + r) : 0.0;
        return p;
    }
    __device__ static __forceinline__ double dot(const Piece &p, const double *y, int q)
    {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < kPart; ++k) acc = madd(p.v[k], y[q * kPart + k], acc);
        return acc;
    }

    // Forward (FORWARD) or back substitution of block row i at a level; every
    // thread of the workgroup calls it, those of a team without a row with
    // `active` false. The blocks are on their way before the right sides are
    // waited for.
    template <bool FORWARD>
    __device__ __forceinline__ void row(const Stage2Grid &g, const CrBox<WP> &bx, const double *stencil, double *cr,
                                        double *rhs, int level, int i, bool active, int r, int q)
    {
        const int t = 1 << level, L = bx.b.L, w = bx.b.w;
        constexpr int nb = WP * WP;
        const bool lo = active && i - t >= 1, up = active && i + t <= L;
        double *f = rhs + bx.b.first + (int64_t)(i - 1) * w;
        Piece b0, b1, b2;
        if (FORWARD) {
            // M, N; at level 0 A D^-1, C D^-1 of the neighbours
            const double *M = active && level > 0 ? bx.pair(cr, level, i >> (level + 1)) : nullptr;
            b0 = load(level > 0 ? M : bx.row(cr, i - 1), r, q, active);
            b2 = load(level > 0 ? M + nb : bx.row(cr, i + 1), r, q, up);
        } else {
            // D^-1, P, Q; at level 0 P = D^-1 A, Q = D^-1 C
            const double *D = bx.row(cr, i);
            b1 = load(D, r, q, active);
            b0 = load(D + nb, r, q, lo && level > 0);
            b2 = load(D + 2 * nb, r, q, up && level > 0);
        }
        if (q < 3) {  // f of rows i - t, i and i + t
            const bool there = r < w && (q == 1 ? active : q == 0 ? lo : up);
            x[q][r] = there ? gload(f + (int64_t)(q - 1) * t * w + r) : 0.0;
        }
        const bool failed = *g.failed != 0;
        const double sa = level == 0 && active ? bx.slot(stencil, i, r, 0) : 1.0;
        const double sc = level == 0 && active ? bx.slot(stencil, i, r, 4) : 1.0;
        __syncthreads();
        double acc;
        if (FORWARD) {
            acc = -sa * dot(b0, x[0], q) - sc * dot(b2, x[2], q);
        } else if (level == 0) {
            if (q == 0) x[1][r] -= sa * x[0][r] + sc * x[2][r];
            __syncthreads();
            acc = dot(b1, x[1], q);
        } else {
            acc = dot(b1, x[1], q) - dot(b0, x[0], q) - dot(b2, x[2], q);
        }
        part[q][r] = acc;
        __syncthreads();
        if (q == 0 && r < w && active) {
            double v = ((part[0][r] + part[1][r]) + part[2][r]) + part[3][r];
            if (FORWARD) {
                gstore(f + r, x[1][r] + v);
            } else {
                gstore(f + r, v);
                int gi, gj;
                stage2_point(bx.b, (uint64_t)(i - 1) * w + r, gi, gj);
                if (!failed) g.u[(size_t)gj * g.n0 + gi] = v;
            }
        }
    }
};

// Substitution at one level, a workgroup per block row. Bound by latency (4 to
// 5 us a launch), but for the lowest levels (6 to 9 us).
template <int WP, bool FORWARD>
__global__ void __launch_bounds__(CrSolve<WP>::kThreads) stage2_cr_solve_kernel(const Stage2Grid g, const SubBox *boxes,
                                                                                const Stage2Cr *tab,
                                                                                const double *stencil, double *cr,
                                                                                double *rhs, int level)
{
    __shared__ CrSolve<WP> s;
    const CrBox<WP> bx(boxes, tab, blockIdx.y);
    const int t = 1 << level, i = FORWARD ? 2 * t * ((int)blockIdx.x + 1) : t * (2 * (int)blockIdx.x + 1);
    if (i > bx.b.L) return;  // whole workgroup
    s.template row<FORWARD>(g, bx, stencil, cr, rhs, level, i, true, threadIdx.x % CrSolve<WP>::kRow,
                            threadIdx.x / CrSolve<WP>::kRow);
}

// All levels from `first` on, forward and back, a workgroup per subdomain: for
// the levels of few rows a launch each costs more than one CU's bandwidth.
// Kept blocks, four strips, a call: 97^2 (blocks of 32) 80 us from 16 rows on, 82
// from 32, 95 from 64, 129^2 82, 86 and 108 us; 65^2 (blocks of 16) 64 us with
// all levels here, 16 us more with a launch for every level.
template <int WP>
constexpr int kTopRows = WP == 16 ? 64 : WP == 32 ? 16 : 8;
constexpr int kTopThreads = 1024;
template <int WP>
__global__ void __launch_bounds__(kTopThreads) stage2_cr_top_kernel(const Stage2Grid g, const SubBox *boxes,
                                                                    const Stage2Cr *tab, const double *stencil,
                                                                    double *cr, double *rhs, int first)
{
    constexpr int kTeam = CrSolve<WP>::kThreads, kTeams = kTopThreads / kTeam;
    __shared__ CrSolve<WP> teams[kTeams];
    const CrBox<WP> bx(boxes, tab, blockIdx.x);
    const int L = bx.b.L, team = threadIdx.x / kTeam, r = threadIdx.x % CrSolve<WP>::kRow;
    const int q = threadIdx.x % kTeam / CrSolve<WP>::kRow;
    CrSolve<WP> &s = teams[team];
    int l = first;
    for (; (2 << l) <= L; ++l)
        for (int m = 0; m < L >> (l + 1); m += kTeams) {
            const int i = (m + team + 1) << (l + 1);
            s.template row<true>(g, bx, stencil, cr, rhs, l, i, i <= L, r, q);
            __syncthreads();
        }
    for (; l >= first; --l)
        for (int m = 0; (2 * m + 1) << l <= L; m += kTeams) {
            const int i = (2 * (m + team) + 1) << l;
            s.template row<false>(g, bx, stencil, cr, rhs, l, i, i <= L, r, q);
            __syncthreads();
        }
}

template <int WP>
hipError_t launch_cyclic_reduction(const Stage2Run &run, const Stage2Grid &g, const SubBox *all, const double *stencil,
                                   const Stage2Plan &plan, hipStream_t s)
{
    const SubBox *boxes = all + run.first;
    const Stage2Cr *tab = plan.cr_tab + run.first;
    const int max_L = run.max_L;
    int levels = 0;
    while ((1 << levels) <= max_L) ++levels;
    const auto odd = [&](int l) { return dim3((unsigned)(((max_L >> l) + 1) / 2), run.n); };
    const auto even = [&](int l, int parts) { return dim3((unsigned)(max_L >> (l + 1)), run.n, parts); };
    hipError_t e = hipSuccess;
    for (int l = 0; l < levels && !plan.factored; ++l) {
        const auto eliminate = l == 0 ? stage2_cr_eliminate_kernel<WP, true> : stage2_cr_eliminate_kernel<WP, false>;
        hipLaunchKernelGGL(eliminate, odd(l), dim3(kCrThreads), 0, s, boxes, tab, stencil, plan.factor, l);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (l + 1 == levels) break;
        if (l == 0)
            hipLaunchKernelGGL((stage2_cr_first_update_kernel<WP>), even(0, 1), dim3(kCrThreads), 0, s, boxes,
                               tab, stencil, plan.factor);
        else
            hipLaunchKernelGGL((stage2_cr_update_kernel<WP>), even(l, 3), dim3(kCrThreads), 0, s, boxes, tab,
                               plan.factor, l);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    int top = 0;
    while ((max_L >> top) >= kTopRows<WP>) ++top;
    for (int l = 0; l < top; ++l) {
        hipLaunchKernelGGL((stage2_cr_solve_kernel<WP, true>), even(l, 1), dim3(CrSolve<WP>::kThreads), 0, s, g, boxes,
                           tab, stencil, plan.factor, plan.rhs, l);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(stage2_cr_top_kernel<WP>, dim3(run.n), dim3(kTopThreads), 0, s, g, boxes, tab, stencil,
                       plan.factor, plan.rhs, top);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int l = top - 1; l >= 0; --l) {
        hipLaunchKernelGGL((stage2_cr_solve_kernel<WP, false>), odd(l), dim3(CrSolve<WP>::kThreads), 0, s, g, boxes,
                           tab, stencil, plan.factor, plan.rhs, l);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_grid_residual(const DevProblem<double> &P, double sigma, const pdd_grid *g, void *r, hipStream_t s)
{
    const bool tab = P.tab != 0 || P.big_trig;
    if (g->dtype == PDD_DTYPE_F32)
        return g->dim == 2 ? (tab ? launch_residual<float, 2, true> : launch_residual<float, 2, false>)(P, sigma, g, r, s)
                           : (tab ? launch_residual<float, 3, true> : launch_residual<float, 3, false>)(P, sigma, g, r, s);
    return g->dim == 2 ? (tab ? launch_residual<double, 2, true> : launch_residual<double, 2, false>)(P, sigma, g, r, s)
                       : (tab ? launch_residual<double, 3, true> : launch_residual<double, 3, false>)(P, sigma, g, r, s);
}

hipError_t launch_stage2_edges(const DevProblem<double> &P, const Stage2Grid &g, const Stage2Edges &a, hipStream_t s)
{
    const uint64_t points = 2ull * (g.n0 + g.n1 - 2), per = kWeightsThreads;
    const uint64_t blocks = a.n_lines + (points + per - 1) / per + std::min<uint64_t>((a.table_words + per - 1) / per, 64);
    hipLaunchKernelGGL(stage2_edges_kernel, dim3((uint32_t)blocks), dim3(kWeightsThreads), 0, s, P, g, a);
    return hipGetLastError();
}

hipError_t launch_stage2_stencils(const DevProblem<double> &P, const Stage2Grid &g, const SubBox *boxes,
                                  int32_t n_boxes, uint32_t max_unknowns, const Stage2Line *lines, int32_t n_lines,
                                  double *stencil, double *rhs, bool parts, int32_t *not_dominant, hipStream_t s)
{
    hipLaunchKernelGGL(stage2_stencil_kernel, dim3((max_unknowns + 255) / 256 + 1, std::max(n_boxes, 1)), dim3(256), 0, s,
                       P, g, boxes, lines, n_lines, stencil, rhs, parts, not_dominant);
    return hipGetLastError();
}

hipError_t launch_stage2_solve(const Stage2Grid &g, const SubBox *boxes,
                               int32_t n_boxes, uint32_t max_unknowns, const double *stencil, const Stage2Plan &plan,
                               hipStream_t s)
{
    if (n_boxes == 0) return hipSuccess;
    hipError_t e = hipSuccess;
    if (!plan.cr_tab) {
        if (!plan.factored) {
            hipLaunchKernelGGL(stage2_lu_kernel, dim3(n_boxes), dim3(kStage2LuThreads), 0, s, boxes, stencil,
                               plan.factor, plan.lmul);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (!plan.resp_tab) {
            hipLaunchKernelGGL(stage2_subst_kernel, dim3(n_boxes), dim3(kStage2SubstThreads), 0, s, g, boxes, stencil,
                               plan.factor, plan.lmul);
            return hipGetLastError();
        }
        if (!plan.resp_ready) {
            const uint32_t groups = (uint32_t)(plan.max_cols + kStage2RespWaves - 1) / kStage2RespWaves;
            hipLaunchKernelGGL(stage2_resp_kernel, dim3(n_boxes, groups), dim3(kStage2SubstThreads), 0, s, boxes,
                               plan.rhs, plan.factor, plan.lmul, plan.resp_tab, plan.rb, plan.resp);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        const uint32_t blocks = std::min<uint32_t>((max_unknowns + 255) / 256, 1024);
        hipLaunchKernelGGL(stage2_apply_kernel, dim3(blocks, n_boxes), dim3(256), 0, s, g, boxes, plan.rhs,
                           plan.resp_tab, plan.rb, plan.resp);
        return hipGetLastError();
    }
    for (int q = 0; q < plan.n_runs && e == hipSuccess; ++q) {
        const Stage2Run &run = plan.runs[q];
        switch (run.wp) {
            case 16: e = launch_cyclic_reduction<16>(run, g, boxes, stencil, plan, s); break;
            case 32: e = launch_cyclic_reduction<32>(run, g, boxes, stencil, plan, s); break;
            case 48: e = launch_cyclic_reduction<48>(run, g, boxes, stencil, plan, s); break;
            default: e = launch_cyclic_reduction<64>(run, g, boxes, stencil, plan, s); break;
        }
    }
    return e;
}

}  // namespace pdd
