// Gradient of a gridded function by second-order finite differences: the
// grad(u~) grids of the pathwise control variate (eq. F:xiControlVariate) when
// only values of u~ on a grid are known, as inside the outer iteration.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "host_runtime.hpp"
#include "pdd.h"

using pdd::fail;

namespace {

// Derivative along one axis at a point whose index along that axis is a (of
// n): central inside, three-point one-sided at the two ends; st is the
// point's stride along the axis, two_dx twice the spacing.
template <class S, class I>
__device__ __forceinline__ S axis_derivative(const S *__restrict__ u, I p, S u0, I st, int a, int n, S two_dx)
{
    const bool low = a == 0, high = a == n - 1;
    // the point before and the point after, or at an end the next two inwards
    const S v1 = u[low ? p + st : p - st];
    const S v2 = u[low ? p + 2 * st : high ? p - 2 * st : p + st];
    const S d = low ? (S)-3 * u0 + (S)4 * v1 - v2 : high ? (S)3 * u0 - (S)4 * v1 + v2 : v2 - v1;
    return d / two_dx;
}

// One thread per grid point (x fastest, so neighbouring threads read
// neighbouring values), all dim components. I: the type that holds a point's
// number (64-bit divisions cost a third of the time: 129^3 FP32 14.4 and 11.2
// us, 34 MB). Bound by memory: 2049^2 FP64 20 us, 101 MB.
template <class S, int D, class I>
__global__ void __launch_bounds__(256) grid_gradient_kernel(const S *__restrict__ u, int n0, int n1, int n2, S dx0, S dx1,
                                                            S dx2, S *__restrict__ g0, S *__restrict__ g1,
                                                            S *__restrict__ g2)
{
    const I m01 = (I)n0 * n1, total = m01 * (D == 3 ? n2 : 1);
    for (I p = blockIdx.x * (I)blockDim.x + threadIdx.x; p < total; p += (I)gridDim.x * blockDim.x) {
        const I jk = p / n0;
        const int k = D == 3 ? (int)(jk / n1) : 0, i = (int)(p - jk * n0), j = D == 3 ? (int)(jk - (I)k * n1) : (int)jk;
        const S u0 = u[p];
        g0[p] = axis_derivative<S, I>(u, p, u0, 1, i, n0, dx0);
        g1[p] = axis_derivative<S, I>(u, p, u0, (I)n0, j, n1, dx1);
        if (D == 3) g2[p] = axis_derivative<S, I>(u, p, u0, m01, k, n2, dx2);
    }
}

template <class S, int D>
hipError_t launch_gradient(const pdd_grid *g, void *const *out, hipStream_t s)
{
    const int n2 = D == 3 ? g->n[2] : 1;
    const uint64_t total = (uint64_t)g->n[0] * g->n[1] * n2;
    const uint64_t blocks = std::min<uint64_t>((total + 255) / 256, 16384);
    S two_dx[3] = {0, 0, 0};
    for (int d = 0; d < D; ++d) two_dx[d] = (S)(2.0 * ((g->hi[d] - g->lo[d]) / (g->n[d] - 1)));
    // (2^31: a thread's next point still fits in 32 bits)
    const auto kernel = total < (1ull << 31) ? grid_gradient_kernel<S, D, uint32_t> : grid_gradient_kernel<S, D, uint64_t>;
    hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(256), 0, s, static_cast<const S *>(g->data), g->n[0], g->n[1],
                       n2, two_dx[0], two_dx[1], two_dx[2], static_cast<S *>(out[0]), static_cast<S *>(out[1]),
                       static_cast<S *>(D == 3 ? out[2] : out[1]));
    return hipGetLastError();
}

}  // namespace

extern "C" pdd_status pdd_grid_residual(pdd_problem *problem, const pdd_grid *u, void *resid, void *stream)
{
    if (!problem || !u || !resid) return fail(PDD_E_INVALID, "NULL argument");
    const int D = u->dim;
    if (D != problem->desc.dim) return fail(PDD_E_INVALID, "grid dim %d != problem dim %d", D, problem->desc.dim);
    if (!u->data) return fail(PDD_E_INVALID, "grid has no data");
    if (u->dtype != PDD_DTYPE_F32 && u->dtype != PDD_DTYPE_F64) return fail(PDD_E_INVALID, "bad grid dtype");
    for (int d = 0; d < D; ++d) {
        if (u->n[d] < 4) return fail(PDD_E_INVALID, "second derivatives at the edges need n >= 4 per axis");
        if (!(u->hi[d] > u->lo[d]) || !std::isfinite(u->hi[d] - u->lo[d]))
            return fail(PDD_E_INVALID, "grid needs finite lo < hi");
    }
    if ((uint64_t)u->n[0] * u->n[1] * (D == 3 ? (uint64_t)u->n[2] : 1) >= (1ull << 40))
        return fail(PDD_E_INVALID, "grid too large");
    HIP_TRY(hipSetDevice(problem->ctx->device));
    // the source is evaluated at the grid's points, which may lie far outside
    // the problem's box: their arguments choose the trig functions
    const int32_t big_trig = !(pdd::trig_revolutions(problem->desc, u->lo, u->hi) <= pdd::kFp64TrigRevolutions);
    const auto launch = [&](const pdd::DevProblem<double> &pd) {
        return pdd::launch_grid_residual(pd, problem->desc.sigma, u, resid, static_cast<hipStream_t>(stream));
    };
    hipError_t e;
    if (big_trig == problem->pd.big_trig) {
        e = launch(problem->pd);
    } else {
        pdd::DevProblem<double> pd = problem->pd;
        pd.big_trig = big_trig;
        e = launch(pd);
    }
    if (e != hipSuccess) return fail(PDD_E_HIP, "grid residual launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

extern "C" pdd_status pdd_grid_gradient(pdd_ctx *ctx, const pdd_grid *u, void *const *grad, void *stream)
{
    if (!ctx || !u || !grad) return fail(PDD_E_INVALID, "NULL argument");
    const int D = u->dim;
    if (D != 2 && D != 3) return fail(PDD_E_INVALID, "grid dim must be 2 or 3");
    if (!u->data) return fail(PDD_E_INVALID, "grid has no data");
    if (u->dtype != PDD_DTYPE_F32 && u->dtype != PDD_DTYPE_F64) return fail(PDD_E_INVALID, "bad grid dtype");
    for (int d = 0; d < D; ++d) {
        if (u->n[d] < 3) return fail(PDD_E_INVALID, "second-order differences need n >= 3 per axis");
        if (!(u->hi[d] > u->lo[d]) || !std::isfinite(u->hi[d] - u->lo[d]))
            return fail(PDD_E_INVALID, "grid needs finite lo < hi");
        if (!grad[d]) return fail(PDD_E_INVALID, "gradient buffer %d is NULL", d);
    }
    if ((uint64_t)u->n[0] * u->n[1] * (D == 3 ? (uint64_t)u->n[2] : 1) >= (1ull << 40))
        return fail(PDD_E_INVALID, "grid too large");
    HIP_TRY(hipSetDevice(ctx->device));
    const hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if (u->dtype == PDD_DTYPE_F32)
        e = D == 2 ? launch_gradient<float, 2>(u, grad, s) : launch_gradient<float, 3>(u, grad, s);
    else
        e = D == 2 ? launch_gradient<double, 2>(u, grad, s) : launch_gradient<double, 3>(u, grad, s);
    if (e != hipSuccess) return fail(PDD_E_HIP, "grid gradient launch: %s", hipGetErrorString(e));
    return PDD_OK;
}
