// The elementary functions of the FP64 walks, one value a thread, so that tests
// can compare each with its exact value.
#include "path_walk.hpp"

namespace pdd {
namespace {

enum { kLn, kSqrt, kTurn, kSinCos, kExp, kNumFunctions };

__global__ void fp64_math_kernel(int function, const uint32_t *words, const double *values, long long n, double *out0,
                                 double *out1)
{
    MathOf<double> mt;
    mt.init();
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < n; q += (long long)gridDim.x * blockDim.x) {
        double a = 0.0, b = 0.0;
        if (function == kLn)
            a = Fp64Math::minus_two_ln(words[q]);
        else if (function == kSqrt)
            a = Fp64Math::sqrt_normal(values[q]);
        else if (function == kTurn)
            Fp64Math::sincos_turn(mt, words[q], a, b);
        else if (function == kSinCos)
            Fp64Math::sincos(mt, values[q], a, b);
        else
            a = Fp64Math::exp_neg(values[q]);
        out0[q] = a;
        out1[q] = b;
    }
}

}  // namespace
}  // namespace pdd

// Function 0: -2 ln((w + 1/2) 2^-32), 1: sqrt x, 2: sine and cosine of 2 pi (w +
// 1/2) 2^-32, 3: sine and cosine of x, 4: exp(-x), of n values in device memory
// (words w or doubles x) into out0 and out1 (the cosines). Returns 0 or a HIP error
// code, after the values are there.
extern "C" int probe_fp64_math(int function, const void *in, long long n, double *out0, double *out1)
{
    if (function < 0 || function >= pdd::kNumFunctions || !in || !out0 || !out1 || n < 1) return (int)hipErrorInvalidValue;
    const unsigned grid = (unsigned)std::min<long long>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(pdd::fp64_math_kernel, dim3(grid), dim3(256), 0, nullptr, function,
                       static_cast<const uint32_t *>(in), static_cast<const double *>(in), n, out0, out1);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    return (int)e;
}
