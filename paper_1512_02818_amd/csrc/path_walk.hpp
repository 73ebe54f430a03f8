// The walk of one path (first-stage PDD nodal solve), shared by the kernels
// that run it: random numbers, coefficients, the Euler-Maruyama step with its
// exit tests, scores, and the queues that hand paths to waves.
//
// Random numbers: Philox4x32-10 (Salmon et al., SC'11) in registers, key =
// problem seed (wave-uniform), counter = (step block, path, node, stream tag).
// In 2D one block gives the two normals of two consecutive steps (words 0,1
// then 2,3), so a lane starts a new path only at an even step; in 3D one block
// per step. The bridge uniform of step s is word s mod 4 of the tag-1 block
// s/4; the block is drawn for every walking lane of the wave at the first step
// of its four-step window at which some lane may have a live face, and cached
// for the rest of the window (drawn per lane inside the rare branch, it would
// be drawn up to four times per window, once for each step at which another
// lane first needs it).
// Box-Muller (1958) on the VALU: in FP32 with the hardware log2, sqrt, sin
// and cos (which take revolutions, so 2 pi u needs no multiply).
#pragma once

#include <type_traits>

#include "pdd_internal.hpp"

namespace pdd {
namespace {

// Device memory that the kernels reach through pointers held in descriptor
// tables (grids, node tables, records). The compiler cannot tell such a
// pointer from an LDS one and would emit flat accesses, which count against
// the same wait counter as the scalar loads of descriptor fields: every wait
// for a field would then also wait for an in-flight grid gather. Casting to
// the global address space gives global loads and stores with their own
// counter.
template <class T>
using Global = __attribute__((address_space(1))) T;
template <class T>
__device__ __forceinline__ T gload(const T *p)
{
    return *(const Global<T> *)p;
}
template <class T>
__device__ __forceinline__ void gstore(T *p, T v)
{
    *(Global<T> *)p = v;
}

constexpr float kLn2f = 0.6931471805599453f;
constexpr float kLog2ef = 1.4426950408889634f;

struct Block4 {
    uint32_t w0, w1, w2, w3;
};

// Philox4x32-10: two 32x32->64 products per round (v_mad_u64_u32) and two
// three-way XORs (v_bitop3_b32 with the XOR3 truth table 0x96), the key bumped
// by the Weyl constants after each round.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The ten round keys of a (wave-uniform) Philox key, in vector registers: the
// XOR3 takes three vector operands at no extra cost, and keeping twenty
// uniform values out of the scalar register file leaves it to the problem
// constants. Used by the FP32 walks, which are bound by instruction issue:
// recomputing the keys would add scalar instructions to every block.
struct KeySchedule {
    uint32_t k0[10], k1[10];
};

// The key as two scalar words, round keys recomputed by scalar adds in every
// block. Used by the FP64 walks, whose vector registers are the scarce
// resource: twenty fewer live values remove their spills.
struct ScalarKey {
    uint32_t k0, k1;
};

template <class T>
using KeysOf = typename std::conditional<sizeof(T) == 8, ScalarKey, KeySchedule>::type;

template <class K>
__device__ __forceinline__ K key_schedule(uint32_t k0, uint32_t k1);

template <>
__device__ __forceinline__ ScalarKey key_schedule<ScalarKey>(uint32_t k0, uint32_t k1)
{
    return {(uint32_t)__builtin_amdgcn_readfirstlane(k0), (uint32_t)__builtin_amdgcn_readfirstlane(k1)};
}

template <>
__device__ __forceinline__ KeySchedule key_schedule<KeySchedule>(uint32_t k0, uint32_t k1)
{
    KeySchedule ks;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint32_t v0, v1;
        asm volatile("v_mov_b32 %0, %1" : "=v"(v0) : "s"(k0));
        asm volatile("v_mov_b32 %0, %1" : "=v"(v1) : "s"(k1));
        ks.k0[r] = v0;
        ks.k1[r] = v1;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return ks;
}

__device__ __forceinline__ Block4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                         const KeySchedule &ks)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, ks.k0[r]);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, ks.k1[r]);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    return {c0, c1, c2, c3};
}

__device__ __forceinline__ Block4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                         const ScalarKey &key)
{
    // opaque to the optimiser, so that the round keys are formed here rather
    // than hoisted out of the walk loop into twenty live registers
    uint32_t ka = key.k0, kb = key.k1;
    asm volatile("" : "+s"(ka), "+s"(kb));
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, ka);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, kb);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        ka += 0x9E3779B9u;
        kb += 0xBB67AE85u;
    }
    return {c0, c1, c2, c3};
}

// Multiply-add with one rounding. The library is built without automatic
// contraction, so every fused operation is written out and all kernels that
// walk the same path round identically.
__device__ __forceinline__ float madd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
// x clamped to [lo, hi] (lo <= hi, x not NaN): one median-of-three.
__device__ __forceinline__ float med3(float x, float lo, float hi) { return __builtin_amdgcn_fmed3f(x, lo, hi); }
__device__ __forceinline__ double med3(double x, double lo, double hi) { return fmin(fmax(x, lo), hi); }
__device__ __forceinline__ double madd(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <class T>
struct Arith;

// What a walk keeps in registers for its elementary functions: in FP64 the
// coefficients of sine and cosine, which a step uses three times.
template <class T>
struct MathOf {
    __device__ __forceinline__ void init() {}
};
template <>
struct MathOf<double> {
    double S[6], C[6];
    __device__ __forceinline__ void init();
};

// FP32 path arithmetic: 24-bit uniforms, hardware transcendentals.
template <>
struct Arith<float> {
    // (w + 1/2) 2^-32 with w rounded to 24 significant bits: within 2^-24
    // (relative) of the FP64 uniform of the same word, in (0, 1]. It is
    // exactly 1 for the top 128 words (w >= 2^32 - 128, probability 2^-25):
    // such a bridge draw cannot end a path, and Box-Muller gives r = 0.
    __device__ static __forceinline__ float unif(uint32_t w)
    {
        return fmaf((float)w, 0x1.0p-32f, 0x1.0p-33f);
    }
    __device__ static __forceinline__ float unif_bridge(uint32_t w) { return unif(w); }
    __device__ static __forceinline__ float radius(uint32_t w)
    {
        return __builtin_amdgcn_sqrtf(-2.0f * kLn2f * __builtin_amdgcn_logf(unif(w)));
    }
    __device__ static __forceinline__ void box_muller(const MathOf<float> &, uint32_t a, uint32_t b, float &n0, float &n1)
    {
        const float r = radius(a);
        const float t = unif(b);  // revolutions
        n0 = r * __builtin_amdgcn_cosf(t);
        n1 = r * __builtin_amdgcn_sinf(t);
    }
    __device__ static __forceinline__ float box_muller_cos(const MathOf<float> &, uint32_t a, uint32_t b)
    {
        return radius(a) * __builtin_amdgcn_cosf(unif(b));
    }
    // k and ph are in revolutions; the hardware sine and cosine reduce any
    // argument within +-256 revolutions themselves.
    template <bool BIG>
    __device__ static __forceinline__ void trig(const MathOf<float> &, const DevProblem<float> &P, int m, int d, float x,
                                                float &s, float &c)
    {
        const DevTrig<float> &t = P.trig[m];
        const float rev = fmaf(t.k[d], x, t.ph[d]);
        s = __builtin_amdgcn_sinf(rev);
        c = __builtin_amdgcn_cosf(rev);
    }
    template <bool BIG>
    __device__ static __forceinline__ float sine(const MathOf<float> &, const DevProblem<float> &P, int m, int d, float x)
    {
        const DevTrig<float> &t = P.trig[m];
        return __builtin_amdgcn_sinf(fmaf(t.k[d], x, t.ph[d]));
    }
    __device__ static __forceinline__ float exp_neg(float x)
    {
        return __builtin_amdgcn_exp2f(-x * kLog2ef);
    }
    __device__ static __forceinline__ float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
};

// FP64 path arithmetic: 32-bit uniforms. The elementary functions are written
// for the arguments that a walk gives them (a uniform of 32 bits, a quarter
// turn with an exact remainder, the trig terms' arguments over the domain, a
// bridge exponent), which leaves out the library's general cases. FP64 walks
// are bound by vector issue, and these functions are most of a step: 18 nodes
// x 200,000 paths on the unit square (h = 1e-3) take 6.6 ms, 9.1 ms with the
// library's functions; 1,792 nodes x 256 paths on [0, 4]^2 16.4 ms, before
// 24.3 ms. Polynomials are minimax in relative error (Remez exchange in 50
// digits). Against the exact value of their argument, at most, in units in the
// last place: the logarithm 0.81, the square root 0.51, the exponential 0.89, sine
// and cosine of a turn's part 1.82 (its product with 2 pi is rounded); sine and
// cosine of a trig term's argument 0.87 units of 2^-53, absolute (and in the last
// place up to pi / 4; next to a zero after many turns the relative error is larger,
// as pi / 2 has two parts).
// Their coefficients come from constant memory by scalar loads at each use:
// as literals the compiler keeps all of them for the whole walk loop in scalar
// registers, which do not hold them, and each use then reads its spilled
// halves back through v_readlane (170 spilled registers).
__constant__ __attribute__((aligned(64))) const double kFp64Tab[40] = {
    // S of sin, highest power first; C of cos
    0x1.5d8fa2e5c73e7p-33, -0x1.ae5e59f4a6204p-26, 0x1.71de356710e0dp-19, -0x1.a01a019bfd15ep-13,
    0x1.111111110f7cap-7, -0x1.5555555555548p-3, -0x1.8ff9ad8c46497p-37, 0x1.1eea890e2e204p-29,
    -0x1.27e4f903ab84cp-22, 0x1.a01a019e24894p-16, -0x1.6c16c16c16131p-10, 0x1.5555555555553p-5,
    // 2 / pi; -pi / 2 in two parts; 2 pi 2^-32
    0x1.45f306dc9c883p-1, -0x1.921fb54442d18p+0, -0x1.1a62633145c07p-54, 0x1.921fb54442d18p-30,
    // L of ln; ln 2 in two parts
    0x1.2f048c754a96ep-3, 0x1.39a1d39b3401dp-3, 0x1.74663dcc62912p-3, 0x1.c71c520f847cdp-3,
    0x1.24924941e89a6p-2, 0x1.999999997fe64p-2, 0x1.5555555555592p-1, 0x1.62e42fefa39efp-1,
    0x1.abc9e3b39803fp-56, 0.0, 0.0, 0.0,
    // E of exp; -log2 e; (ln 2 above)
    0x1.af632ad6abee8p-26, 0x1.28b410d73d492p-22, 0x1.71ddf6b3f10d1p-19, 0x1.a01993b37a9cap-16,
    0x1.a01a01b00c2c6p-13, 0x1.6c16c18601e8cp-10, 0x1.111111110f803p-7, 0x1.55555555503e3p-5,
    0x1.5555555555558p-3, 0x1.0000000000009p-1, -0x1.71547652b82fep+0, 0.0};

struct Fp64Math {
    using Tab = const __attribute__((address_space(4))) double *;
    // The table's entries from `at` on, opaque to the optimiser.
    __device__ static __forceinline__ Tab tab(int at)
    {
        Tab t = (Tab)(kFp64Tab + at);
        asm volatile("" : "+s"(t));
        return t;
    }
    // sin x and cos x for |x| <= pi / 4:  x + x z S(z), 1 - z / 2 + z^2 C(z),
    // z = x^2 (S to 2^-57.9, C to 2^-62.1).
    // The angle is x + dx, dx below a unit in the last place of x.
    __device__ static __forceinline__ void sincos_octant(const MathOf<double> &m, double x, double dx, double &s,
                                                         double &c)
    {
        const double z = x * x;
        double S = m.S[0], C = m.C[0];
#pragma unroll
        for (int i = 1; i < 6; ++i) {
            S = madd(S, z, m.S[i]);
            C = madd(C, z, m.C[i]);
        }
        s = x + madd(x * z, S, dx);
        const double w = madd(-0.5, z, 1.0);
        c = w + madd(z * z, C, madd(-x, dx, madd(-0.5, z, 1.0 - w)));  // 1 - w - z / 2: what rounding w left out
    }
    // Of x + q pi / 2 from those of x.
    __device__ static __forceinline__ void quadrant(uint32_t q, double &s, double &c)
    {
        const double a = (q & 1u) ? c : s, b = (q & 1u) ? s : c;
        s = sign_flip(a, q << 30);
        c = sign_flip(b, (q + 1u) << 30);
    }
    // v with its sign changed if bit 31 of `bit` is set.
    __device__ static __forceinline__ double sign_flip(double v, uint32_t bit)
    {
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        const uint32_t hi = (uint32_t)(b >> 32) ^ (bit & 0x80000000u);
        return __longlong_as_double((long long)(((uint64_t)hi << 32) | (uint32_t)b));
    }
    // sin and cos of 2 pi (w + 1/2) 2^-32: the nearest quarter turn and the
    // remainder are exact integers of w.
    __device__ static __forceinline__ void sincos_turn(const MathOf<double> &m, uint32_t w, double &s, double &c)
    {
        const uint32_t q = (w + 0x20000000u) >> 30;
        const double r = (double)(int32_t)(w - (q << 30)) + 0.5;
        sincos_octant(m, r * 0x1.921fb54442d18p-30, 0.0, s, c);
        quadrant(q, s, c);
    }
    // sin and cos of x, |x| < 2^31: two-part reduction by pi / 2, whose
    // products are exact in the fused operations.
    __device__ static __forceinline__ void sincos(const MathOf<double> &m, double x, double &s, double &c)
    {
        const Tab t = tab(12);
        const double n = __builtin_rint(x * t[0]);
        const double a = madd(n, t[1], x), r = madd(n, t[2], a);
        sincos_octant(m, r, madd(n, t[2], a - r), s, c);
        quadrant((uint32_t)(int32_t)n, s, c);
    }
    // -2 ln((w + 1/2) 2^-32), arranged as in Sun's fdlibm (the coefficients are not
    // its): ln(1 + f) = 2 atanh(s), s = f / (2 + f), is
    // f - f^2 / 2 + s (f^2 / 2 + z L(z)), z = s^2, which keeps the relative
    // accuracy near 1 (L to 2^-59.5 for sqrt(1/2) <= 1 + f < sqrt(2)).
    __device__ static __forceinline__ double minus_two_ln(uint32_t w)
    {
        const uint64_t b = (uint64_t)__double_as_longlong((double)w + 0.5);
        const int32_t hi = (int32_t)(b >> 32);
        const int32_t k = (hi - 0x3fe6a09e) >> 20;  // d = (1 + f) 2^k
        const double f =
            __longlong_as_double((long long)(((uint64_t)(uint32_t)(hi - (k << 20)) << 32) | (uint32_t)b)) - 1.0;
        const double den = 2.0 + f;
        double y = __builtin_amdgcn_rcp(den);
        y = madd(y, madd(-den, y, 1.0), y);
        y = madd(y, madd(-den, y, 1.0), y);
        double t = f * y;
        t = madd(madd(-den, t, f), y, t);
        const double z = t * t;
        const Tab l = tab(16);
        double L = l[0];
#pragma unroll
        for (int i = 1; i < 7; ++i) L = madd(L, z, l[i]);
        const double h = 0.5 * f * f;
        const double e = (double)(k - 32);
        const double ln = madd(e, l[7], f - (h - madd(t, madd(z, L, h), e * l[8])));
        return -2.0 * ln;
    }
    // sqrt x for normal x: two coupled Newton steps (Goldschmidt) and a
    // residual correction.
    __device__ static __forceinline__ double sqrt_normal(double x)
    {
        const double y = __builtin_amdgcn_rsq(x);
        double g = x * y, h = 0.5 * y;
        double r = madd(-h, g, 0.5);
        g = madd(g, r, g);
        h = madd(h, r, h);
        g = madd(madd(-g, g, x), h, g);
        return madd(madd(-g, g, x), h, g);
    }
    // exp(-x), 0 <= x below some hundreds: 2^n (1 + r + r^2 E(r)) (E to 2^-56.8).
    __device__ static __forceinline__ double exp_neg(double x)
    {
        const Tab t = tab(23), ec = t + 5;
        const double n = __builtin_rint(x * ec[10]);
        const double a = madd(n, -t[0], -x), r = madd(n, -t[1], a), dr = madd(n, -t[1], a - r);
        double E = ec[0];
#pragma unroll
        for (int i = 1; i < 10; ++i) E = madd(E, r, ec[i]);
        return __builtin_ldexp(1.0 + (r + madd(r * r, E, dr)), (int)n);
    }
};

__device__ __forceinline__ void MathOf<double>::init()
{
#pragma unroll
    for (int i = 0; i < 12; ++i) {  // opaque moves: otherwise the loads would move to the uses
        const uint64_t b = (uint64_t)__double_as_longlong(kFp64Tab[i]);
        uint32_t lo, hi;
        asm volatile("v_mov_b32 %0, %1" : "=v"(lo) : "s"((uint32_t)b));
        asm volatile("v_mov_b32 %0, %1" : "=v"(hi) : "s"((uint32_t)(b >> 32)));
        (i < 6 ? S[i] : C[i - 6]) = __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    }
}

template <>
struct Arith<double> {
    __device__ static __forceinline__ double unif_bridge(uint32_t w)
    {
        return ((double)w + 0.5) * 0x1.0p-32;
    }
    __device__ static __forceinline__ void box_muller(const MathOf<double> &m, uint32_t a, uint32_t b, double &n0,
                                                      double &n1)
    {
        const double r = Fp64Math::sqrt_normal(Fp64Math::minus_two_ln(a));
        double s, c;
        Fp64Math::sincos_turn(m, b, s, c);
        n0 = r * c;
        n1 = r * s;
    }
    __device__ static __forceinline__ double box_muller_cos(const MathOf<double> &m, uint32_t a, uint32_t b)
    {
        double s, c;
        Fp64Math::sincos_turn(m, b, s, c);
        return Fp64Math::sqrt_normal(Fp64Math::minus_two_ln(a)) * c;
    }
    // BIG: arguments may reach 2^31 and take the library's functions then.
    template <bool BIG>
    __device__ static __forceinline__ void trig(const MathOf<double> &mt, const DevProblem<double> &P, int m, int d,
                                                double x, double &s, double &c)
    {
        const double arg = madd(P.trig[m].k[d], x, P.trig[m].ph[d]);
        if (BIG && P.big_trig)
            ::sincos(arg, &s, &c);
        else
            Fp64Math::sincos(mt, arg, s, c);
    }
    template <bool BIG>
    __device__ static __forceinline__ double sine(const MathOf<double> &mt, const DevProblem<double> &P, int m, int d,
                                                  double x)
    {
        double s, c;
        trig<BIG>(mt, P, m, d, x, s, c);
        return s;
    }
    __device__ static __forceinline__ double exp_neg(double x) { return Fp64Math::exp_neg(x); }
    __device__ static __forceinline__ double sqrt_(double x) { return sqrt(x); }
};

// Sum of monomials coef * x^e0 y^e1 z^e2 (exponents read from a wave-uniform
// packed word, so the power loops are scalar-controlled).
template <class T, int D>
__device__ __forceinline__ T poly_value(const DevPoly<T> *terms, int n, const T *x)
{
    T acc = (T)0;
    for (int m = 0; m < n; ++m) {
        const uint32_t e = terms[m].e;
        T v = terms[m].coef;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int ed = (int)((e >> (8 * d)) & 0xffu);
            for (int i = 0; i < ed; ++i) v *= x[d];
        }
        acc += v;
    }
    return acc;
}

// Dense polynomial in nested Horner form (no loops at run time): in 2D
// sum_j y^j sum_{i <= 5 - j} c_ij x^i, coefficients ordered by j then i;
// in 3D sum_k z^k sum_j y^j sum_{i <= 4 - j - k} c_ijk x^i, ordered by k, j, i.
template <class T, int D>
__device__ __forceinline__ T dense_poly(const T *c, const T *x)
{
    if (D == 2) {
        constexpr int deg = kDenseDeg2;
        T acc = (T)0;
        int off = (deg + 1) * (deg + 2) / 2;
#pragma unroll
        for (int j = deg; j >= 0; --j) {
            off -= deg - j + 1;  // first coefficient of row j
            T p = c[off + deg - j];
#pragma unroll
            for (int i = deg - j - 1; i >= 0; --i) p = madd(p, x[0], c[off + i]);
            acc = (j == deg) ? p : madd(acc, x[1], p);
        }
        return acc;
    }
    constexpr int deg = kDenseDeg3;
    T accz = (T)0;
    int off = kMaxDense;
#pragma unroll
    for (int k = deg; k >= 0; --k) {
        T accy = (T)0;
#pragma unroll
        for (int j = deg - k; j >= 0; --j) {
            off -= deg - j - k + 1;  // row (j, k)
            T p = c[off + deg - j - k];
#pragma unroll
            for (int i = deg - j - k - 1; i >= 0; --i) p = madd(p, x[0], c[off + i]);
            accy = (j == deg - k) ? p : madd(accy, x[1], p);
        }
        accz = (k == deg) ? accy : madd(accz, x[2 % D], accy);
    }
    return accz;
}

template <class T, int D>
__device__ __forceinline__ T interp_cells(const GridView<T> &g, const T *x);
template <class T, int D>
__device__ __forceinline__ void grid_cell(const GridView<T> &g, const T *x, int *i, T *w);
template <class T, int D>
__device__ __forceinline__ size_t cell_index(const GridView<T> &g, const int *i);
template <class T, int D>
__device__ __forceinline__ T interp_corners(const T *p, const T *w);
template <class T>
__device__ __forceinline__ T interp_corner_values(T c00, T c10, T c01, T c11, const T *w);
template <class T, int D, bool BIG>
__device__ __forceinline__ void analytic_source(const MathOf<T> &mt, const DevProblem<T> &P, const T *x, const T *b, T c, T &f,
                                                const T *cf);

// b(x), c(x) and, when asked, f(x) = F(x) + sum over trig terms T of
// (1/2) sigma^2 Lap T + b.grad T + c T, where Lap T = -|k|^2 T and
// d_d T = amp k_d cos(k_d x_d + ph_d) prod_{e != d} sin(k_e x_e + ph_e).
// The dense coefficients of F come from `cf` (a copy of P.fdense in LDS).
// Tabulated coefficients (bit q of `tab`: tabv[q] replaces b_0, b_1, b_2, c,
// f) are interpolated instead; the analytic f always uses the analytic b, c.
template <class T>
using Vec4 = T __attribute__((ext_vector_type(4)));

// The four 16-byte chunks of the pair records that hold a cell's corners
// (p00, p01, p10, p11 at rec[0..3]). Each lane of a quad whose four lanes are
// all active loads chunk m = lane & 3 of every quad member's record, so that a
// load instruction touches 16 cache lines rather than 64 (one per lane: the
// gather of divergent 64-byte records is what bounds these walks), and the
// wave's LDS block `tr` (4 x 64 chunks) hands each lane its own four chunks
// back. Lanes of other quads load their record themselves. The values are
// those of the direct loads, bit for bit.
template <class T>
__device__ __forceinline__ void pair_chunks(const Vec4<T> *base, uint32_t rec, Vec4<T> *tr, Vec4<T> &p00,
                                            Vec4<T> &p01, Vec4<T> &p10, Vec4<T> &p11)
{
    const int lane = __lane_id();
    const uint64_t act = __builtin_amdgcn_read_exec();
    if (tr != nullptr && ((act >> (lane & ~3)) & 0xfull) == 0xfull) {
        const uint32_t m = (uint32_t)lane & 3u;
        // record offset of quad lane k (quad_perm k,k,k,k), chunk m of it
        const uint32_t r0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)rec, 0x00, 0xf, 0xf, false);
        const uint32_t r1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)rec, 0x55, 0xf, 0xf, false);
        const uint32_t r2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)rec, 0xaa, 0xf, 0xf, false);
        const uint32_t r3 = (uint32_t)__builtin_amdgcn_mov_dpp((int)rec, 0xff, 0xf, 0xf, false);
        const Vec4<T> v0 = gload(base + r0 + m), v1 = gload(base + r1 + m), v2 = gload(base + r2 + m),
                      v3 = gload(base + r3 + m);
        tr[0 * 64 + lane] = v0;
        tr[1 * 64 + lane] = v1;
        tr[2 * 64 + lane] = v2;
        tr[3 * 64 + lane] = v3;
        // chunk m of quad lane k sits at tr[k * 64 + quad + m]
        const Vec4<T> *mine = tr + (lane & 3) * 64 + (lane & ~3);
        p00 = mine[0];
        p01 = mine[1];
        p10 = mine[2];
        p11 = mine[3];
    } else {
        p00 = gload(base + rec);
        p01 = gload(base + rec + 1);
        p10 = gload(base + rec + 2);
        p11 = gload(base + rec + 3);
    }
}

template <class T, int D, bool BIG>
__device__ __forceinline__ void coefficients(const MathOf<T> &mt, const DevProblem<T> &P, const T *x, T *b, T &c,
                                             T &f, bool want_f, const T *cf, uint32_t tab,
                                             Vec4<T> *tr = nullptr)
{
#pragma unroll
    for (int i = 0; i < D; ++i) {
        T v = P.b0[i];
#pragma unroll
        for (int j = 0; j < D; ++j) v = madd(P.B[i][j], x[j], v);
        b[i] = v;
    }
    T r2 = (T)0;
#pragma unroll
    for (int d = 0; d < D; ++d) r2 = madd(x[d], x[d], r2);
    c = madd(P.c_b, r2, P.c_a);
    if (tab & 64u) {  // every coefficient tabulated, interleaved
        int i[D];
        T w[D];
        grid_cell<T, D>(P.tabv[3], x, i, w);
        if (D == 2 && (tab & 128u)) {  // pair records of the cell's two lower corners: all four
            const uint32_t n0 = (uint32_t)P.tabv[3].n[0];
            Vec4<T> p00, p01, p10, p11;
            pair_chunks<T>(reinterpret_cast<const Vec4<T> *>(P.tab_fused), 2u * ((uint32_t)i[1] * n0 + (uint32_t)i[0]),
                           tr, p00, p01, p10, p11);
            b[0] = interp_corner_values<T>(p00.x, p10.x, p01.x, p11.x, w);
            b[1 % D] = interp_corner_values<T>(p00.y, p10.y, p01.y, p11.y, w);
            c = interp_corner_values<T>(p00.z, p10.z, p01.z, p11.z, w);
            if (want_f) f = interp_corner_values<T>(p00.w, p10.w, p01.w, p11.w, w);
            return;
        }
        const T *rec = P.tab_fused + cell_index<T, D>(P.tabv[3], i) * (size_t)((D + 2) << D);
#pragma unroll
        for (int d = 0; d < D; ++d) b[d] = interp_corners<T, D>(rec + (d << D), w);
        c = interp_corners<T, D>(rec + (D << D), w);
        if (want_f) f = interp_corners<T, D>(rec + ((D + 1) << D), w);
        return;
    }
    if (tab) {
        if (want_f && (tab & 16u)) {
            f = interp_cells<T, D>(P.tabv[4], x);
            want_f = false;
        }
        if (want_f) analytic_source<T, D, BIG>(mt, P, x, b, c, f, cf);
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (tab & (1u << d)) b[d] = interp_cells<T, D>(P.tabv[d], x);
        if (tab & 8u) c = interp_cells<T, D>(P.tabv[3], x);
        return;
    }
    if (want_f) analytic_source<T, D, BIG>(mt, P, x, b, c, f, cf);
}

// The analytic source for the analytic b and c.
template <class T, int D, bool BIG>
__device__ __forceinline__ void analytic_source(const MathOf<T> &mt, const DevProblem<T> &P, const T *x, const T *b, T c, T &f,
                                                const T *cf)
{
    T acc = (T)0;
    if (P.f_mode == kPolyDense)
        acc = dense_poly<T, D>(cf, x);
    else if (P.f_mode == kPolySparse)
        acc = poly_value<T, D>(P.fpoly, P.n_f, x);
    for (int m = 0; m < P.n_trig; ++m) {
        const DevTrig<T> &t = P.trig[m];
        T s[D], co[D];
#pragma unroll
        for (int d = 0; d < D; ++d) Arith<T>::template trig<BIG>(mt, P, m, d, x[d], s[d], co[d]);
        T prod = s[0];
#pragma unroll
        for (int d = 1; d < D; ++d) prod *= s[d];
        acc = madd(madd(c, t.amp, t.nhk2a), prod, acc);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int last = d == D - 1 ? D - 2 : D - 1;  // factor taken by the fused add
            T g = b[d] * t.ak[d] * co[d];
#pragma unroll
            for (int e = 0; e < D; ++e)
                if (e != d && e != last) g *= s[e];
            acc = madd(g, s[last], acc);
        }
    }
    f = acc;
}

// g = G + sum(trig) at a boundary point.
template <class T, int D, bool BIG>
__device__ __forceinline__ T boundary_value(const MathOf<T> &mt, const DevProblem<T> &P, const T *x, uint32_t tab)
{
    if (tab & 32u) return interp_cells<T, D>(P.tabv[5], x);  // tabulated g
    T u = poly_value<T, D>(P.gpoly, P.n_g, x);
    for (int m = 0; m < P.n_trig; ++m) {
        const DevTrig<T> &t = P.trig[m];
        T v = t.amp;
#pragma unroll
        for (int d = 0; d < D; ++d) v *= Arith<T>::template sine<BIG>(mt, P, m, d, x[d]);
        u += v;
    }
    return u;
}

// Cell of a grid holding x and the weights within it: cell index floor(t)
// clamped to [0, n - 2] and weight t - index clamped to [0, 1], for
// t = (x - lo) inv. Clamping t to [0, n - 1] first gives exactly those values
// (below 0: cell 0, weight 0; from n - 1 up: cell n - 2, weight 1) with one
// truncation and no floor.
template <class T, int D>
__device__ __forceinline__ void grid_cell(const GridView<T> &g, const T *x, int *i, T *w)
{
#pragma unroll
    for (int d = 0; d < D; ++d) {
        T t = (x[d] - g.lo[d]) * g.inv[d];
        t = med3(t, (T)0, g.top[d]);
        int id = (int)t;
        id = id < g.n[d] - 2 ? id : g.n[d] - 2;
        i[d] = id;
        w[d] = t - (T)id;
    }
}

// Bilinear (2D) / trilinear (3D) interpolation of a grid at x.
template <class T, int D>
__device__ __forceinline__ T interp(const GridView<T> &g, const T *x)
{
    int i[D];
    T w[D];
    grid_cell<T, D>(g, x, i, w);
    const int nx = g.n[0];
    if (D == 2) {
        const T *r0 = g.data + (size_t)i[1] * nx + i[0];
        const T *r1 = r0 + nx;
        const T l0 = madd(w[0], gload(r0 + 1), ((T)1 - w[0]) * gload(r0));
        const T l1 = madd(w[0], gload(r1 + 1), ((T)1 - w[0]) * gload(r1));
        return madd(w[1], l1, ((T)1 - w[1]) * l0);
    }
    const int ny = g.n[1];
    T acc = (T)0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        T layer = (T)0;
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
            const T *row = g.data + ((size_t)(i[2 % D] + dz) * ny + (i[1] + dy)) * nx + i[0];
            const T line = madd(w[0], gload(row + 1), ((T)1 - w[0]) * gload(row));
            layer = madd(dy ? w[1] : (T)1 - w[1], line, layer);
        }
        acc = madd(dz ? w[2 % D] : (T)1 - w[2 % D], layer, acc);
    }
    return acc;
}

// The same interpolation from the grid's cell layout: the corners of the
// cell come in one aligned vector load (two in 3D) instead of 2^D gathers;
// operands and operations are those of interp, so the value is identical.
// interp_cell_at takes the cell and weights already found by grid_cell (for
// several grids of one geometry).
template <class T, int D>
__device__ __forceinline__ size_t cell_index(const GridView<T> &g, const int *i)
{
    const size_t mx = (size_t)(g.n[0] - 1);
    if (D == 2) return (uint32_t)i[1] * (uint32_t)(g.n[0] - 1) + (uint32_t)i[0];
    return ((size_t)i[2 % D] * (size_t)(g.n[1] - 1) + i[1]) * mx + i[0];
}

// Bilinear interpolation from the four corner values of a cell ((0,0),
// (1,0), (0,1), (1,1)), the operations of interp_corners.
template <class T>
__device__ __forceinline__ T interp_corner_values(T c00, T c10, T c01, T c11, const T *w)
{
    const T l0 = madd(w[0], c10, ((T)1 - w[0]) * c00);
    const T l1 = madd(w[0], c11, ((T)1 - w[0]) * c01);
    return madd(w[1], l1, ((T)1 - w[1]) * l0);
}

// Interpolation from the 2^D corner values of one cell, stored together at p.
template <class T, int D>
__device__ __forceinline__ T interp_corners(const T *p, const T *w)
{
    typedef T V4 __attribute__((ext_vector_type(4)));
    if (D == 2) {
        const V4 c = gload(reinterpret_cast<const V4 *>(p));
        const T l0 = madd(w[0], c.y, ((T)1 - w[0]) * c.x);
        const T l1 = madd(w[0], c.w, ((T)1 - w[0]) * c.z);
        return madd(w[1], l1, ((T)1 - w[1]) * l0);
    }
    const V4 *cv = reinterpret_cast<const V4 *>(p);
    T acc = (T)0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {
        const V4 c = gload(cv + dz);
        const T line0 = madd(w[0], c.y, ((T)1 - w[0]) * c.x);
        const T line1 = madd(w[0], c.w, ((T)1 - w[0]) * c.z);
        T layer = madd((T)1 - w[1], line0, (T)0);
        layer = madd(w[1], line1, layer);
        acc = madd(dz ? w[2 % D] : (T)1 - w[2 % D], layer, acc);
    }
    return acc;
}

template <class T, int D>
__device__ __forceinline__ T interp_cell_at(const GridView<T> &g, const int *i, const T *w)
{
    return interp_corners<T, D>(g.cells + (cell_index<T, D>(g, i) << D), w);
}

template <class T, int D>
__device__ __forceinline__ T interp_cells(const GridView<T> &g, const T *x)
{
    int i[D];
    T w[D];
    grid_cell<T, D>(g, x, i, w);
    return interp_cell_at<T, D>(g, i, w);
}

// Domain, exit test and increment law: read from the problem and item at run
// time, or fixed at compile time for the common box / bridge / Gaussian case,
// which removes their branches and frees the registers of the other cases.
// `dense`: the form of the bridge test for walks in which many lanes of a
// wave are near a face at every step (short paths, a wide step against the
// box), where the per-lane branches of the other form would run at nearly
// every step; both give the same bits.
struct RuntimeMode {
    static constexpr bool kBigTrig = true;
    template <class T>
    __device__ static __forceinline__ int domain(const DevProblem<T> &P) { return P.domain; }
    template <class T>
    __device__ static __forceinline__ bool dense(const ItemCore<T> &a) { return a.dense_bridge != 0; }
    template <class T>
    __device__ static __forceinline__ int exit(const ItemCore<T> &a) { return a.exit_mode; }
    template <class T>
    __device__ static __forceinline__ int law(const ItemCore<T> &a) { return a.law; }
    template <class T>
    __device__ static __forceinline__ uint32_t tab(const DevProblem<T> &P) { return P.tab; }
};
template <bool DENSE>
struct BoxBridgeGaussT {
    static constexpr bool kBigTrig = false;
    template <class T>
    __device__ static constexpr int domain(const DevProblem<T> &) { return kBox; }
    template <class T>
    __device__ static constexpr int exit(const ItemCore<T> &) { return kExitBridge; }
    template <class T>
    __device__ static constexpr int law(const ItemCore<T> &) { return kLawGauss; }
    template <class T>
    __device__ static constexpr uint32_t tab(const DevProblem<T> &) { return 0u; }
    template <class T>
    __device__ static constexpr bool dense(const ItemCore<T> &) { return DENSE; }
};
using BoxBridgeGauss = BoxBridgeGaussT<false>;
using BoxBridgeGaussDense = BoxBridgeGaussT<true>;

template <class T, int D>
__device__ __forceinline__ T inner_distance(const DevProblem<T> &P, int domain, const T *x)
{
    if (domain == kBox) {
        T m = x[0] - P.lo[0];
        m = fmin(m, P.hi[0] - x[0]);
#pragma unroll
        for (int d = 1; d < D; ++d) {
            m = fmin(m, x[d] - P.lo[d]);
            m = fmin(m, P.hi[d] - x[d]);
        }
        return m;
    }
    T r2 = (T)0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const T t = x[d] - P.center[d];
        r2 = madd(t, t, r2);
    }
    return P.radius - Arith<T>::sqrt_(r2);
}

// Distance of a step's new point to the boundary (not positive outside).
template <class T, int D>
__device__ __forceinline__ T point_distance(const DevProblem<T> &P, int domain, const T *x)
{
    if (domain == kBox) return inner_distance<T, D>(P, kBox, x);
    T r2 = (T)0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const T t = x[d] - P.center[d];
        r2 = madd(t, t, r2);
    }
    return r2 < P.radius2 ? P.radius - Arith<T>::sqrt_(r2) : (T)-1;
}

template <class T, int D>
__device__ __forceinline__ void radial(const DevProblem<T> &P, const T *x, T *out)
{
    T r2 = (T)0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const T t = x[d] - P.center[d];
        r2 = madd(t, t, r2);
    }
    const T r = Arith<T>::sqrt_(r2);
#pragma unroll
    for (int d = 0; d < D; ++d)
        out[d] = r > (T)0 ? madd(P.radius, (x[d] - P.center[d]) / r, P.center[d])
                          : P.center[d] + (d == 0 ? P.radius : (T)0);
}

// Closest boundary point: inside a box the nearest face (ties to the lowest
// face index, faces ordered x-lo, x-hi, y-lo, ...), outside the clamp.
template <class T, int D>
__device__ __forceinline__ void project(const DevProblem<T> &P, int domain, const T *x, T *out)
{
    if (domain == kBall) {
        radial<T, D>(P, x, out);
        return;
    }
    bool inside = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        out[d] = x[d];
        inside = inside && (x[d] > P.lo[d]) && (x[d] < P.hi[d]);
    }
    if (inside) {
        int best = 0;
        T bd = x[0] - P.lo[0];
#pragma unroll
        for (int f = 1; f < 2 * D; ++f) {
            const int d = f >> 1;
            const T t = (f & 1) ? P.hi[d] - x[d] : x[d] - P.lo[d];
            if (t < bd) {
                bd = t;
                best = f;
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if ((best >> 1) == d) out[d] = (best & 1) ? P.hi[d] : P.lo[d];
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d) out[d] = fmin(fmax(out[d], P.lo[d]), P.hi[d]);
    }
}

// State of the path a lane is walking.
// RNG_TABLE: items may be merged solves with a per-node RNG table (batch
// kernel); the single-item kernel takes the stream tag from its item.
// Score of an ended path, written as its record r: phi = g(X_tau) Y + Z
// (plain), e = (g - u_prev)(X_tau) Y - R (correction), phi and phi + xi (Ito),
// and the exit step word.
template <class T, int D, int EST, class M>
__device__ __forceinline__ void score_path(const MathOf<T> &mt, const ItemCore<T> &a, const DevProblem<T> &P, const T *Xt, T Y, double Z,
                                           double R, uint32_t word, uint64_t r)
{
    const T gv = boundary_value<T, D, M::kBigTrig>(mt, P, Xt, M::tab(P));
    if (EST == kEstIto) {  // phi and phi + xi
        const double phi = madd((double)gv, (double)Y, Z);
        gstore(a.rec_phi + r, phi);
        gstore(a.rec_e + r, phi + R);
    } else if (a.score_plain) {
        gstore(a.rec_phi + r, madd((double)gv, (double)Y, Z));
    }
    if (EST == kEstCorrection) {
        const T up = interp<T, D>(a.u_prev, Xt);
        gstore(a.rec_e + r, madd((double)gv - (double)up, (double)Y, -R));
    }
    gstore(a.rec_steps + r, word);
}

// Ended paths of a wave waiting to be scored (batch kernel; dense-bridge and
// generic forms of the single-item kernel): a ring in the wave's LDS (dynamic
// shared memory, one ring per wave).
template <class T, int D>
struct EndedPath {
    T Xt[D];
    T Y;
    uint32_t word;  // exit step | capped bit
    double Z, R;
    uint64_t r;     // record index
};
constexpr uint32_t kEndRing = 128;  // holds a batch of 64 and the up to 64 ended at one turn
template <class T, int D>
struct EndRing {
    EndedPath<T, D> e[kEndRing];
};

// The same object behind a pointer that the optimiser cannot see through, in
// FP64: fields read after this are loaded again (by scalar loads) instead of
// being kept from an earlier part of the step in scalar registers, which the
// FP64 coefficients fill (each spilled value costs a v_writelane and a
// v_readlane per step).
template <class T, class X>
__device__ __forceinline__ const X &reread(const X &x)
{
    if constexpr (sizeof(T) == 8) {
        const uint64_t v = reinterpret_cast<uint64_t>(&x);
        uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
        asm volatile("" : "+s"(lo), "+s"(hi));
        typedef const __attribute__((address_space(4))) X ConstX;
        return *(const X *)(ConstX *)(((uint64_t)hi << 32) | lo);
    } else {
        return x;
    }
}

template <class T, int D, int EST, class M, bool RNG_TABLE, class KEYS = KeysOf<T>>
struct Walker {
    T X[D], Xt[D];
    T Y;
    T m;  // distance from X to the boundary (inside; cached between steps)
    double Z, R;  // R: sum h Y r (correction estimator) or xi (Ito control variate)
    uint64_t slot;
    uint32_t k, j, node, capped;
    uint32_t tag;  // stream tag of the path's solve (RNG_TABLE)

    // Stream tag of the path: its own with an RNG table, else the item's
    // (a wave-uniform scalar).
    __device__ __forceinline__ uint32_t stream(const ItemCore<T> &a) const { return RNG_TABLE ? tag : a.stream_tag; }
    uint32_t bb_blk;
    uint64_t bw01, bw23;  // cached bridge block, words (0,1) and (2,3)
    KEYS ks;
    MathOf<T> mt;
    const T *cf;          // dense source coefficients of the problem, in LDS
    Vec4<T> *tr;          // the wave's LDS block for gathering pair records (single-item kernel)

    // Starts path r (slot within the item) of item a. Returns false when it
    // ends before any step (a node inside the shift band of the shifted test).
    __device__ __forceinline__ bool start(const ItemCore<T> &a, const DevProblem<T> &P, uint64_t r, const uint32_t *node_rng)
    {
        slot = r;
        uint64_t jj;
        if (a.node_start == nullptr) {
            if (a.n_slots <= 0xffffffffull) {
                const uint32_t q = (uint32_t)r / (uint32_t)a.uniform_n;
                node = q;
                jj = (uint32_t)r - q * (uint32_t)a.uniform_n;
            } else {
                node = (uint32_t)(r / a.uniform_n);
                jj = r - (uint64_t)node * a.uniform_n;
            }
        } else {
            uint32_t lo = 0, hi = a.n_nodes;  // node_start[lo] <= r < node_start[hi]
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (gload(a.node_start + mid) <= r)
                    lo = mid;
                else
                    hi = mid;
            }
            node = lo;
            jj = r - gload(a.node_start + lo);
        }
        // the path's RNG counter: its node, stream and path index in its own solve
        j = (uint32_t)(a.path_offset + jj);
        uint32_t rnode = node;
        if (RNG_TABLE) {
            tag = a.stream_tag;
            if (node_rng) {
                typedef uint32_t U4 __attribute__((ext_vector_type(4)));
                const U4 v = gload(reinterpret_cast<const U4 *>(node_rng) + node);
                rnode = v.x;
                tag = v.y;
                j = v.z + (uint32_t)jj;
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) X[d] = (T)gload(a.nodes + (size_t)node * D + d);
        node = rnode;
        m = inner_distance<T, D>(P, M::domain(P), X);
        Y = (T)1;
        Z = 0.0;
        R = 0.0;
        k = 0;
        capped = 0;
        bb_blk = 0xffffffffu;
        if (M::exit(a) == kExitShift && m <= a.gm_thresh) {
            project<T, D>(P, M::domain(P), X, Xt);
            return false;
        }
        return true;
    }

    // Bridge block of step s for every active lane when some lane needs it
    // and does not hold it (wave-uniform branch).
    __device__ __forceinline__ void bridge_block(const ItemCore<T> &a, uint32_t s, bool need)
    {
        const uint32_t blk = s >> 2;
        if (__ballot(need && blk != bb_blk)) {
            const Block4 q = philox(blk, j, node, stream(a) | 1u, ks);
            bw01 = (uint64_t)q.w0 | ((uint64_t)q.w1 << 32);
            bw23 = (uint64_t)q.w2 | ((uint64_t)q.w3 << 32);
            bb_blk = blk;
        }
    }
    // The bridge uniform of step s: from the block bridge_block has drawn
    // (boundary-dense walks), or drawn here for this lane.
    __device__ __forceinline__ T bridge_uniform(const ItemCore<T> &a, uint32_t s)
    {
        if (!M::dense(a)) {
            const uint32_t blk = s >> 2;
            if (blk != bb_blk) {
                const Block4 q = philox(blk, j, node, stream(a) | 1u, ks);
                bw01 = (uint64_t)q.w0 | ((uint64_t)q.w1 << 32);
                bw23 = (uint64_t)q.w2 | ((uint64_t)q.w3 << 32);
                bb_blk = blk;
            }
        }
        // word s mod 4, picked with a shift (a select chain becomes a stack array)
        const uint32_t w = (uint32_t)(((s & 2) ? bw23 : bw01) >> ((s & 1) << 5));
        return Arith<T>::unif_bridge(w);
    }

    // The increments of one step from the words that feed them.
    __device__ __forceinline__ void draw(const ItemCore<T> &a, uint32_t wa, uint32_t wb, uint32_t wc, uint32_t wd,
                                         T *n) const
    {
        if (M::law(a) == kLawGauss) {
            Arith<T>::box_muller(mt, wa, wb, n[0], n[1]);
            if (D == 3) n[2 % D] = Arith<T>::box_muller_cos(mt, wc, wd);
        } else {
            n[0] = (wa >> 31) ? (T)1 : (T)-1;
            n[1] = (wb >> 31) ? (T)1 : (T)-1;
            if (D == 3) n[2 % D] = (wc >> 31) ? (T)1 : (T)-1;
        }
    }

    template <class A>
    __device__ __forceinline__ bool step(const A &a, const DevProblem<T> &P, uint32_t wa,
                                         uint32_t wb, uint32_t wc, uint32_t wd)
    {
        T n[D];
        draw(a, wa, wb, wc, wd, n);
        return advance(a, P, n);
    }

    // One step of the walk with its increments n. Returns false when the path
    // has ended (exit point in Xt). Everything that ends a path (leaving the
    // domain, a live bridge face, the shift band of the next step, the step
    // cap) goes through one rarely taken branch.
    template <class A>
    __device__ __forceinline__ bool advance(const A &a0, const DevProblem<T> &P0, const T *n)
    {
        T b[D], c, f = (T)0;
        {
            const A &a = reread<T>(a0);
            const DevProblem<T> &P = reread<T>(P0);
            coefficients<T, D, M::kBigTrig>(mt, P, X, b, c, f, EST == kEstIto || a.score_plain != 0, cf, M::tab(P),
                               RNG_TABLE ? nullptr : tr);
        }
        const A &a = reread<T>(a0);
        const DevProblem<T> &P = reread<T>(P0);
        const T hY = a.h * Y;
        if (EST == kEstIto || a.score_plain) Z -= (double)(hY * f);
        if (EST == kEstCorrection) R += (double)(hY * interp_cells<T, D>(a.resid, X));
        if constexpr (EST == kEstIto) {
            // eq. F:xiControlVariate, left-point rule: -Y sigma grad(u~)(X_k)
            // . sqrt(h) N_k, with this step's normals; the gradient grids
            // share one geometry, so the cell is found once, and their cell
            // layouts are interleaved, so its corners of every component are
            // one record (32 bytes in 2D FP32: one L2 request, not two)
            int gi[D];
            T gw[D];
            grid_cell<T, D>(a.grad[0], X, gi, gw);
            const T *rec = a.grad[0].cells + cell_index<T, D>(a.grad[0], gi) * (size_t)(D << D);
            T gn = (T)0;
#pragma unroll
            for (int d = 0; d < D; ++d) gn = madd(interp_corners<T, D>(rec + (d << D), gw), n[d], gn);
            R -= (double)((Y * a.sig_sqh) * gn);
        }
        Y = madd(hY, c, Y);
        T Xn[D];
#pragma unroll
        for (int d = 0; d < D; ++d) Xn[d] = madd(a.sig_sqh, n[d], madd(a.h, b[d], X[d]));
        const uint32_t s = k;
        k = k + 1;

        const T mn = point_distance<T, D>(P, M::domain(P), Xn);
        const bool shift = M::exit(a) == kExitShift;
        // Bridge: a face f is live when a_f a'_f 2/(sigma^2 h) <= 36 ln 2; since
        // a_f >= m and a'_f >= mn, no face is live unless m mn passes that test.
        const bool out = !shift && !(mn > (T)0);
        const bool maybe = M::exit(a) == kExitBridge && m * mn * a.two_over_s2h <= a.bridge_thresh;
        if (M::exit(a) == kExitBridge && M::dense(a)) bridge_block(a, s, maybe);
        const bool next_stop = k == a.max_steps || (shift && mn <= a.gm_thresh);
        if (out || maybe || next_stop) {
            if (out) {  // outside (or on) the boundary: the nearest point is the clamp
                if (M::domain(P) == kBox) {
#pragma unroll
                    for (int d = 0; d < D; ++d) Xt[d] = med3(Xn[d], P.lo[d], P.hi[d]);
                } else {
                    radial<T, D>(P, Xn, Xt);
                }
                return false;
            }
            if (maybe && bridge_exit(a, P, Xn, mn, s)) return false;
            if (shift && mn <= a.gm_thresh) {  // stops before the next step
                project<T, D>(P, M::domain(P), Xn, Xt);
                return false;
            }
            if (k == a.max_steps) {
                capped = 1;
                project<T, D>(P, M::domain(P), Xn, Xt);
                return false;
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) X[d] = Xn[d];
        m = mn;
        return true;
    }

    // Brownian-bridge exit between X and Xn (both inside, Xn at distance mn).
    // Per flat face P(cross) = exp(-2 a a' / (sigma^2 h)), faces combined as
    // independent; exit onto the live face with the largest probability.
    __device__ __forceinline__ bool bridge_exit(const ItemCore<T> &a, const DevProblem<T> &P,
                                                const T *Xn, T mn, uint32_t s)
    {
        if (M::domain(P) == kBox && M::dense(a)) {
            // Per axis the face with the smaller argument: unless both faces
            // of the axis are live (a box narrow against the step), it is the
            // only one that can be, so one exponential per axis gives the
            // combined probability and the exit face of the face-by-face rule
            // (live faces combined in face order, the exit face the first of
            // the largest probabilities), with the same operands and
            // roundings. Lanes with both faces of an axis live take every face
            // in turn.
            T alo[D], ahi[D], ad[D];
            bool both = false, live[D], up[D];
            int nlive = 0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                alo[d] = ((X[d] - P.lo[d]) * (Xn[d] - P.lo[d])) * a.two_over_s2h;
                ahi[d] = ((P.hi[d] - X[d]) * (P.hi[d] - Xn[d])) * a.two_over_s2h;
                both = both || (alo[d] <= a.bridge_thresh && ahi[d] <= a.bridge_thresh);
                up[d] = ahi[d] < alo[d];
                ad[d] = up[d] ? ahi[d] : alo[d];
                live[d] = ad[d] <= a.bridge_thresh;
                nlive += live[d] ? 1 : 0;
            }
            // one live axis (the usual case): its face alone
            T amin = ad[0];
            int bestf = up[0] ? 1 : 0;
#pragma unroll
            for (int d = 1; d < D; ++d) {
                amin = live[d] ? ad[d] : amin;
                bestf = live[d] ? 2 * d + (up[d] ? 1 : 0) : bestf;
            }
            T Pe = nlive ? Arith<T>::exp_neg(amin) : (T)0;
            if (nlive > 1) {  // near a corner: the live axes in order
                T bestp = (T)0;
                Pe = (T)0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const T p = Arith<T>::exp_neg(ad[d]);
                    Pe = live[d] ? madd(p, (T)1 - Pe, Pe) : Pe;
                    const bool better = live[d] && p > bestp;
                    bestp = better ? p : bestp;
                    bestf = better ? 2 * d + (up[d] ? 1 : 0) : bestf;
                }
            }
            if (__builtin_expect(__ballot(both) != 0, 0)) {
                if (both) {  // every live face, in face order
                    Pe = (T)0;
                    T bestp = (T)0;
#pragma unroll
                    for (int q = 0; q < 2 * D; ++q) {
                        const T aq = (q & 1) ? ahi[q >> 1] : alo[q >> 1];
                        const bool live = aq <= a.bridge_thresh;
                        const T p = Arith<T>::exp_neg(aq);
                        Pe = live ? madd(p, (T)1 - Pe, Pe) : Pe;
                        const bool better = live && p > bestp;
                        bestp = better ? p : bestp;
                        bestf = better ? q : bestf;
                    }
                }
            }
            if (bridge_uniform(a, s) < Pe) {
#pragma unroll
                for (int d = 0; d < D; ++d)
                    Xt[d] = (bestf >> 1) == d ? ((bestf & 1) ? P.hi[d] : P.lo[d]) : Xn[d];
                return true;
            }
            return false;
        }
        if (M::domain(P) == kBox) {  // few lanes near a face: per face, one exponential for one live face
            T arg[2 * D];
            T amin = (T)0;
            int fmin = -1, nlive = 0;
#pragma unroll
            for (int q = 0; q < 2 * D; ++q) {
                const int d = q >> 1;
                const T prod = (q & 1) ? (P.hi[d] - X[d]) * (P.hi[d] - Xn[d])
                                       : (X[d] - P.lo[d]) * (Xn[d] - P.lo[d]);
                arg[q] = prod * a.two_over_s2h;
                if (arg[q] <= a.bridge_thresh) {
                    ++nlive;
                    if (fmin < 0 || arg[q] < amin) {
                        amin = arg[q];
                        fmin = q;
                    }
                }
            }
            if (nlive == 0) return false;
            // One live face (the usual case): P is its p and it is the exit
            // face. Several (near a corner): combine them in face order.
            T Pe = Arith<T>::exp_neg(amin);
            int bestf = fmin;
            if (nlive > 1) {
                T bestp = (T)-1;
                Pe = (T)0;
#pragma unroll
                for (int q = 0; q < 2 * D; ++q) {
                    if (arg[q] <= a.bridge_thresh) {
                        const T p = Arith<T>::exp_neg(arg[q]);
                        Pe = madd(p, (T)1 - Pe, Pe);
                        if (p > bestp) {
                            bestp = p;
                            bestf = q;
                        }
                    }
                }
            }
            if (bridge_uniform(a, s) < Pe) {
#pragma unroll
                for (int d = 0; d < D; ++d)
                    Xt[d] = (bestf >> 1) == d ? ((bestf & 1) ? P.hi[d] : P.lo[d]) : Xn[d];
                return true;
            }
            return false;
        }
        const T Pe = Arith<T>::exp_neg(m * mn * a.two_over_s2h);
        if (bridge_uniform(a, s) < Pe) {
            radial<T, D>(P, Xn, Xt);
            return true;
        }
        return false;
    }

    // Score the ended path and write its record at slot - rec_base.
    __device__ __forceinline__ void finish(const ItemCore<T> &a, const DevProblem<T> &P,
                                           uint64_t rec_base)
    {
        score_path<T, D, EST, M>(mt, a, P, Xt, Y, Z, R, k | (capped ? kCappedBit : 0u), slot - rec_base);
    }

    // The walking path's state, for another kernel to walk on from (only
    // between blocks of random numbers: k is even in 2D).
    __device__ __forceinline__ void hand_over(TailState<T, D> &t, uint32_t stream_tag) const
    {
#pragma unroll
        for (int d = 0; d < D; ++d) gstore(&t.X[d], X[d]);
        gstore(&t.Y, Y);
        gstore(&t.m, m);
        gstore(&t.Z, Z);
        gstore(&t.R, R);
        gstore(&t.slot, slot);
        gstore(&t.k, k);
        gstore(&t.j, j);
        gstore(&t.node, node);
        gstore(&t.tag, RNG_TABLE ? tag : stream_tag);
    }
    __device__ __forceinline__ void take_over(const TailState<T, D> &t)
    {
#pragma unroll
        for (int d = 0; d < D; ++d) X[d] = gload(&t.X[d]);
        Y = gload(&t.Y);
        m = gload(&t.m);
        Z = gload(&t.Z);
        R = gload(&t.R);
        slot = gload(&t.slot);
        k = gload(&t.k);
        j = gload(&t.j);
        node = gload(&t.node);
        tag = gload(&t.tag);
        capped = 0;
        bb_blk = 0xffffffffu;
    }

    // What scoring the ended path needs, for scoring later from the ring.
    __device__ __forceinline__ void stash(EndedPath<T, D> &e, uint64_t rec_base) const
    {
#pragma unroll
        for (int d = 0; d < D; ++d) e.Xt[d] = Xt[d];
        e.Y = Y;
        e.word = k | (capped ? kCappedBit : 0u);
        e.Z = Z;
        e.R = R;
        e.r = slot - rec_base;
    }
};

// Item whose slot range holds group slot s (items are sorted, non-empty
// ranges never overlap). Wave-uniform: a scalar binary search.
template <class T>
__device__ __forceinline__ int find_item(const ItemDesc<T> *__restrict__ items, int n, uint64_t s)
{
    int lo = 0, hi = n;  // items[lo].slot_begin <= s < items[hi].slot_begin
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (items[mid].slot_begin <= s)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Per-item queues of a batch launch. A wave walks the paths of one item at a
// time and may move to another item only once all its lanes are idle, so it
// takes its tickets from its own item's queue for as long as that has slots:
// a single shared queue would hand it the next slots of the whole launch,
// which with many waves lie in another item almost every time and would make
// it wait for its slowest lane at nearly every refill. Waves start spread over
// the items in proportion to their slots; a wave whose item has run dry looks
// for the next item that still has slots (64 candidates per probe).
// The group-walk kernel's queues hold the paths handed over to it instead
// (TAIL): item q's entries [tail_off[q], tail_off[q] + tail_n[q]).
template <class T, bool TAIL = false>
struct ItemQueue {
    __device__ static __forceinline__ void range(const LaunchArgs &L, uint32_t k, uint32_t &lo, uint32_t &hi)
    {
        if (TAIL && L.tail) {
            lo = L.tail_off[k];
            hi = min(lo + L.tail_n[k], L.tail_off[k + 1]);
        } else {
            lo = L.seg[2 * k];
            hi = L.seg[2 * k + 1];
        }
    }

    int cur = -1;                     // item of the wave (wave-uniform)
    uint32_t seg_lo = 0, seg_hi = 0;  // its launch-relative slots
    uint32_t next = 0, end = 0;       // the wave's current ticket
    uint32_t grab = 1;                // paths of a ticket (TAIL)
    bool dry = true;                  // the current item's queue is used up
    bool done = false;                // every queue of the launch is used up

    // Next ticket of the current item's queue, or dry.
    __device__ __forceinline__ void take(const LaunchArgs &L, int lane)
    {
        uint32_t base = 0;
        const uint32_t n = TAIL ? grab : (uint32_t)L.grab;
        if (lane == 0) base = atomicAdd(L.counter + (cur - L.item_lo), n);
        base = __builtin_amdgcn_readfirstlane(base);
        if (base < seg_hi - seg_lo) {
            next = seg_lo + base;
            end = min(next + n, seg_hi);
        } else {
            dry = true;
        }
    }

    // Moves the (idle) wave to an item with slots left, starting with queue k
    // and then probing the ones after it, and takes a ticket there; done when
    // none has slots left. Counters only grow, so every failed attempt means
    // another wave took those slots and the search ends.
    __device__ __forceinline__ void move(const ItemDesc<T> *__restrict__ items, const LaunchArgs &L, int lane,
                                         uint32_t k)
    {
        const uint32_t n = L.n_seg;
        for (;;) {
            cur = __builtin_amdgcn_readfirstlane(L.item_lo + (int)k);
            range(L, k, seg_lo, seg_hi);
            if (TAIL) {  // a wave's share of the item's paths (if all items have as many), a power of two
                const uint32_t waves = gridDim.x * (blockDim.x >> 6);
                const uint64_t share = ((uint64_t)(seg_hi - seg_lo) * n + waves - 1) / waves;
                grab = share > 8 ? 16u : share <= 1 ? 1u : 1u << (32 - __builtin_clz((uint32_t)share - 1));
                grab = __builtin_amdgcn_readfirstlane(grab);
            }
            dry = false;
            take(L, lane);
            if (!dry) return;
            // the probe window nearest after k that has slots left; in it, the
            // item with the most slots left (spreads the waves that move)
            uint32_t found = n;
            for (uint32_t off = 1; off < n && found == n; off += 64) {
                const uint32_t i = off + (uint32_t)lane;
                uint32_t key = 0;  // slots left (capped) << 6 | 63 - lane: the largest wins
                if (i < n) {
                    uint32_t kk = k + i;
                    if (kk >= n) kk -= n;
                    uint32_t lo, hi;
                    range(L, kk, lo, hi);
                    const uint32_t taken =
                        __hip_atomic_load(L.counter + kk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (taken < hi - lo) key = (min(hi - lo - taken, 0x3ffffffu) << 6) | (uint32_t)(63 - lane);
                }
#pragma unroll
                for (int x = 32; x >= 1; x >>= 1) key = max(key, (uint32_t)__shfl_xor((int)key, x));
                key = __builtin_amdgcn_readfirstlane(key);  // every lane holds the maximum
                if (key) {
                    found = k + off + (63 - (key & 63));
                    if (found >= n) found -= n;
                }
            }
            if (found == n) {
                done = true;
                return;
            }
            k = found;
        }
    }
};

}  // namespace
}  // namespace pdd
