// Boys function tables, computed by the compiler.
//
// H(T) = erf(sqrt T)/sqrt T = (2/sqrt(pi)) F0(T) is tabulated about T_k = k h; a kernel reads
// its rows with the argument on the grid (T' = T / h) and its own accumulator scale, so the
// rows are stored that way: coefficient m times h^m sqrt(h) and the scale.  The tables depend
// on nothing but constants of the build, so they are part of the code object: computing them
// on the device took a launch of 16 us per call (a serial series per row), and scaling them
// again in every workgroup a loop of divisions.
#pragma once

#include "hfk_internal.hpp"

namespace hfk {

struct BoysRows {
    double c[kBoysOrderG + 1];
};

// exp(-x), x >= 0: x = n ln 2 + r, Taylor series of exp(-r), |r| <= ln 2 / 2.
constexpr double boys_expm(double x)
{
    const double ln2_hi = 0x1.62e42fefa0000p-1, ln2_lo = 0x1.cf79abc9e3b3ap-40;
    const int n = (int)(x * 1.4426950408889634 + 0.5);
    const double r = (x - n * ln2_hi) - n * ln2_lo;
    double term = 1.0, sum = 1.0;
    for (int i = 1; i < 24; ++i) {
        term *= -r / i;
        sum += term;
    }
    for (int i = 0; i < n; ++i) sum *= 0.5;
    return sum;
}

// F_0 .. F_order at T: the highest order from its positive Kummer series (no cancellation),
// the lower ones from the downward recursion F_m = (2T F_{m+1} + e^-T) / (2m + 1), which is
// stable in that direction.
constexpr BoysRows boys_functions(double T, int order)
{
    BoysRows f{};
    const double et = boys_expm(T);
    double term = 1.0 / (2.0 * order + 1.0), sum = term;
    for (int i = 1; i < 400; ++i) {
        term *= 2.0 * T / (2.0 * order + 2.0 * i + 1.0);
        sum += term;
        if (term < 1e-18 * sum) break;
    }
    f.c[order] = et * sum;
    for (int m = order - 1; m >= 0; --m) f.c[m] = (2.0 * T * f.c[m + 1] + et) / (2.0 * m + 1.0);
    return f;
}

// Taylor coefficients of H about T: (2/sqrt(pi)) (-1)^m F_m(T) / m! for m < order, and with
// shift = 1 those of F1's part: (2/sqrt(pi)) (-1)^m F_{m+1}(T) / m!.
constexpr BoysRows boys_taylor(double T, int order, int shift)
{
    const BoysRows f = boys_functions(T, order);
    BoysRows t{};
    double fact = 1.0;
    for (int m = 0; m < order; ++m) {
        if (m > 0) fact *= m;
        t.c[m] = kTwoOverSqrtPi * ((m & 1) ? -1.0 : 1.0) * f.c[m + shift] / fact;
    }
    return t;
}

// FP64 forward rows: degree 5, the Chebyshev economisation on [T_k - h/2, T_k + h/2] of the
// degree-7 Taylor row; with u = (T - T_k) / r, r = h/2 (b_m = c_m r^m), T7(u)/64 and T6(u)/32
// are dropped, keeping the lower-degree parts of u^7 and u^6:
//   u^7 = (T7 + 112 u^5 - 56 u^3 + 7 u) / 64,   u^6 = (T6 + 48 u^4 - 18 u^2 + 1) / 32
// Scale: h^m sqrt(h) times -2 (the forward kernel's accumulator).
struct BoysForward64 {
    double v[kBoysGrid * kBoysStride];
};
constexpr BoysForward64 make_boys_forward64()
{
    static_assert(kBoysOrder == 6 && kBoysOrderG == 8, "degree-7 rows economised to degree 5");
    BoysForward64 t{};
    for (int k = 0; k < kBoysGrid; ++k) {
        const BoysRows a = boys_taylor(k * kBoysH, kBoysOrderG, 0);
        const double r = 0.5 * kBoysH;
        double b[8] = {}, rm = 1.0;
        for (int m = 0; m < 8; ++m) {
            b[m] = a.c[m] * rm;
            rm *= r;
        }
        b[5] += b[7] * (112.0 / 64.0);
        b[3] -= b[7] * (56.0 / 64.0);
        b[1] += b[7] * (7.0 / 64.0);
        b[4] += b[6] * (48.0 / 32.0);
        b[2] -= b[6] * (18.0 / 32.0);
        b[0] += b[6] * (1.0 / 32.0);
        rm = 1.0;
        double sc = kSqrtBoysH * -2.0;
        for (int m = 0; m < kBoysStride; ++m) {
            t.v[k * kBoysStride + m] = b[m] / rm * sc;
            rm *= r;
            sc *= kBoysH;
        }
    }
    return t;
}

// The direct form's FP64 rows: the same without any scale.
struct BoysPlain64 {
    double v[kBoysGrid * kBoysStride];
};
constexpr BoysPlain64 make_boys_plain64()
{
    const BoysForward64 f = make_boys_forward64();
    BoysPlain64 t{};
    for (int k = 0; k < kBoysGrid; ++k) {
        double sc = kSqrtBoysH * -2.0;
        for (int m = 0; m < kBoysStride; ++m) {
            t.v[k * kBoysStride + m] = f.v[k * kBoysStride + m] / sc;
            sc *= kBoysH;
        }
    }
    return t;
}

// FP64 gradient rows: H of degree 7 (its derivative gives g(T) = -(4/sqrt(pi)) F1(T) = 2 H'(T)),
// rows of kBoysStrideG values with a zero pad; scale h^m sqrt(h) times -2.
struct BoysGrad64 {
    double v[kBoysGrid * kBoysStrideG];
};
constexpr BoysGrad64 make_boys_grad64()
{
    BoysGrad64 t{};
    for (int k = 0; k < kBoysGrid; ++k) {
        const BoysRows a = boys_taylor(k * kBoysH, kBoysOrderG, 0);
        double sc = kSqrtBoysH * -2.0;
        for (int m = 0; m < kBoysOrderG; ++m) {
            t.v[k * kBoysStrideG + m] = a.c[m] * sc;
            sc *= kBoysH;
        }
    }
    return t;
}

// FP32 rows of degree 3: H's (scale h^m sqrt(h)), then g's, -(4/sqrt(pi)) F1 (scale
// h^m h^(3/2)), rounded once from FP64; plain: H's without a scale (the direct form).
struct BoysFloat {
    float v[2 * kBoysGridF * kBoysStrideF];
};
constexpr BoysFloat make_boys_float(bool plain)
{
    BoysFloat t{};
    for (int k = 0; k < kBoysGridF; ++k) {
        const BoysRows a = boys_taylor(k * kBoysHF, kBoysOrderF, 0), g = boys_taylor(k * kBoysHF, kBoysOrderF, 1);
        double sc = 0.25;   // sqrt(1/16)
        for (int m = 0; m < kBoysOrderF; ++m) {
            t.v[k * kBoysStrideF + m] = (float)(plain ? a.c[m] : a.c[m] * sc);
            t.v[(kBoysGridF + k) * kBoysStrideF + m] = (float)(-2.0 * g.c[m] * sc * kBoysHF);
            sc *= kBoysHF;
        }
    }
    return t;
}

// Fills `len` values of a workgroup's table from a constant table.
template <typename R>
__device__ inline void load_boys(R *__restrict__ dst, const R *__restrict__ src, int len, int tid, int threads)
{
    for (int x = tid; x < len; x += threads) dst[x] = src[x];
}

}  // namespace hfk
