// Double-precision exp and erf for the solver kernels, the pair
// (erf S, exp(-S^2)) of a split flux, and the cross-lane sums of their points.
//
// exp: x = k ln2 + r with k = rint(x / ln2) and r formed with ln2 split into
// a high and a low part, e^r = 1 + r + r^2 Q(r) with Q of degree 10, scaled
// by 2^k.  erf: x P(x^2) with P of degree 11 for |x| < 1, and beyond
// 1 - exp(-x^2) erfcx(x).  The coefficients (lskum_math_coef.h) are near-minimax Chebyshev
// fits written by gen_lskum_math.py; evaluated with fused multiply-adds both
// are within one unit in the last place of the correctly rounded values on
// the reduced ranges.
//
// The coefficients are read from __constant__ tables: the loads are uniform,
// hoisted out of the neighbour loops, and the values stay in scalar
// registers, so every Horner step is one v_fma_f64 with a scalar operand.
// Written with literal coefficients, each step costs two more instructions
// (the literal is rebuilt in a register pair before every step), which made
// the library's polynomials and literal-coefficient versions of these about
// 10% slower in the residual kernel.
#pragma once
// Defines __constant__ tables: include it from one translation unit only
// (the solver kernels' lskum_device.hip).

#include <hip/hip_runtime.h>

#include "lskum_math_coef.h"

namespace lskum {

__constant__ double cExpQ[11] = {kExpQ[0], kExpQ[1], kExpQ[2], kExpQ[3], kExpQ[4], kExpQ[5],
                                 kExpQ[6], kExpQ[7], kExpQ[8], kExpQ[9], kExpQ[10]};
__constant__ double cExpN[13] = {kExpN[0], kExpN[1], kExpN[2],  kExpN[3],  kExpN[4],
                                 kExpN[5], kExpN[6], kExpN[7],  kExpN[8],  kExpN[9],
                                 kExpN[10], kExpN[11], kExpN[12]};
static_assert(kExpN[10] == 0.5 && kExpN[12] == 1.0, "inline operands of exp_neg_poly");
__constant__ double cErfP[12] = {kErfP[0], kErfP[1], kErfP[2], kErfP[3], kErfP[4],  kErfP[5],
                                 kErfP[6], kErfP[7], kErfP[8], kErfP[9], kErfP[10], kErfP[11]};

// round-to-nearest-even double -> int32 with the hardware's defined result
// out of range (saturated; 0 for NaN), where a C++ conversion is undefined
__device__ __forceinline__ int cvt_i32_sat(double k) {
    int r;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(k));
    return r;
}

__device__ __forceinline__ double exp_fast(double x) {
    const double k = rint(x * kLog2e);
    double r = fma(-k, kLn2Hi, x);
    r = fma(-k, kLn2Lo, r);
    // the first step with literals: two fewer scalar register pairs
    double q = fma(kExpQ[0], r, kExpQ[1]);
#pragma unroll
    for (int i = 2; i < 11; ++i) q = fma(q, r, cExpQ[i]);
    const double e = 1.0 + fma(r * r, q, r);
    return ldexp(e, cvt_i32_sat(k));
}

// The leading coefficients of the two polynomials below, held in vector
// registers: a fused step takes one scalar operand, so the first step of a
// polynomial would rebuild its leading coefficient each time.
struct PolyLead {
    double erf, exp;
};
template <class T = double>  // unused by single precision
__device__ __forceinline__ PolyLead poly_lead() {
    PolyLead l{kErfP[0], kExpN[0]};
    if constexpr (std::is_same_v<T, double>) asm volatile("" : "+v"(l.erf), "+v"(l.exp));
    return l;
}

__device__ __forceinline__ double exp_neg_poly(double u, const PolyLead& l) {
    double e = fma(l.exp, u, cExpN[1]);
#pragma unroll
    for (int i = 2; i < 10; ++i) e = fma(e, u, cExpN[i]);
    e = fma(e, u, 0.5);
    e = fma(e, u, cExpN[11]);
    return fma(e, u, 1.0);
}

// e^x by the same polynomial on the reduced argument -r.
__device__ __forceinline__ double exp_lead(double x, const PolyLead& l) {
    const double k = rint(x * kLog2e);
    double u = fma(k, kLn2Hi, -x);
    u = fma(k, kLn2Lo, u);
    return ldexp(exp_neg_poly(u, l), cvt_i32_sat(k));
}

// erf(S) and e^(1/2) exp(-t), t = S^2, for |S| < 1 by two polynomials in t: on
// this range exp(-t) needs no range reduction, and callers fold the factor
// kExpHalf = e^(-1/2) into a constant of their own (13 instructions where the
// general exp has 19).
__device__ __forceinline__ void erf_exp_unit(double S, double t, const PolyLead& l, double& er,
                                             double& g) {
    double p = fma(l.erf, t, cErfP[1]);
#pragma unroll
    for (int i = 2; i < 12; ++i) p = fma(p, t, cErfP[i]);
    er = S * p;
    g = exp_neg_poly(t - 0.5, l);
}

// erf(S) and exp(-t) for 1 <= |S| (and NaN, which both results keep): erf =
// sign(S) (1 - exp(-t) erfcx(|S|)), erfcx by a polynomial in v = (|S| - 3)/
// (|S| + 3) up to 6, beyond which the product is below half a unit of the last
// place.  Rare in subsonic flow: literal coefficients, so that it holds no
// registers.
__device__ __forceinline__ void erf_exp_outer(double S, double t, double& er, double& g) {
    const double x = fmin(fabs(S), 6.0), d = x + 3.0;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double v = (x - 3.0) * r;
    double w = kErfcxW[0];
#pragma unroll
    for (int i = 1; i < 15; ++i) w = fma(w, v, kErfcxW[i]);
    g = exp_fast(-t);
    er = copysign(fma(-g, w, 1.0), S);
}

// erf(S) and exp(-S^2)
__device__ __forceinline__ void erf_exp(double S, double& er, double& g) {
    const double t = S * S;
    if (t < 1.0) {
        erf_exp_unit(S, t, PolyLead{kErfP[0], kExpN[0]}, er, g);
        g *= kExpHalf;
    } else {
        erf_exp_outer(S, t, er, g);
    }
}

// single precision, for the mixed sweeps
__device__ __forceinline__ void erf_exp(float S, float& er, float& g) {
    er = erff(S);
    g = expf(-(S * S));
}

}  // namespace lskum
