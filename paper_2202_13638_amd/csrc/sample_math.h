// The exponential of the kernel row, shared by the sample evaluation (gp_step.hip) and the rollout with one workgroup per
// trajectory (rollout.hip), which must give the same bits.
#pragma once

#include <hip/hip_runtime.h>

namespace {

// 2^t without a table: split off the integer part, evaluate 2^(f/2) for |f| <= 1/2 with a degree-7
// polynomial and square it (relative error 4e-13), scale with ldexp.  Twelve vector instructions and
// no LDS access.  c7 comes in a scalar and c6 in a vector register: the first Horner step is then a
// single three-operand FMA (an FMA takes at most one scalar operand).
struct exp2_coefficients {
    double c7 = 1.192611307487823e-07, c6 = 2.409383341728244e-06, c5 = 4.1667353769980764e-05, c4 = 0.0006011326659205452,
           c3 = 0.006938013583872582, c2 = 0.060056626759929704, c1 = 0.3465735902799663, c0 = 0.9999999999998426;
};

__device__ __forceinline__ double exp2_poly(double t, const exp2_coefficients &c)
{
    const double n = rint(t);
    const double f = t - n;                       // exact, |f| <= 1/2
    double p = fma(c.c7, f, c.c6);
    p = fma(p, f, c.c5);
    p = fma(p, f, c.c4);
    p = fma(p, f, c.c3);
    p = fma(p, f, c.c2);
    p = fma(p, f, c.c1);
    p = fma(p, f, c.c0);
    return ldexp(p * p, (int)n);
}

// for two arguments side by side
__device__ __forceinline__ void exp2_poly2(double t0, double t1, const exp2_coefficients &c, double &k0, double &k1)
{
    const double n0 = rint(t0), n1 = rint(t1);
    const double f0 = t0 - n0, f1 = t1 - n1;
    double p0 = fma(c.c7, f0, c.c6), p1 = fma(c.c7, f1, c.c6);
    p0 = fma(p0, f0, c.c5); p1 = fma(p1, f1, c.c5);
    p0 = fma(p0, f0, c.c4); p1 = fma(p1, f1, c.c4);
    p0 = fma(p0, f0, c.c3); p1 = fma(p1, f1, c.c3);
    p0 = fma(p0, f0, c.c2); p1 = fma(p1, f1, c.c2);
    p0 = fma(p0, f0, c.c1); p1 = fma(p1, f1, c.c1);
    p0 = fma(p0, f0, c.c0); p1 = fma(p1, f1, c.c0);
    k0 = ldexp(p0 * p0, (int)n0);
    k1 = ldexp(p1 * p1, (int)n1);
}

}  // namespace
