// Exponentials shared by kernels that must give the same bits: that of the kernel row by the sample evaluation (gp_step.hip) and the rollout
// with one workgroup per trajectory (rollout.hip), that of the cost by all end-of-step kernels.
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

// exp(x) for the saturating cost: x = n log 2 + r with log 2 in two parts, and the Taylor polynomial of degree 13 in r, with what
// r and 1 + r are rounded by added at the end.  A negative cost weight makes x positive, without a bound where a trajectory diverges: x is held
// to the range past whose ends the result is 0 or infinite, as nothing is left of r for a large n (not a number stays so).
// Largest and root mean square relative error, x from -708 to 709 (ten ranges of 0.2 million): 1.11e-16 and 4.7e-17, the library's 1.37e-16 and
// 4.9e-17.  The compiler keeps the constants of the library's function, 19 vector registers, from step to step of
// rollout.hip, where the rows need them; here they are scalars, and made anew where each is used (with all of them made ahead of the chain others
// had to make room: a saturating launch of rollout.hip took 823 instead of 795 us at B = 100, N = 2200, H = 300 and 293 instead of 283 at B = 256,
// N = 512, H = 100).  The end-of-step kernels take as long with the library's function (saturating, 60-60, B = 777: 4.83 us, 100-37 6.1, 256-256,
// B = 4096 14.9; policy.hip at 100-37 11.2): they have this one for the same bits.
__host__ __device__ __forceinline__ double cost_exp(double x)
{
#ifdef __HIP_DEVICE_COMPILE__
#define BAGEL_ANEW(value, after) asm volatile("" : "+s"(value) : "v"(after))
#else
#define BAGEL_ANEW(value, after)
#endif
    double c[14] = {0.0, 0.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800,
                    1.0 / 479001600, 1.0 / 6227020800.0};
    double log2e = 1.4426950408889634, hi = -0x1.62e42fefa0000p-1, lo = -0x1.cf79abc9e3b3ap-40;
    x = x < -746.0 ? -746.0 : x > 710.0 ? 710.0 : x;
    BAGEL_ANEW(log2e, x);
    BAGEL_ANEW(hi, x);
    BAGEL_ANEW(lo, x);
    const double n = rint(x * log2e);
    const double r0 = fma(n, hi, x), r = fma(n, lo, r0), dr = fma(n, lo, r0 - r);
    BAGEL_ANEW(c[13], r);
    double p = c[13];
#pragma unroll
    for (int k = 12; k >= 2; --k) {
        BAGEL_ANEW(c[k], p);
        p = fma(p, r, c[k]);
    }
#undef BAGEL_ANEW
    const double t = 1.0 + r;
    p = t + fma(r * r, p, ((1.0 - t) + r) + dr);
    return ldexp(p, (int)n);
}

}  // namespace
