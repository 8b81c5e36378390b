// sin and cos of the phase k r of the Helmholtz Green's function, FP64, and
// (device) 1 / r.
//
// Method: Cody-Waite reduction x = n (pi/2) + r with pi/2 split into three
// parts (33 + 33 + 53 significant bits, so that n * P1 and n * P2 are exact
// for |n| < 2^20) applied with fused multiply-adds, then Taylor polynomials
// of sin (through r^17) and cos (through r^16) on |r| <= pi/4, where the
// truncation error is below 1e-19, and quadrant selection from n mod 4.
// Valid for |x| < 1e5 (exact reduction); problems whose phases could exceed
// that are rejected when they are created.
// The split constants and the coefficients 1/n! were generated for this
// file from the decimal expansion of pi with exact rational arithmetic.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace bemtx {

constexpr double kPhaseMax = 1.0e5;   // largest |k r| the reduction is exact for

__host__ __device__ inline void phase_sincos(double x, double *s, double *c)
{
    constexpr double kTwoOverPi = 0.6366197723675814;
    constexpr double P1 = 1.5707963267341256;      // pi/2, leading 33 bits
    constexpr double P2 = 6.077100506303966e-11;   // next 33 bits
    constexpr double P3 = 2.0222662487959506e-21;  // remainder
    const double n = rint(x * kTwoOverPi);
    double r = fma(-n, P1, x);
    r = fma(-n, P2, r);
    r = fma(-n, P3, r);
    const double z = r * r;
    double ps = 2.8114572543455206e-15;            //  1/17!
    ps = fma(ps, z, -7.647163731819816e-13);       // -1/15!
    ps = fma(ps, z, 1.6059043836821613e-10);       //  1/13!
    ps = fma(ps, z, -2.505210838544172e-08);       // -1/11!
    ps = fma(ps, z, 2.7557319223985893e-06);       //  1/9!
    ps = fma(ps, z, -0.0001984126984126984);       // -1/7!
    ps = fma(ps, z, 0.008333333333333333);         //  1/5!
    ps = fma(ps, z, -0.16666666666666666);         // -1/3!
    const double sr = fma(r * z, ps, r);
    double pc = 4.779477332387385e-14;             //  1/16!
    pc = fma(pc, z, -1.1470745597729725e-11);      // -1/14!
    pc = fma(pc, z, 2.08767569878681e-09);         //  1/12!
    pc = fma(pc, z, -2.755731922398589e-07);       // -1/10!
    pc = fma(pc, z, 2.48015873015873e-05);         //  1/8!
    pc = fma(pc, z, -0.001388888888888889);        // -1/6!
    pc = fma(pc, z, 0.041666666666666664);         //  1/4!
    pc = fma(pc, z, -0.5);                         // -1/2!
    const double cr = fma(z, pc, 1.0);
    const int q = (int)n & 3;
    double sv = (q & 1) ? cr : sr;
    double cv = (q & 1) ? sr : cr;
    if (q & 2) sv = -sv;
    if ((q + 1) & 2) cv = -cv;
    *s = sv;
    *c = cv;
}

// 1 / sqrt(x) of a positive finite x: the hardware estimate (relative error e
// below 2^-20) with one third-order step, 1 + e/2 + 3 e^2 / 8 (error below
// 2^-60); without the library function's handling of 0 and infinity.
__device__ inline double rsqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// fma(a, b, c) with c in scalar registers (a constant): the compiler's own
// choice copies c into vector registers first (v_fmac needs its addend
// there), one instruction more per polynomial step.
__device__ inline double fma_const(double a, double b, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// sin and cos of a small angle t: the Taylor series of sin(t)/t and cos t as
// polynomials in z = t^2, economised by Chebyshev polynomials (Lanczos) on
// the range of z.  HALF: |t| <= 1/2, degrees 5 and 6, errors below 2e-17 and
// 1e-19; else |t| <= 1, degree 7, errors below 1e-19 and 2e-18.
template <bool HALF> __device__ inline void small_sincos(double t, double &s, double &c)
{
    const double z = t * t;
    double ps, pc;
    if constexpr (HALF) {
        ps = fma_const(-2.493193700544346e-08, z, 2.7556981496282986e-06);
        ps = fma_const(ps, z, -0.00019841269403639427);
        ps = fma_const(ps, z, 0.008333333333076967);
        ps = fma_const(ps, z, -0.16666666666666116);
        pc = fma_const(2.077661169102768e-09, z, -2.7556975230704026e-07);
        pc = fma_const(pc, z, 2.4801586715453357e-05);
        pc = fma_const(pc, z, -0.0013888888888376136);
        pc = fma_const(pc, z, 0.04166666666666453);
    } else {
        ps = fma_const(-7.535488064487613e-13, z, 1.6057233337039862e-10);
        ps = fma_const(ps, z, -2.5052093083699724e-08);
        ps = fma_const(ps, z, 2.7557319152309194e-06);
        ps = fma_const(ps, z, -0.00019841269841087476);
        ps = fma_const(ps, z, 0.008333333333333106);
        ps = fma_const(ps, z, -0.16666666666666666);
        pc = fma_const(-1.1281052794952459e-11, z, 2.0873682510844006e-09);
        pc = fma_const(pc, z, -2.755729324310771e-07);
        pc = fma_const(pc, z, 2.4801587179897263e-05);
        pc = fma_const(pc, z, -0.0013888888888579293);
        pc = fma_const(pc, z, 0.0416666666666628);
    }
    s = fma(t * z, ps, t);
    pc = fma(pc, z, -0.5);
    c = fma(z, pc, 1.0);
}

// exp(u) of a small u by its even and odd parts, economised as above: |u| <= 1/2
// (HALF, degrees 6 and 5 in u^2, errors below 1e-19 and 2e-17) or |u| <= 1
// (degree 7, errors below 2e-18 and 1e-19).
template <bool HALF> __device__ inline double small_exp(double u)
{
    const double z = u * u;
    double po, pe;
    if constexpr (HALF) {
        po = fma_const(2.517282343175421e-08, z, 2.755697945753373e-06);
        po = fma_const(po, z, 0.00019841270281873433);
        po = fma_const(po, z, 0.00833333333307511);
        po = fma_const(po, z, 0.1666666666666722);
        pe = fma_const(2.097735036131617e-09, z, 2.755697317701901e-07);
        pe = fma_const(pe, z, 2.480158789165942e-05);
        pe = fma_const(pe, z, 0.001388888888837246);
        pe = fma_const(pe, z, 0.041666666666668815);
        pe = fma_const(pe, z, 0.49999999999999994);
    } else {
        po = fma_const(7.760411617749028e-13, z, 1.60571992722078e-10);
        po = fma_const(po, z, 2.505212401145532e-08);
        po = fma_const(po, z, 2.7557319150687833e-06);
        po = fma_const(po, z, 0.00019841269841456506);
        po = fma_const(po, z, 0.0083333333333331);
        po = fma_const(po, z, 0.16666666666666669);
        pe = fma_const(1.1663425624683784e-11, z, 2.087361778743318e-09);
        pe = fma_const(pe, z, 2.7557345820982554e-07);
        pe = fma_const(pe, z, 2.4801587176816665e-05);
        pe = fma_const(pe, z, 0.0013888888889206652);
        pe = fma_const(pe, z, 0.041666666666662695);
        pe = fma_const(pe, z, 0.5000000000000002);
    }
    return 1.0 + fma(z, pe, fma(u * z, po, u));
}

}  // namespace bemtx
