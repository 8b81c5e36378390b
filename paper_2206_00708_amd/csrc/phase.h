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

// 1 / sqrt(x) of a positive finite x: the hardware estimate y and one
// third-order step, 1 + e/2 + 3 e^2 / 8 with e = 1 - x y^2; of |e| < 2^-19 (y
// within 2^-20) it leaves 5 e^3 / 16 < 2^-58; without the library function's
// handling of 0 and infinity.
__device__ inline double rsqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// fma(a, b, c) with c in scalar registers (a constant): the compiler's own
// choice copies c into vector registers first (v_fmac needs its addend
// there), one instruction more per polynomial step.
template <class R> __host__ __device__ inline R fma_const(R a, R b, double c)
{
#ifdef __HIP_DEVICE_COMPILE__
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
#else
    return std::fma(a, b, R(c));
#endif
}

// sin and cos of a small angle t, |t| <= 1 or, SHORT, |t| <= kShortPhase: t + t z
// ps(z) and 1 - z/2 + z^2 pc(z), z = t^2.  ps and pc are minimax polynomials
// (Remez) of the error they leave in sin(t)/t and cos t, made one coefficient at a
// time from the lowest: each is rounded to a double before the rest is fitted
// again.  (A fitted linear term of cos t rounds to a double that is further off than
// all the rest.)  The errors of these coefficients, in exact arithmetic: sin(t)/t
// below 2e-19 and cos t 3e-18, SHORT 2e-18 and 1e-20.  R: double, or a wider type on
// the host.
constexpr double kShortPhase = 0.4;
template <bool SHORT, class R> __host__ __device__ inline void small_sincos(R t, R &s, R &c)
{
    using std::fma;
    const R z = t * t;
    R ps, pc;
    if constexpr (SHORT) {
        ps = fma_const(R(-2.4976067312917476e-08), z, 2.755718514904267e-06);
        ps = fma_const(ps, z, -0.0001984126973393321);
        ps = fma_const(ps, z, 0.008333333333295828);
        ps = fma_const(ps, z, -0.16666666666666624);
        pc = fma_const(R(2.0816733191749955e-09), z, -2.7557199177696807e-07);
        pc = fma_const(pc, z, 2.4801587188281747e-05);
        pc = fma_const(pc, z, -0.0013888888888839263);
        pc = fma_const(pc, z, 0.04166666666666659);
    } else {
        ps = fma_const(R(-7.533046014929189e-13), z, 1.6057158896981951e-10);
        ps = fma_const(ps, z, -2.5052092231784496e-08);
        ps = fma_const(ps, z, 2.7557319147879288e-06);
        ps = fma_const(ps, z, -0.00019841269841078057);
        ps = fma_const(ps, z, 0.008333333333333104);
        ps = fma_const(ps, z, -0.16666666666666666);
        pc = fma_const(R(-1.1291217635465988e-11), z, 2.0874052633329625e-09);
        pc = fma_const(pc, z, -2.755729858163397e-07);
        pc = fma_const(pc, z, 2.480158721850318e-05);
        pc = fma_const(pc, z, -0.0013888888888724743);
        pc = fma_const(pc, z, 0.04166666666666546);
    }
    pc = fma(pc, z, R(-0.5));
    s = fma(t * z, ps, t);
    c = fma(z, pc, R(1));
}

// exp(u) of a small u, |u| in the same ranges, by its odd and even parts u + u z
// po(z) and 1 + z/2 + z^2 pe(z), z = u^2, made alike: errors below 5e-18, SHORT 1e-18.
template <bool SHORT, class R> __host__ __device__ inline R small_exp(R u)
{
    using std::fma;
    const R z = u * u;
    R po, pe;
    if constexpr (SHORT) {
        po = fma_const(R(2.513215181439118e-08), z, 2.7557168716934236e-06);
        po = fma_const(po, z, 0.00019841269972635465);
        po = fma_const(po, z, 0.008333333333281427);
        po = fma_const(po, z, 0.16666666666666738);
        pe = fma_const(R(2.0936373936805533e-09), z, 2.755720112542241e-07);
        pe = fma_const(pe, z, 2.4801587411782334e-05);
        pe = fma_const(pe, z, 0.0013888888888841302);
        pe = fma_const(pe, z, 0.04166666666666674);
    } else {
        po = fma_const(R(7.766168042632597e-13), z, 1.6056980220536488e-10);
        po = fma_const(po, z, 2.5052127169502674e-08);
        po = fma_const(po, z, 2.755731912852184e-06);
        po = fma_const(po, z, 0.0001984126984153636);
        po = fma_const(po, z, 0.008333333333332965);
        po = fma_const(po, z, 0.16666666666666669);
        pe = fma_const(R(1.1653018610758553e-11), z, 2.0873996840137114e-09);
        pe = fma_const(pe, z, 2.7557340351663354e-07);
        pe = fma_const(pe, z, 2.4801587216386585e-05);
        pe = fma_const(pe, z, 0.001388888888905748);
        pe = fma_const(pe, z, 0.04166666666666542);
    }
    pe = fma(pe, z, R(0.5));
    return R(1) + fma(z, pe, fma(u * z, po, u));
}

// sin and cos of a small angle t, |t| <= 1, FP32, made alike: errors of sin(t)/t below
// 4e-10 and of cos t 2e-9, far below FP32 rounding.  R: float, or a wider type on the host.
template <class R> __host__ __device__ inline void small_sincos_f32(R t, R &s, R &c)
{
    using std::fma;
    const R z = t * t;
    R ps = fma(R(2.7279914e-06f), z, R(-0.00019842645f));
    ps = fma(ps, z, R(0.008333355f));
    ps = fma(ps, z, R(-0.16666667f));
    s = fma(t * z, ps, t);
    R pc = fma(R(2.4213992e-05f), z, R(-0.0013884894f));
    pc = fma(pc, z, R(0.041666582f));
    pc = fma(pc, z, R(-0.5f));
    c = fma(z, pc, R(1));
}

}  // namespace bemtx
