// rpdla_fastmath.hpp -- double-precision sine/cosine, exponential, logarithm
// and reciprocal for the push and ionization kernels, branch-free so that every
// lane of a wave takes the same instruction stream.
//
//   sincos: Cody-Waite reduction x = n pi/2 + r with pi/2 split in three
//           doubles (products kept exact by fma), |r| <= pi/4, then
//           sin r = r + r^3 S(r^2), cos r = 1 - r^2/2 + r^4 C(r^2) and the
//           quadrant n mod 4 applied by a swap and sign-bit flips (n rounded
//           by the 1.5 2^52 addition, its low word the integer).  Accurate to
//           a few ulp for |x| < 2^30 (the arguments here are phases of at
//           most ~1e4 rad).
//   cis:    e^{ix} in half-angle form: x = n pi + r (pi in three parts),
//           |r| <= pi/2, sigma = sqrt2 sin(r/2) = r P(r^2), kappa = sqrt2
//           cos(r/2) = sqrt2 - (sqrt2/8) r^2 + r^4 Q(r^2); then cos x =
//           (-1)^n (1 - sigma^2) and sin x = (-1)^n sigma kappa.  The caller
//           applies (-1)^n to a common factor, so no quadrant swap is needed.
//   exp:    x = n ln2 + r (ln 2 in two parts), exp r = 1 + r + r^2 E(r),
//           scaled by 2^n with ldexp; 0 below -745, exact at 0.
//   log:    x = 2^e m, m in [sqrt(1/2), sqrt(2)), ln m = 2 atanh((m-1)/(m+1))
//           by its series, ln x = e ln2 + ln m (positive finite x only).
//   rcp:    hardware reciprocal estimate refined by one third-order step
//           (error cubed: 2^-26 estimates reach full precision).
//   rsqrt:  hardware reciprocal-square-root estimate refined by one
//           third-order step, for arguments in [1, 2^1000] (here 1 + u.u),
//           and in [2^-960, 2^960] (the rate's |a|^2, smaller ones give a
//           zero rate before it is needed).
// S, C, P, Q, E are Remez fits generated by gen_fastmath.py.
#pragma once

#include <math.h>

#include "rpdla_fastmath_coeffs.hpp"

#if defined(__HIPCC__)
#define RPDLA_HD __host__ __device__
#else
#define RPDLA_HD
#endif

namespace rpdla {
namespace fm {

// Nearest integer of a double below 2^51 in magnitude by the round-to-nearest
// addition of 1.5 2^52: the sum's low 32 bits are that integer (two's
// complement), the sum minus 1.5 2^52 is it as a double.
constexpr double kRoundMagic = 6755399441055744.0;  // 1.5 * 2^52

RPDLA_HD inline int low_word(double v)
{
    unsigned long long b;
    __builtin_memcpy(&b, &v, sizeof b);
    return (int)(unsigned)b;
}

// v with its sign bit flipped where the bit 31 of m is set (m is 0 or 2^31).
RPDLA_HD inline double flip_sign(double v, unsigned m)
{
    unsigned long long b;
    __builtin_memcpy(&b, &v, sizeof b);
    b ^= (unsigned long long)m << 32;
    double r;
    __builtin_memcpy(&r, &b, sizeof r);
    return r;
}

// The constants of one radial-field evaluation and of the reciprocal steps, as
// a record: a kernel with a long loop copies it into registers once (see
// keep_in_sgpr / keep_in_vgpr in rpdla_device.hpp).  A double is no literal
// operand on this machine, so each constant that is not in a register costs
// two scalar moves at every use.  kCoef, the default everywhere, folds to the
// constants themselves.  The reduction constants are held negated: fma(n, -c, x)
// is fma(-n, c, x), and the accumulator form of the instruction is shorter.
struct Coef {
    double magic = kRoundMagic;
    double log2e = kLog2e, nln2_1 = -kLn2_1, nln2_2 = -kLn2_2;
    double ex[10] = {kExp[0], kExp[1], kExp[2], kExp[3], kExp[4],
                     kExp[5], kExp[6], kExp[7], kExp[8], kExp[9]};
    double inv_pi = kOneOverPi, npi_1 = -kPi_1, npi_2 = -kPi_2, npi_3 = -kPi_3;
    double sg[7] = {kSigma[0], kSigma[1], kSigma[2], kSigma[3], kSigma[4], kSigma[5], kSigma[6]};
    double kp[6] = {kKappa[0], kKappa[1], kKappa[2], kKappa[3], kKappa[4], kKappa[5]};
    double ns2o8 = -kSqrt2Over8, s2 = kSqrt2;
    // brackets of the radial field, and the third-order rsqrt step (c375)
    double c375 = 0.375, c1_0625 = 1.0625, c1875 = 0.1875, c5 = 5.0;
};
constexpr Coef kCoef{};

// The logarithm's constants beside those (the tunnelling rate takes both).
struct LogCoef {
    double rsqrt2 = 0.70710678118654752;
    // atanh series, 2/19 down to 2/3
    double at[9] = {2.0 / 19.0, 2.0 / 17.0, 2.0 / 15.0, 2.0 / 13.0, 2.0 / 11.0,
                    2.0 / 9.0,  2.0 / 7.0,  2.0 / 5.0,  2.0 / 3.0};
};
constexpr LogCoef kLogCoef{};

// sin r, cos r for |r| <= pi/4 (a little beyond), rotated to quadrant q.
RPDLA_HD inline void sincos_reduced(double r, int q, double* s_out, double* c_out)
{
    const double t = r * r;
    double ps = kSin[5];
    ps = fma(ps, t, kSin[4]);
    ps = fma(ps, t, kSin[3]);
    ps = fma(ps, t, kSin[2]);
    ps = fma(ps, t, kSin[1]);
    ps = fma(ps, t, kSin[0]);
    const double s = fma(r * t, ps, r);
    double pc = kCos[5];
    pc = fma(pc, t, kCos[4]);
    pc = fma(pc, t, kCos[3]);
    pc = fma(pc, t, kCos[2]);
    pc = fma(pc, t, kCos[1]);
    pc = fma(pc, t, kCos[0]);
    // cos = (1 - t/2) + t^2 C: 1 - t/2 lies in [0.69, 1], so its rounding is at
    // most 2^-54 (absolute, which is what the field amplitudes need)
    const double c = fma(t * t, pc, 1.0 - 0.5 * t);
    const bool swap = (q & 1) != 0;
    const double sv = swap ? c : s;
    const double cv = swap ? s : c;
    // quadrant signs: sin negative for q = 2, 3, cos for q = 1, 2 (mod 4)
    *s_out = flip_sign(sv, ((unsigned)q << 30) & 0x80000000u);
    *c_out = flip_sign(cv, ((unsigned)q << 30) + 0x40000000u & 0x80000000u);
}

RPDLA_HD inline void sincos_f64(double x, double* s_out, double* c_out)
{
    const double tq = fma(x, kTwoOverPi, kRoundMagic);
    const double n = tq - kRoundMagic;
    double r = fma(-n, kPio2_1, x);
    r = fma(-n, kPio2_2, r);
    r = fma(-n, kPio2_3, r);
    sincos_reduced(r, low_word(tq), s_out, c_out);
}

// sin and cos of the unevaluated sum x_hi + x_lo (|x_lo| a few units at
// most): x_lo joins after the leading reduction step, when the remainder is
// already small, so the argument is not rounded to a multiple of ulp(x_hi).
RPDLA_HD inline void sincos2_f64(double x_hi, double x_lo, double* s_out, double* c_out)
{
    const double tq = fma(x_hi + x_lo, kTwoOverPi, kRoundMagic);
    const double n = tq - kRoundMagic;
    double r = fma(-n, kPio2_1, x_hi) + x_lo;
    r = fma(-n, kPio2_2, r);
    r = fma(-n, kPio2_3, r);
    sincos_reduced(r, low_word(tq), s_out, c_out);
}

// e^{i (x_hi + x_lo)} in half-angle form (|x_lo| a few units at most, joined
// after the leading reduction step as in sincos2_f64): writes sigma and kappa
// with cos x = (-1)^n (1 - sigma^2), sin x = (-1)^n sigma kappa, and returns
// (-1)^n as a sign mask (0 or 2^31) for flip_sign.
RPDLA_HD inline unsigned cis_half2_f64(double x_hi, double x_lo, double* sigma, double* kappa,
                                       const Coef& k = kCoef)
{
    const double tq = fma(x_hi + x_lo, k.inv_pi, k.magic);
    const double n = tq - k.magic;
    double r = fma(n, k.npi_1, x_hi) + x_lo;
    r = fma(n, k.npi_2, r);
    r = fma(n, k.npi_3, r);
    const double t = r * r;
    double p = k.sg[6];
    p = fma(p, t, k.sg[5]);
    p = fma(p, t, k.sg[4]);
    p = fma(p, t, k.sg[3]);
    p = fma(p, t, k.sg[2]);
    p = fma(p, t, k.sg[1]);
    p = fma(p, t, k.sg[0]);
    *sigma = r * p;
    double q = k.kp[5];
    q = fma(q, t, k.kp[4]);
    q = fma(q, t, k.kp[3]);
    q = fma(q, t, k.kp[2]);
    q = fma(q, t, k.kp[1]);
    q = fma(q, t, k.kp[0]);
    q = fma(q, t, k.ns2o8);
    *kappa = fma(q, t, k.s2);
    return (unsigned)low_word(tq) << 31;
}

RPDLA_HD inline double exp_f64(double x)
{
    const double n = rint(x * kLog2e);
    double r = fma(-n, kLn2_1, x);
    r = fma(-n, kLn2_2, r);
    double p = kExp[9];
    p = fma(p, r, kExp[8]);
    p = fma(p, r, kExp[7]);
    p = fma(p, r, kExp[6]);
    p = fma(p, r, kExp[5]);
    p = fma(p, r, kExp[4]);
    p = fma(p, r, kExp[3]);
    p = fma(p, r, kExp[2]);
    p = fma(p, r, kExp[1]);
    p = fma(p, r, kExp[0]);
    const double e = fma(r * r, p, r) + 1.0;
    const double ni = n < -1100.0 ? -1100.0 : n;   // keeps ldexp's exponent in range
    const double v = ldexp(e, (int)ni);
    return x < -745.2 ? 0.0 : v;
}

// The same exponential without the range guards, for finite arguments of
// magnitude below 2^31 ln 2 (n rounded by the 1.5 2^52 addition): below about
// -745 the scaling by 2^n flushes to zero by itself.
RPDLA_HD inline double exp_fin_f64(double x, const Coef& k = kCoef)
{
    const double tn = fma(x, k.log2e, k.magic);
    const double n = tn - k.magic;
    double r = fma(n, k.nln2_1, x);
    r = fma(n, k.nln2_2, r);
    double p = k.ex[9];
    p = fma(p, r, k.ex[8]);
    p = fma(p, r, k.ex[7]);
    p = fma(p, r, k.ex[6]);
    p = fma(p, r, k.ex[5]);
    p = fma(p, r, k.ex[4]);
    p = fma(p, r, k.ex[3]);
    p = fma(p, r, k.ex[2]);
    p = fma(p, r, k.ex[1]);
    p = fma(p, r, k.ex[0]);
    const double e = fma(r * r, p, r) + 1.0;
    return ldexp(e, low_word(tn));
}

RPDLA_HD inline double rcp_f64(double d);

// Natural logarithm of a positive finite x (normal or subnormal).  x = 2^e m
// with m in [sqrt(1/2), sqrt(2)); ln m = 2 atanh(f), f = (m - 1)/(m + 1),
// |f| <= 0.1716, by the atanh series 2f (1 + f^2/3 + f^4/5 + ... + f^18/19)
// (the first term left out, f^20/21, is below 2^-55 of the sum).  f comes from
// the refined reciprocal with one residual correction, m + 1 carried exactly
// as b + bl.  ln x = e ln2 + ln m, ln2 in two parts.  A few ulp.
RPDLA_HD inline double log_pos_f64(double x, const Coef& k = kCoef, const LogCoef& l = kLogCoef)
{
    int e;
    double m = frexp(x, &e);                      // m in [0.5, 1)
    const bool lo = m < l.rsqrt2;
    m = lo ? m + m : m;
    e = lo ? e - 1 : e;
    const double a = m - 1.0;                     // exact
    const double b = m + 1.0;
    const double bl = m - (b - 1.0);              // m + 1 = b + bl exactly
    const double r = rcp_f64(b);
    double f = a * r;
    f = fma(fma(-f, b, a), r, f);                 // a / b
    f = fma(-f * bl, r, f);                       // a / (b + bl)
    // the series term by term from the smallest, each coefficient a multiplier
    // (so that it need not be held in a vector register across a loop)
    const double z = f * f;
    const double z2 = z * z, z4 = z2 * z2, z8 = z4 * z4;
    double p = l.at[0] * z8;
    p = fma(l.at[1], z4 * z2 * z, p);
    p = fma(l.at[2], z4 * z2, p);
    p = fma(l.at[3], z4 * z, p);
    p = fma(l.at[4], z4, p);
    p = fma(l.at[5], z2 * z, p);
    p = fma(l.at[6], z2, p);
    p = fma(l.at[7], z, p);
    p = p + l.at[8];
    const double lnm = fma(f * z, p, f + f);
    const double ed = (double)e;
    return fma(-ed, k.nln2_1, fma(-ed, k.nln2_2, lnm));
}

RPDLA_HD inline double rcp_f64(double d)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = __builtin_amdgcn_rcp(d);
#else
    double y = (double)(1.0f / (float)d);
#endif
    // one third-order step: 1/d = y / (1 - e) = y (1 + e + e^2 + ...), e = 1 - d y
    const double e = fma(-d, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// Reciprocal square root for x in [2^-960, 2^960] (no scaling of the argument):
// the hardware estimate refined by one third-order step, as rsqrt_ge1_f64.
RPDLA_HD inline double rsqrt_mid_f64(double x, const Coef& k = kCoef)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = __builtin_amdgcn_rsq(x);
#else
    // a float estimate where float holds x as a normal number
    double y = (x > 1e-30 && x < 1e30) ? (double)(1.0f / sqrtf((float)x)) : 1.0 / sqrt(x);
#endif
    const double e = fma(-x, y * y, 1.0);
    return fma(y, e * fma(k.c375, e, 0.5), y);
}

RPDLA_HD inline double rsqrt_ge1_f64(double x, const Coef& k = kCoef)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = __builtin_amdgcn_rsq(x);
#else
    double y = (double)(1.0f / sqrtf((float)x));
#endif
    // one third-order step: x^-1/2 = y (1 - e)^-1/2 = y (1 + e/2 + 3e^2/8 + ...),
    // e = 1 - x y^2
    const double e = fma(-x, y * y, 1.0);
    return fma(y, e * fma(k.c375, e, 0.5), y);
}

}  // namespace fm
}  // namespace rpdla
