// Device-side building blocks shared by the forward and adjoint evaluators.
//
// Tables are read through the constant address space so that wave-uniform
// reads become scalar loads, and the +-1 coefficient masks are tested with
// scalar bit tests: only the non-zero coefficients cost vector instructions.
#pragma once

#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>

#include <cstdint>
#else
// compiled at run time (hipRTC): no standard headers
typedef __hip_internal::uint64_t uint64_t;
typedef __hip_internal::int64_t int64_t;
typedef __hip_internal::uint32_t uint32_t;
typedef __hip_internal::int32_t int32_t;
typedef __hip_internal::uint8_t uint8_t;
typedef __hip_internal::int8_t int8_t;
#endif

// A value made opaque to the optimizer (an empty asm that may change it; no
// instruction): generated code copies a group's operands through it so that
// equal products of different groups are not merged into long-lived values.
#ifndef AMI_OPAQUE
#define AMI_OPAQUE(x) asm volatile("" : "+v"(x))
#endif

// The same for a wave-uniform value.
#ifndef AMI_OPAQUE_S
#ifdef __HIP_DEVICE_COMPILE__
#define AMI_OPAQUE_S(x) asm volatile("" : "+s"(x))
#else
#define AMI_OPAQUE_S(x)
#endif
#endif

// A scheduling fence: the compiler moves no instruction across it.  Generated
// code puts one between chunks of independent work, so that the loads and
// values of a later chunk do not stay live through an earlier one.
#ifndef AMI_SCHED_FENCE
#define AMI_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#endif

namespace ami {

typedef const __attribute__((address_space(4))) uint64_t *cu64;
typedef const __attribute__((address_space(4))) uint32_t *cu32;
typedef const __attribute__((address_space(4))) double *cdbl;
typedef const __attribute__((address_space(4))) int32_t *ci32;

// LDS columns, by pointers in their own address space (a pointer that went
// through AMI_OPAQUE stays an LDS pointer).
typedef __attribute__((address_space(3))) double *lds;
typedef const __attribute__((address_space(3))) double *clds;

constexpr int kMaxExtDev = 4;

// Packed evaluation tables (built by the host, see construct.cpp):
//   leaf[l]  bits 0-15 energies with coefficient +1, bits 16-31 with -1,
//            bit 32 set for a Bose-type leaf (sigma = -1)
//   den[r]   bits 0-15 / 16-31 energy masks as above, bits 32-63 the external
//            frequency coefficients as four int8
//   line[j]  bits 0-15 / 16-31 frequency/momentum slots with coefficient +1/-1
//   term[t]  leaf indices of term t, one byte each; term_sign[t] its prefactor
//   group[g] denominator indices of group g, one byte each;
//            terms of group g are group_start[g] .. group_start[g+1]-1
struct PackedTabs {
    const uint64_t *leaf;
    const uint64_t *den;
    const uint32_t *line;
    const uint64_t *term;
    const double *term_sign;
    const int32_t *group_start;
    const uint64_t *group;
    int L, D, G, T;
    int n_eps, n_int, n_ext, n_freq, n_g, dpt;
    uint32_t fermi_used;    // energies that appear in Fermi-type leaves
    int use_products;       // Fermi leaves from products of exp(beta E_i)
};

// ---- elementary functions -------------------------------------------------

// What bounds these functions is the number of FP64 instructions: every one
// holds a SIMD for four cycles per wave (v_rcp_f64 for sixteen), 32-bit
// integer operations for two to four, and a pair of v_cndmask_b32 on vcc for
// about ten.  So the reductions round by adding kRintMagic (the integer is then
// the sum's low word: no rndne, no conversion), the polynomials are minimax
// ones (Remez, on the stated intervals, each coefficient rounded before the
// next were fitted; their truncation errors stand beside them), and selections
// and signs are bit operations.

// Added to a double x with |x| < 2^31, it leaves the sum's low word equal to
// the integer nearest to x (two's complement): that integer as a double is the
// sum minus kRintMagic.
constexpr double kRintMagic = 0x1.8p52;

__device__ __forceinline__ uint64_t dbits(double x) { return __builtin_bit_cast(uint64_t, x); }
__device__ __forceinline__ double bitsd(uint64_t u) { return __builtin_bit_cast(double, u); }

// x with its sign flipped where bit `bit` of n is set.
__device__ __forceinline__ double flip_sign(double x, uint32_t n, int bit) {
    return bitsd(dbits(x) ^ (static_cast<uint64_t>((n << (31 - bit)) & 0x80000000u) << 32));
}

// mask ? x : y for an all-ones or all-zeros mask, on the bits.
__device__ __forceinline__ double mask_select(uint32_t mask, double x, double y) {
    const uint32_t xl = static_cast<uint32_t>(dbits(x)), xh = static_cast<uint32_t>(dbits(x) >> 32);
    const uint32_t yl = static_cast<uint32_t>(dbits(y)), yh = static_cast<uint32_t>(dbits(y) >> 32);
    const uint32_t lo = (xl & mask) | (yl & ~mask), hi = (xh & mask) | (yh & ~mask);
    return bitsd((static_cast<uint64_t>(hi) << 32) | lo);
}

// Reciprocal: the hardware estimate r (relative error at most 2^-24.3,
// measured over [1, 2] and at 1e-300 and 1e10), refined by one step of third
// order: with e = 1 - d r, 1/d = r (1 + e + e^2 + ...), and e^3 < 2^-72.
// Finite, non-zero, normal-range arguments.
__device__ __forceinline__ double rcp_nr(double d) {
    const double r = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// sin, cos and cos - 1: x = n pi/2 + r with pi/2 split in two (53 + 53 bits;
// x - n hi is a multiple of 2^-52 below 1 and so exact in the fma), |r| <=
// pi/4, sin r = r + r z S(z), cos r = 1 + z C(z) with z = r^2 and minimax S
// (degree 5, truncation error of sin r 2^-59.1) and C (degree 6, of cos r 2^-64).
// cos - 1 keeps its relative precision next to the multiples of 2 pi.  What the
// two parts leave of pi/2 is below 2^-108, so r is off by n 2^-108, 2^-86 at the
// largest argument in use, |x| < 6e6 (n itself is right up to 2^31).
__device__ __forceinline__ void sincos_cosm1(double x, double &s, double &c, double &cm1) {
    constexpr double kTwoOverPi = 0x1.45f306dc9c883p-1;
    constexpr double kPio2Hi = 0x1.921fb54442d18p+0;
    constexpr double kPio2Lo = 0x1.1a62633145c07p-54;
    const double t = fma(x, kTwoOverPi, kRintMagic);
    const double kf = t - kRintMagic;
    const uint32_t n = static_cast<uint32_t>(dbits(t));
    const double r = fma(-kf, kPio2Lo, fma(-kf, kPio2Hi, x));
    const double z = r * r;
    double ps = 0x1.5d61cfd1331c9p-33;
    ps = fma(ps, z, -0x1.ae5da9e9f2ad5p-26);
    ps = fma(ps, z, 0x1.71de346756b04p-19);
    ps = fma(ps, z, -0x1.a01a019aa3717p-13);
    ps = fma(ps, z, 0x1.111111110ea87p-7);
    ps = fma(ps, z, -0x1.555555555553dp-3);
    const double sr = fma(r * z, ps, r);
    double pc = -0x1.8fb130e396e84p-37;
    pc = fma(pc, z, 0x1.1ee9f1526ed3ap-29);
    pc = fma(pc, z, -0x1.27e4f812b64e3p-22);
    pc = fma(pc, z, 0x1.a01a019cbf628p-16);
    pc = fma(pc, z, -0x1.6c16c16c1521fp-10);
    pc = fma(pc, z, 0x1.555555555554cp-5);
    pc = fma(pc, z, -0.5);
    const double cr = fma(z, pc, 1.0);
    const uint32_t odd = 0u - (n & 1u);
    s = flip_sign(mask_select(odd, cr, sr), n, 1);
    c = flip_sign(mask_select(odd, sr, cr), n + 1u, 1);
    cm1 = (n & 3u) == 0u ? z * pc : c - 1.0;
}

__device__ __forceinline__ void sincos_red(double x, double &s, double &c) {
    double cm1;
    sincos_cosm1(x, s, c, cm1);
    (void)cm1;
}

// x - 2 pi n with n = rint(x / 2pi): 2 pi split in two (53 + 53 bits; x - n hi
// exact in the fma) for |x| < 6e6.  The energies depend on momenta only
// through cos/sin of integer combinations, so reducing every momentum
// component first keeps every later argument small.
__device__ __forceinline__ double reduce_2pi(double x) {
    constexpr double kOneOver2Pi = 0x1.45f306dc9c883p-3;
    constexpr double k2PiHi = 0x1.921fb54442d18p+2;
    constexpr double k2PiLo = 0x1.1a62633145c07p-52;
    const double n = __builtin_rint(x * kOneOver2Pi);
    return fma(-n, k2PiLo, fma(-n, k2PiHi, x));
}

// cos alone: x = n pi + r with pi split as above, |r| <= pi/2, cos x =
// (-1)^n (1 + z P(z)), z = r^2, minimax P of degree 7 (truncation error
// 2^-57.3).  For |x| < 6e6, as above.
__device__ __forceinline__ double cos_red(double x) {
    constexpr double kOneOverPi = 0x1.45f306dc9c883p-2;
    constexpr double kPiHi = 0x1.921fb54442d18p+1;
    constexpr double kPiLo = 0x1.1a62633145c07p-53;
    const double t = fma(x, kOneOverPi, kRintMagic);
    const double kf = t - kRintMagic;
    const double r = fma(-kf, kPiLo, fma(-kf, kPiHi, x));
    const double z = r * r;
    double p = 0x1.9fc80589c1077p-45;
    p = fma(p, z, -0x1.935738973aee4p-37);
    p = fma(p, z, 0x1.1eecfad41d5c9p-29);
    p = fma(p, z, -0x1.27e4f9f2e8cddp-22);
    p = fma(p, z, 0x1.a01a019ba6080p-16);
    p = fma(p, z, -0x1.6c16c16c101f5p-10);
    p = fma(p, z, 0x1.55555555554ddp-5);
    p = fma(p, z, -0.5);
    return flip_sign(fma(z, p, 1.0), static_cast<uint32_t>(dbits(t)), 0);
}

// The reduction of e^z: z = n ln2 + r with ln2 split in two (53 + 53 bits;
// z - n hi exact in the fma), |r| <= ln2/2, and q with e^r = 1 + r + r^2 q
// (minimax of degree 9; relative truncation error of e^r - 1 2^-55.6, of e^r
// 2^-56.9).  For |z| < 1e6.
__device__ __forceinline__ void exp_reduce(double z, int &n, double &r, double &q) {
    constexpr double kLog2e = 0x1.71547652b82fep+0;
    constexpr double kLn2Hi = 0x1.62e42fefa39efp-1;
    constexpr double kLn2Lo = 0x1.abc9e3b39803fp-56;
    const double t = fma(z, kLog2e, kRintMagic);
    const double kf = t - kRintMagic;
    n = static_cast<int>(static_cast<uint32_t>(dbits(t)));
    r = fma(-kf, kLn2Lo, fma(-kf, kLn2Hi, z));
    q = 0x1.ae993696b5742p-26;
    q = fma(q, r, 0x1.28a16c96d6ce5p-22);
    q = fma(q, r, 0x1.71de6633fa366p-19);
    q = fma(q, r, 0x1.a019a7d5890f2p-16);
    q = fma(q, r, 0x1.a01a01874628ep-13);
    q = fma(q, r, 0x1.6c16c17ec6b36p-10);
    q = fma(q, r, 0x1.1111111114d16p-7);
    q = fma(q, r, 0x1.5555555552271p-5);
    q = fma(q, r, 0x1.555555555554fp-3);
    q = fma(q, r, 0x1.0000000000005p-1);
}

// e^z for |z| < 708: 2^n (1 + r (1 + r q)).
__device__ __forceinline__ double exp_scaled(double z) {
    int n;
    double r, q;
    exp_reduce(z, n, r, q);
    return __builtin_ldexp(fma(fma(q, r, 1.0), r, 1.0), n);
}

// e^z and e^z - 1 from one reduction, with p = e^r - 1 = r + r^2 q:
// t = 2^n (1 + p) and m = 2^n p + (2^n - 1); the last form has no cancellation
// for any n (2^n - 1 is exact for |n| < 54), so m keeps full relative precision
// near z = 0 and t near its underflow.  For |z| < 708.
__device__ __forceinline__ void exp_split(double z, double &t, double &m) {
    int n;
    double r, q;
    exp_reduce(z, n, r, q);
    const double p = fma(r * r, q, r);
    const double s = __builtin_ldexp(1.0, n);
    t = fma(s, p, s);
    m = fma(s, p, s - 1.0);
}

// A leaf f_sigma(y) = 1/(sigma e^y + 1) and its mirror f_sigma(-y) = 1 - f_sigma(y),
// both with full relative precision everywhere: with e = e^y and m = e^y - 1
// (exp_split),
//   Fermi  (sigma = +1): 1/(1 + e) and e/(1 + e)
//   Bose-type (-1):      -1/m and e/m
// (no selection by the sign of y: where e is small the first is 1 - e, where it
// is large the second is 1 - 1/e, and each quotient is formed directly; the
// second corrected by its residual, so that it and the slope, their product,
// carry the reciprocal's rounding once).
// Arguments are clamped at +-700 (the small leaves there are below 1e-304), so
// nothing overflows.  Root mean square errors in units of 2^-53, over |y| < 30 and
// log-uniform 1e-8 < |y| < 600, beside those of the form by e^-|y| that this one
// replaced: Fermi f 0.62 and 0.70 (0.76, 0.70), f(-y) 0.63 and 0.70 (0.76, 0.70),
// slope 1.17 and 1.24 (1.49, 1.37); Bose-type f 0.66 and 0.60 (0.82, 0.63), f(-y)
// 0.64 and 0.71 (0.82, 0.63; never a result by itself), slope 1.08 and 1.16 (1.61,
// 1.29).  Without the correction the slopes were at 1.31 and 1.41, 1.43 and 1.34.
// A leaf alone takes 24 (Fermi) and 25 (Bose-type) FP64 instructions, a pair 27 and
// 29, where the form by e^-|y|, its Taylor series and two selections took 35-37
// (order 4, 52 terms, 10^6 samples: forward call 40.6 -> 34.4 us).
__device__ __forceinline__ void leaf_pair(bool bose, double y, double &f, double &fm) {
    const double z = fmin(fmax(y, -700.0), 700.0);
    if (bose) {
        double e, m;
        exp_split(z, e, m);
        const double r = rcp_nr(m), p = e * r;
        f = -r;
        fm = fma(fma(-m, p, e), r, p);
    } else {
        const double e = exp_scaled(z), d = 1.0 + e;
        const double r = rcp_nr(d), p = e * r;
        f = r;
        fm = fma(fma(-d, p, e), r, p);
    }
}

// f_sigma(y) and f_sigma'(y) = -f_sigma(y) f_sigma(-y) together.
__device__ __forceinline__ void leaf_and_slope(bool bose, double y, double &f, double &dv) {
    double fm;
    leaf_pair(bose, y, f, fm);
    dv = -(f * fm);
}

// f_sigma'(y) alone.
__device__ __forceinline__ double leaf_deriv(bool bose, double y) {
    double f, dv;
    leaf_and_slope(bose, y, f, dv);
    return dv;
}

// A leaf at a complex argument y = yr + i yi (complex energies): with
// z = -y where yr is positive and z = y elsewhere (so Re z = -|yr| <= 0; pos
// is the clear sign bit of yr, and at yr = 0 either form holds),
// w = e^z = t (cos zi + i sin zi), t = e^-|yr|, and Q = sigma + w, the leaf is
// w/Q where yr > 0 and sigma/Q elsewhere (no overflow of |Q|^2 on either side).
// For the Bose-type Q = w - 1, its real part is written m cos zi + (cos zi - 1)
// with m = t - 1 (exp_split) and cos zi - 1 from its own series
// (sincos_cosm1), so Q keeps full relative precision near y = 0.
struct ComplexLeafParts {
    uint32_t neg;              // all ones where yr is negative
    double wr, wi, qr, qi, r;  // w, Q, 1/|Q|^2
};

__device__ __forceinline__ ComplexLeafParts complex_leaf_parts(bool bose, double yr, double yi) {
    ComplexLeafParts p;
    const uint32_t hi = static_cast<uint32_t>(dbits(yr) >> 32);
    p.neg = 0u - (hi >> 31);
    double t, m = 0.0, s, c, cm1;
    const double z = -fmin(fabs(yr), 700.0);
    if (bose) exp_split(z, t, m);
    else t = exp_scaled(z);
    sincos_cosm1(yi, s, c, cm1);
    s = flip_sign(s, ~hi, 31);             // sin zi
    p.wr = t * c;
    p.wi = t * s;
    p.qr = bose ? fma(m, c, cm1) : 1.0 + p.wr;
    p.qi = p.wi;
    p.r = rcp_nr(fma(p.qr, p.qr, p.qi * p.qi));
    return p;
}

// The leaf and f(-y): for -y the same z, w and Q arise, with the two quotients
// exchanged: f(y) = w/Q and f(-y) = sigma/Q where yr > 0, the other way round
// elsewhere.  The adjoint's slope is f'(y) = -f(y) f(-y).
__device__ __forceinline__ void leaf_complex_pair(bool bose, double yr, double yi, double &fr, double &fi,
                                                  double &mr, double &mi) {
    const ComplexLeafParts p = complex_leaf_parts(bose, yr, yi);
    const double ir = p.qr * p.r, ii = -p.qi * p.r;                                        // 1/Q
    const double ar = fma(p.wr, ir, -p.wi * ii), ai = fma(p.wr, ii, p.wi * ir);   // w/Q
    const double br = bose ? -ir : ir, bi = bose ? -ii : ii;                         // sigma/Q
    fr = mask_select(p.neg, br, ar);
    fi = mask_select(p.neg, bi, ai);
    mr = mask_select(p.neg, ar, br);
    mi = mask_select(p.neg, ai, bi);
}

// The leaf alone: the numerator (w or sigma) is selected before the quotient.
__device__ __forceinline__ void leaf_complex(bool bose, double yr, double yi, double &fr, double &fi) {
    const ComplexLeafParts p = complex_leaf_parts(bose, yr, yi);
    const double ir = p.qr * p.r, ii = -p.qi * p.r;   // 1/Q
    const double nr = mask_select(p.neg, bose ? -1.0 : 1.0, p.wr);
    const double ni = mask_select(p.neg, 0.0, p.wi);
    fr = fma(nr, ir, -ni * ii);
    fi = fma(nr, ii, ni * ir);
}

// ---- counter-based random numbers -----------------------------------------

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror and Shaw, SC'11): each round
// multiplies words 0 and 2 by the two round constants (64-bit products) and
// forms (hi1 ^ c1 ^ k0, lo1, hi0 ^ c3 ^ k1, lo0); the key grows by the Weyl
// increments after every round.
__device__ __forceinline__ void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c[0];
        const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c[2];
        const uint32_t n0 = static_cast<uint32_t>(p1 >> 32) ^ c[1] ^ k0;
        const uint32_t n2 = static_cast<uint32_t>(p0 >> 32) ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = static_cast<uint32_t>(p1);
        c[2] = n2;
        c[3] = static_cast<uint32_t>(p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// A uniform momentum component in (-pi, pi) from one 32-bit word:
// (u - 1/2) * 2 pi with u = (word + 1/2) / 2^32 (exact up to the last product).
__device__ __forceinline__ double word_to_momentum(uint32_t w) {
    const double u = (static_cast<double>(w) + 0.5) * 0x1p-32;
    return (u - 0.5) * 0x1.921fb54442d18p+2;
}

// sum_i (+-1) E_i over the bits of two 16-bit masks (scalar bit tests).
template <int NE>
__device__ __forceinline__ double combo(uint32_t pos, uint32_t neg, const double (&E)[NE]) {
    double x = 0.0;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        if (pos & (1u << i)) x += E[i];
        else if (neg & (1u << i)) x -= E[i];
    }
    return x;
}

// Scatter a value into per-energy accumulators with the mask signs.
template <int NE>
__device__ __forceinline__ void combo_adj(uint32_t pos, uint32_t neg, double v, double (&g)[NE]) {
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        if (pos & (1u << i)) g[i] += v;
        else if (neg & (1u << i)) g[i] -= v;
    }
}

// A double moved across lanes by one DPP control (all rows and banks, bound
// control on: a lane whose source lane falls outside the wave or the row
// receives 0), as two 32-bit halves.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_mov_dpp(static_cast<int>(static_cast<unsigned>(u)), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(static_cast<int>(static_cast<unsigned>(u >> 32)), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) |
                                          static_cast<unsigned>(lo));
}

// Sum over the 64 lanes of a wave (every lane active), left in lane 63:
// inclusive prefix sums within each row of 16 lanes (row_shr 1, 2, 4, 8), so
// lane 15 of row r holds the row's sum S_r; row_bcast:15 then adds lane 15 of
// the previous row (lane 63: S_3 + S_2), and row_bcast:31 adds lane 31 (by then
// S_1 + S_0) into rows 2-3.  Register moves only: no LDS round trips, no waits.
__device__ __forceinline__ double wave_sum_lane63(double v) {
    v += dpp_move<0x111>(v);   // row_shr:1
    v += dpp_move<0x112>(v);   // row_shr:2
    v += dpp_move<0x114>(v);   // row_shr:4
    v += dpp_move<0x118>(v);   // row_shr:8
    v += dpp_move<0x142>(v);   // row_bcast:15
    v += dpp_move<0x143>(v);   // row_bcast:31
    return v;
}

// The same sum broadcast to every lane (readlane of lane 63).
__device__ __forceinline__ double wave_sum(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, wave_sum_lane63(v));
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(u)), 63));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(u >> 32)), 63));
    return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

// Element (column c, sample at byte offset off) of a [column][sample]
// workspace with leading dimension ld: the column's base is wave-uniform and
// the offset a 32-bit lane value, in the global address space, so each access
// is one global_load/store with a scalar base and no vector address arithmetic
// (a generic pointer made them flat accesses with a 64-bit vector add each, and
// the LDS counter to wait for).  The leading dimension is taken through an
// empty asm per access: the bases are then formed where they are used, on the
// scalar unit, instead of being kept for the whole kernel in spilled SGPRs.
typedef __attribute__((address_space(1))) char *gchar;
typedef const __attribute__((address_space(1))) char *cgchar;

__device__ __forceinline__ uint64_t ws_column(const double *ws, int64_t ld, int c) {
    AMI_OPAQUE_S(ld);
    const uint64_t p = reinterpret_cast<uint64_t>(ws) + 8u * static_cast<uint64_t>(c) * static_cast<uint64_t>(ld);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ double ws_load(const double *ws, int64_t ld, int c, uint32_t off) {
    return *(const __attribute__((address_space(1))) double *)((cgchar)ws_column(ws, ld, c) + off);
}

__device__ __forceinline__ void ws_store(double *ws, int64_t ld, int c, uint32_t off, double v) {
    *(__attribute__((address_space(1))) double *)((gchar)ws_column(ws, ld, c) + off) = v;
}

// gfx950 lane exchanges of a double, as two 32-bit halves: swap32 exchanges
// lanes 32-63 of x with lanes 0-31 of y (afterwards x holds the lower halves
// of both, y the upper halves); swap16 exchanges rows 1 and 3 of x with rows 0
// and 2 of y (x then holds the even rows of both, y the odd ones).  Every lane
// of the wave takes part.
__device__ __forceinline__ void swap32(double &x, double &y) {
    const unsigned long long ux = __builtin_bit_cast(unsigned long long, x);
    const unsigned long long uy = __builtin_bit_cast(unsigned long long, y);
    const auto lo = __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(ux), static_cast<unsigned>(uy), false,
                                                     false);
    const auto hi = __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(ux >> 32), static_cast<unsigned>(uy >> 32),
                                                     false, false);
    x = __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi[0])) << 32) |
                                       static_cast<unsigned>(lo[0]));
    y = __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi[1])) << 32) |
                                       static_cast<unsigned>(lo[1]));
}

__device__ __forceinline__ void swap16(double &x, double &y) {
    const unsigned long long ux = __builtin_bit_cast(unsigned long long, x);
    const unsigned long long uy = __builtin_bit_cast(unsigned long long, y);
    const auto lo = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(ux), static_cast<unsigned>(uy), false,
                                                     false);
    const auto hi = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(ux >> 32), static_cast<unsigned>(uy >> 32),
                                                     false, false);
    x = __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi[0])) << 32) |
                                       static_cast<unsigned>(lo[0]));
    y = __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi[1])) << 32) |
                                       static_cast<unsigned>(lo[1]));
}

// Inclusive prefix sums within each row of 16 lanes: lane 15 of a row holds
// the row's sum.
__device__ __forceinline__ double row_sums(double v) {
    v += dpp_move<0x111>(v);   // row_shr:1
    v += dpp_move<0x112>(v);   // row_shr:2
    v += dpp_move<0x114>(v);   // row_shr:4
    v += dpp_move<0x118>(v);   // row_shr:8
    return v;
}

// The wave's totals of (vr, vi), stored at dst[0] and dst[stride]: one swap32
// folds the two halves of the wave, leaving vr's 32 partial sums in rows 0-1
// and vi's in rows 2-3; after the row sums, row_bcast:15 adds row 0 into lane
// 31 (vr's total) and row 2 into lane 63 (vi's total).  Register moves only:
// no LDS, no barrier.
__device__ __forceinline__ void wave_store2(double vr, double vi, int lane, double *dst, int64_t stride) {
    swap32(vr, vi);
    double v = row_sums(vr + vi);
    v += dpp_move<0x142>(v);   // row_bcast:15
    if (lane == 31) dst[0] = v;
    if (lane == 63) dst[stride] = v;
}

// The wave's totals of four values, v_k stored at *p_k (a null p_k: not
// stored).  swap32 on the pairs (v0, v1) and (v2, v3) folds the halves of the
// wave; swap16 on the two results folds row pairs, leaving one value per row
// (rows 0-3: v0, v2, v1, v3), whose row sums end in lanes 15, 31, 47 and 63.
__device__ __forceinline__ void wave_store4(double v0, double v1, double v2, double v3, int lane, double *p0,
                                            double *p1, double *p2, double *p3) {
    swap32(v0, v1);
    swap32(v2, v3);
    double x = v0 + v1, y = v2 + v3;
    swap16(x, y);
    const double v = row_sums(x + y);
    double *const p = lane == 15 ? p0 : lane == 31 ? p2 : lane == 47 ? p1 : lane == 63 ? p3 : nullptr;
    if (p) *p = v;
}

__device__ __forceinline__ void block_sum2(double vr, double vi, double *red, int tid, int B, double *dst) {
    vr = wave_sum(vr);
    vi = wave_sum(vi);
    const int wave = tid >> 6, nwaves = B >> 6;
    if ((tid & 63) == 0) {
        red[2 * wave] = vr;
        red[2 * wave + 1] = vi;
    }
    __syncthreads();
    if (tid == 0) {
        double sr = 0.0, si = 0.0;
        for (int w = 0; w < nwaves; ++w) {
            sr += red[2 * w];
            si += red[2 * w + 1];
        }
        dst[0] = sr;
        dst[1] = si;
    }
    __syncthreads();
}

}  // namespace ami
