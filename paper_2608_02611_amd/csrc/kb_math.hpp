// kb_math.hpp -- binary64 logarithm, square root and sine / cosine for the
// seeded generator, and their binary32 forms for 16-bit outputs.
//
// The generator's arguments are 32-bit words mapped to (0, 1] and [0, 2 pi),
// so none of what a general library function carries is needed: no
// Payne-Hanek reduction, no double-double tail, no special values.  A
// Box-Muller pair takes about 70 binary64 operations this way, where the
// general functions took about 300 (the generator is bound by instruction
// issue, not by memory; 3 x 33.5 million fp16 normals: 297 -> 170 us, the
// Student-t of 16.8 million elements, taken literally: 245 -> 150 us).  The
// logarithm, root, sine and cosine are within 2.6 units in the last place of
// binary64, the Student-t within 4.4, so the binary32 rounding of a result
// moves about as rarely as between two general libraries: a few values in 10^8
// differ by one unit in the last place of binary32 from what those gave.
//
// Method: argument reduction, then a polynomial whose coefficients are the
// minimax ones of the stated function on the stated interval (computed by
// the Remez exchange in 300-bit arithmetic, then rounded to binary64).
// Reciprocals and inverse square roots start from a seed of relative error
// about 2^-24 and take one third-order step (error about 2^-72, then
// rounding).
//
// Plain C++: the host can compile it too (a Seed type supplies the seeds), so
// the error bounds are checked on the CPU, at the ends of every interval and on
// words spread over the range.
#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define KB_MATH __host__ __device__ __forceinline__
#else
#define KB_MATH inline
#endif

namespace kb {

KB_MATH double math_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// T = -2 ln u for u = (x + 1) 2^-32 in (0, 1]; 0 for u = 1.  u = f 2^e with f
// in [sqrt(1/2), sqrt(2)), s = (f - 1) / (f + 1), w = s^2 < 0.0295:
// -2 ln f = s (-4 + w Q(w)), Q(w) = -4 (atanh(s) / s - 1) / w (minimax,
// relative error of -2 ln f 2^-59.5).  f - 1 is exact and e = 0 for u near 1,
// so the result keeps its relative accuracy as it goes to zero.
template <class Seed>
KB_MATH double neg2_log_u01(uint32_t x) {
    const double v = (double)x + 1.0;  // exact, 1 .. 2^32
    double f = Seed::frexp_mant(v);    // [1/2, 1)
    const int below = f < 0x1.6a09e667f3bcdp-1 ? 1 : 0;
    f = Seed::ldexp(f, below);
    const double e = (double)(Seed::frexp_exp(v) - 32 - below);
    const double n = f - 1.0, d = f + 1.0;
    const double y = Seed::rcp(d);
    const double r = math_fma(-d, y, 1.0);
    const double q = n * y;
    const double s = math_fma(q, math_fma(r, r, r), q);
    const double w = s * s;
    double Q = -0x1.2f0d8e947b4f2p-2;
    Q = math_fma(Q, w, -0x1.39a0f5130ff64p-2);
    Q = math_fma(Q, w, -0x1.7466462b0f919p-2);
    Q = math_fma(Q, w, -0x1.c71c51e80442cp-2);
    Q = math_fma(Q, w, -0x1.249249421787dp-1);
    Q = math_fma(Q, w, -0x1.999999997fb34p-1);
    Q = math_fma(Q, w, -0x1.5555555555593p+0);
    return math_fma(e, -0x1.62e42fefa39efp+0, s * math_fma(Q, w, -4.0));
}

// sqrt(x), x >= 0 (no subnormals).
template <class Seed>
KB_MATH double math_sqrt(double x) {
    // (a seed of 1/sqrt(0) would be infinite; with the floor, x = 0 gives 0)
    const double y = Seed::rsq(__builtin_fmax(x, 0x1p-1000));
    const double g = x * y;
    const double e = math_fma(-g, y, 1.0);
    return math_fma(g * e, math_fma(e, 0.375, 0.5), g);
}

// 1 / sqrt(x), x >= 2^-1000.
template <class Seed>
KB_MATH double math_rsqrt(double x) {
    const double y = Seed::rsq(x);
    const double e = math_fma(-(x * y), y, 1.0);
    return math_fma(y * e, math_fma(e, 0.375, 0.5), y);
}

// Sine and cosine of theta, the binary64 rounding of 2 pi u (2 pi rounded to
// binary64 too), u = x 2^-32.  The quadrant comes from x; theta minus its
// multiple of pi / 2, in two parts, is exact up to its last rounding (also
// where the sine or cosine is nearly zero).
KB_MATH void sincos_2pi_u(uint32_t x, double& sn, double& cs) {
    const double theta = 0x1.921fb54442d18p-30 * (double)x;  // (2 pi 2^-32) x
    const uint32_t q = ((x >> 29) + 1u) >> 1;                // 0 .. 4, nearest multiple
    const double qd = (double)q;
    double r = math_fma(-qd, 0x1.921fb54442d18p+0, theta);
    r = math_fma(-qd, 0x1.1a62633145c07p-54, r);
    const double z = r * r;
    // sin r = r + r z S(z) (2^-58 relative), cos r = 1 + z (-1/2 + z C(z)) (2^-64)
    double S = 0x1.5d9318136495dp-33;
    S = math_fma(S, z, -0x1.ae5e668766e82p-26);
    S = math_fma(S, z, 0x1.71de357814d5dp-19);
    S = math_fma(S, z, -0x1.a01a019c12010p-13);
    S = math_fma(S, z, 0x1.111111110f87dp-7);
    S = math_fma(S, z, -0x1.5555555555549p-3);
    const double s = math_fma(r * z, S, r);
    double C = -0x1.8faeb6333d309p-37;
    C = math_fma(C, z, 0x1.1ee9ec192f146p-29);
    C = math_fma(C, z, -0x1.27e4f80a34992p-22);
    C = math_fma(C, z, 0x1.a01a019cb217dp-16);
    C = math_fma(C, z, -0x1.6c16c16c15181p-10);
    C = math_fma(C, z, 0x1.555555555554cp-5);
    const double c = math_fma(z, math_fma(z, C, -0.5), 1.0);
    const bool odd = (q & 1u) != 0u;
    const uint64_t sb = __builtin_bit_cast(uint64_t, odd ? c : s);
    const uint64_t cb = __builtin_bit_cast(uint64_t, odd ? s : c);
    sn = __builtin_bit_cast(double, sb ^ ((uint64_t)((q << 30) & 0x80000000u) << 32));
    cs = __builtin_bit_cast(double, cb ^ ((uint64_t)(((q + 1u) << 30) & 0x80000000u) << 32));
}

// Box-Muller on one word pair: rho cos(theta), rho sin(theta) with
// rho = sqrt(-2 ln u1), theta = 2 pi u2, u1 = (xa + 1) 2^-32, u2 = xb 2^-32.
template <class Seed>
KB_MATH void box_muller64(uint32_t xa, uint32_t xb, double& zc, double& zs) {
    const double rho = math_sqrt<Seed>(neg2_log_u01<Seed>(xa));
    double s, c;
    sincos_2pi_u(xb, s, c);
    zc = rho * c;
    zs = rho * s;
}

// The same pair in binary32, for results that are stored in 16 bits.
//
// rho = sqrt(-2 ln u): u rounded to 24 bits as f, log2 of f 2^-32 by the
// hardware (v_log_f32), and the rounding of u put back to first order where
// it matters: log2(u) - log2(f 2^-32) = lo log2(e) / v, lo = v - f, with
// 1 / u taken as 2 - u (exact to (1 - u)^2 where the logarithm goes to zero;
// below u = 1/2 the term is under 2^-24 of the logarithm anyway).  Sure where
// 1 - u is above about 2^-21.5.
// Largest error over all 2^32 words on the device, against the binary64
// functions: rho 2^-22.6 of its value wherever it is sure, sin and cos 2^-22.3;
// on the host rho 2^-22.9 with the logarithm and the root as rounded, 2^-22.2
// with both off by one unit in the last place.
template <class Seed>
KB_MATH float rho32(uint32_t x, bool& sure) {
    const uint32_t v = x + 1u;  // (0 for u = 1: f = 0, not sure)
    const float f = (float)v;
    const float u = f * 0x1p-32f;
    const float lo = (float)(int32_t)(v - Seed::to_u32(f));
    const float L = __builtin_fmaf(lo * 0x1.715476p-32f, 2.0f - u, Seed::log2(u));  // log2(u) <= 0
    sure = L < -0x1p-21f && v != 0u;
    return Seed::sqrt32(L * -0x1.62e43p+0f);
}

// sin and cos of 2 pi x 2^-32 in binary32: the quadrant and the remainder r
// (|r| <= pi / 4) come from the integer, so the relative error holds at the
// zeros too.  sin r = r + r z (S0 + S1 z + S2 z^2) (minimax, 2^-28), cos r =
// 1 - z / 2 + z^2 (C0 + C1 z + C2 z^2) (2^-33), z = r^2.  Not sure next to a
// multiple of pi / 2, where the binary64 path's rounding of theta shows.
KB_MATH void sincos32(uint32_t x, float& sn, float& cs, bool& sure) {
    const uint32_t q = ((x >> 29) + 1u) >> 1;
    const int32_t ri = (int32_t)(x - (q << 30));
    sure = (uint32_t)(ri + 16) >= 32u;
    const float r = (float)ri * 0x1.921fb6p-30f;
    const float z = r * r;
    float S = __builtin_fmaf(-0x1.994388p-13f, z, 0x1.11073ap-7f);
    S = __builtin_fmaf(S, z, -0x1.555546p-3f);
    const float s = __builtin_fmaf(r * z, S, r);
    float C = __builtin_fmaf(0x1.99eb4ap-16f, z, -0x1.6c0c32p-10f);
    C = __builtin_fmaf(C, z, 0x1.55554ap-5f);
    C = __builtin_fmaf(C, z, -0.5f);
    const float c = __builtin_fmaf(C, z, 1.0f);
    const bool odd = (q & 1u) != 0u;
    const uint32_t sb = __builtin_bit_cast(uint32_t, odd ? c : s);
    const uint32_t cb = __builtin_bit_cast(uint32_t, odd ? s : c);
    sn = __builtin_bit_cast(float, sb ^ ((q << 30) & 0x80000000u));
    cs = __builtin_bit_cast(float, cb ^ (((q + 1u) << 30) & 0x80000000u));
}

// Student-t with 3 degrees of freedom of one block's words x, y, z (, w): the
// ratio of the first normal to the root of the other three's mean square (a
// chi-square over its degrees of freedom).  With T1, T2 = -2 ln u of the two
// pairs and theta the angle of the first,
//   z0 = sqrt(T1) cos theta, z1^2 = T1 sin^2 theta, z2^2 + z3^2 = T2
// (sin^2 + cos^2 = 1: the second pair's angle drops out), so
//   t = cos theta sqrt(3 T1 / D), D = T1 sin^2 theta + T2
//     = cos theta A rsqrt(A D),   A = 3 T1:
// one sine and cosine, one inverse root and no quotient, where the definition
// read literally takes two, three and one.  Bound by instruction issue: 16.8
// million fp32 elements 87 us, 121 us taken literally.
template <class Seed>
KB_MATH double student_t3_64(uint32_t x, uint32_t y, uint32_t z) {
    const double T1 = neg2_log_u01<Seed>(x), T2 = neg2_log_u01<Seed>(z);
    double s, c;
    sincos_2pi_u(y, s, c);
    const double A = 3.0 * T1, D = math_fma(T1 * s, s, T2);
    // A = 0 gives 0 (the floor keeps the inverse root finite); D = 0 (u = 1
    // in the second pair and z1 = 0) gives the quotient by zero
    double r = math_rsqrt<Seed>(__builtin_fmax(A * D, 0x1p-1000));
    r = D == 0.0 ? __builtin_inf() : r;
    return c * (A * r);
}

}  // namespace kb
