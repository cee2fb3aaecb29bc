// Counter-based normal draws shared by the kernels that draw the up-front
// noise of Algorithm 1 (the prior point and every step's noise): Philox4x32-10
// (Salmon, Moraes, Dror, Shaw, SC'11) with Box-Muller in double precision.
// Counter block q of stream s is (q mod 2^32, q / 2^32, s, 0) under the key
// (seed mod 2^32, seed / 2^32); it gives values 4q .. 4q + 3 of the stream.
#pragma once

#include <cstdint>

namespace pd {

constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

__device__ __forceinline__ void philox4x32_10(uint32_t& c0, uint32_t& c1, uint32_t& c2,
                                              uint32_t& c3, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += kPhiloxW0;
            k1 += kPhiloxW1;
        }
        // whole 64-bit products (one multiply each)
        const uint64_t p0 = (uint64_t)kPhiloxM0 * c0, p1 = (uint64_t)kPhiloxM1 * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = hi1 ^ c1 ^ k0;
        const uint32_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
}

// Box-Muller on u = (r + 0.5) 2^-32, in double precision.  The arguments are
// few and regular, so each function needs only its series on a short interval,
// with no range checks: the coefficients interpolate the functions' own power
// series at Chebyshev nodes (errors below, relative).  The results are within
// 2^-48 of the exact ones, so that their rounding to float differs from it in
// about one value of ten million.  36.9 million normals take 62 us,
// 119 with the math library's log, sincos and sqrt.

// -2 log(u): u = m 2^e with m in [sqrt(1/2), sqrt 2), log m = 2 atanh(z) at
// z = (m - 1) / (m + 1), |z| < 0.172 (series error 2^-50)
__device__ __forceinline__ double neg_2_log_u(uint32_t r) {
    const double d = (double)r + 0.5;                       // exact
    double m = __builtin_amdgcn_frexp_mant(d);              // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(d) - 32;
    const bool low = m < 0.70710678118654752;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double a = m - 1.0, b = m + 1.0;                  // exact (m has 33 bits)
    double y = __builtin_amdgcn_rcp(b);
    y = __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
    double z = a * y;
    z = __builtin_fma(__builtin_fma(-b, z, a), y, z);
    const double w = z * z;
    double p = 0.1662194703841815;
    p = __builtin_fma(p, w, 0.1814018520643775);
    p = __builtin_fma(p, w, 0.22222862476743502);
    p = __builtin_fma(p, w, 0.2857142413651753);
    p = __builtin_fma(p, w, 0.40000000011212195);
    p = __builtin_fma(p, w, 0.6666666666666208);
    const double lm = __builtin_fma(z * w, p, z + z);
    return -2.0 * __builtin_fma((double)e, 0.6931471805599453, lm);
}
// sqrt(a), a > 0 and normal, from the hardware's estimate of a^-1/2 (2^-23) by
// two steps on the square root
__device__ __forceinline__ double sqrt_pos(double a) {
    const double y = __builtin_amdgcn_rsq(a), h = 0.5 * y;
    double g = a * y;
    g = __builtin_fma(__builtin_fma(-g, g, a), h, g);
    return __builtin_fma(__builtin_fma(-g, g, a), h, g);
}
// (cos, sin)(2 pi u): the nearest quarter turn by integer arithmetic, the rest
// |x| <= pi / 4 by series (2^-49.7 and 2^-55.6)
__device__ __forceinline__ void cos_sin_u(uint32_t r, double& c, double& s) {
    const uint32_t q = (r + 0x20000000u) >> 30;
    const double x = __builtin_fma((double)(int32_t)(r - (q << 30)), 1.4629180792671596e-09, 7.314590396335798e-10);
    const double w = x * x;
    double ps = 1.591811582755219e-10;
    ps = __builtin_fma(ps, w, -2.505113165923371e-08);
    ps = __builtin_fma(ps, w, 2.7557316101663618e-06);
    ps = __builtin_fma(ps, w, -0.00019841269836756842);
    ps = __builtin_fma(ps, w, 0.008333333333330948);
    ps = __builtin_fma(ps, w, -0.16666666666666666);
    const double sx = __builtin_fma(x * w, ps, x);
    double pc = 2.070058293634169e-09;
    pc = __builtin_fma(pc, w, -2.755636950611903e-07);
    pc = __builtin_fma(pc, w, 2.480158521036432e-05);
    pc = __builtin_fma(pc, w, -0.0013888888887276698);
    pc = __builtin_fma(pc, w, 0.04166666666666468);
    const double cx = __builtin_fma(w * w, pc, __builtin_fma(w, -0.5, 1.0));
    const double a = (q & 1) ? sx : cx, b = (q & 1) ? cx : sx;
    c = ((q + 1) & 2) ? -a : a;
    s = (q & 2) ? -b : b;
}

// Values 4q .. 4q + 3 of counter stream rng_stream, rounded to float.
__device__ __forceinline__ void normals4(uint64_t seed, uint32_t rng_stream, int64_t q, float (&v)[4]) {
    uint32_t c0 = (uint32_t)q, c1 = (uint32_t)((uint64_t)q >> 32), c2 = rng_stream, c3 = 0;
    philox4x32_10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
    const double r01 = sqrt_pos(neg_2_log_u(c0)), r23 = sqrt_pos(neg_2_log_u(c2));
    double s1, co1, s3, co3;
    cos_sin_u(c1, co1, s1);
    cos_sin_u(c3, co3, s3);
    v[0] = (float)(r01 * co1);
    v[1] = (float)(r01 * s1);
    v[2] = (float)(r23 * co3);
    v[3] = (float)(r23 * s3);
}

}  // namespace pd
