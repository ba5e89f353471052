// Counter-based Gaussian noise for the GLE thermostat, device side.
//
// Generator: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, "Parallel random
// numbers: as easy as 1, 2, 3", SC'11): ten rounds of two 32x32->64-bit
// multiplications by fixed odd constants, with a Weyl-sequence key schedule.
//
// Counter layout (one block = four normals, for four consecutive replicas):
//   key     = (seed mod 2^32, seed >> 32)
//   counter = (dof i, step n, (component j << 16) | (replica r >> 2), stream)
// Word w = r & 3 of the block belongs to replica r.  Each word x becomes
// u = (2 (x >> 9) + 1) 2^-24, an odd multiple of 2^-24 in (0, 1), exact in
// FP32 and FP64.  Box-Muller on words (0, 1) and (2, 3): the even word gives
// sqrt(-2 ln u_even) cos(2 pi u_odd), the odd word the same radius times
// sin(2 pi u_odd).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace fth {
namespace dev {

struct Block4 {
    uint32_t w[4];
};

__device__ __forceinline__ Block4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1) {
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
    constexpr uint32_t kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t pa = uint64_t(kMulA) * c0;
        const uint64_t pb = uint64_t(kMulB) * c2;
        // three-way XOR in one v_bitop3_b32 (truth table 0x96)
        const uint32_t x0 = __builtin_amdgcn_bitop3_b32(uint32_t(pb >> 32), c1, k0, 0x96);
        const uint32_t x2 = __builtin_amdgcn_bitop3_b32(uint32_t(pa >> 32), c3, k1, 0x96);
        c1 = uint32_t(pb);
        c3 = uint32_t(pa);
        c0 = x0;
        c2 = x2;
        k0 += kWeylA;
        k1 += kWeylB;
    }
    return Block4{{c0, c1, c2, c3}};
}

// u = (2 (x >> 9) + 1) 2^-24 in FP32 without a conversion: the top 23 bits
// as the mantissa of a float in [1, 2) give 1 + (x >> 9) 2^-23, and
// subtracting 1 - 2^-24 is exact (Sterbenz: both operands lie in [1/2, 2]).
// The bit pattern 0x3f800000 | (x >> 9) is the low word of the 64-bit value
// {0x7f, x} shifted right by 9: one v_alignbit_b32 instead of a shift and an or.
__device__ __forceinline__ float uniform_f32(uint32_t x) {
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7fu, x, 9u)) - 0x1.fffffep-1f;
}

// Box-Muller in FP32 with the hardware transcendental unit: v_log_f32 is
// log2, v_sin_f32 / v_cos_f32 take their argument in revolutions, so
// sin(2 pi u) needs no multiply.
__device__ __forceinline__ void box_muller(uint32_t a, uint32_t b, float& zc, float& zs) {
    const float ua = uniform_f32(a);
    const float ub = uniform_f32(b);
    const float l2 = __builtin_amdgcn_logf(ua);                      // log2(ua) < 0
    const float rad = __builtin_amdgcn_sqrtf(-1.3862943611198906f * l2);  // sqrt(-2 ln ua)
    zc = rad * __builtin_amdgcn_cosf(ub);
    zs = rad * __builtin_amdgcn_sinf(ub);
}

// sqrt(-2 ln u) in FP64 for u = (2 (x >> 9) + 1) 2^-24, the only arguments there
// are.  u is exact in FP32, so the reduction u = 2^e f, f in [sqrt(1/2), sqrt(2)),
// is integer work, and f - 1 and f + 1 are exact in FP64:
//   ln f = 2 artanh(s), s = (f - 1) / (f + 1), = 2 s + s^3 R(s^2),
// R the degree-6 interpolant at Chebyshev nodes (error 2^-57 of 2 s).  The
// quotient and the root start from the FP32 hardware estimates and take one
// Newton step each and a correction by the exact residual, so neither needs the
// scaling and special cases of a general division or root.  Against 80-bit
// arithmetic over all 2^23 arguments: at most 0.86 ulp, 0.27 on average (the same
// as a correctly rounded-to-0.52-ulp log followed by a correctly rounded root).
__device__ __forceinline__ double radius_f64(uint32_t x) {
    const uint32_t ix = __float_as_uint(uniform_f32(x)) + (0x3f800000u - 0x3f3504f3u);  // 0x3f3504f3: sqrt(1/2)
    const float ff = __uint_as_float((ix & 0x007fffffu) + 0x3f3504f3u);
    const double w = double(254 - 2 * int(ix >> 23));  // -2 e
    const double f = double(ff), num = f - 1.0, den = f + 1.0;
    double rc = double(__builtin_amdgcn_rcpf(ff + 1.0f));
    rc = __builtin_fma(rc, __builtin_fma(-den, rc, 1.0), rc);
    const double s0 = num * rc, ds = __builtin_fma(-s0, den, num) * rc, s = s0 + ds;
    const double z = s * s;
    double r = 0x1.2b584aae78a57p-3;
    r = __builtin_fma(r, z, 0x1.39fe606542ddep-3);
    r = __builtin_fma(r, z, 0x1.7462b4ab2ef6bp-3);
    r = __builtin_fma(r, z, 0x1.c71c62e5800a1p-3);
    r = __builtin_fma(r, z, 0x1.2492492df148dp-2);
    r = __builtin_fma(r, z, 0x1.99999999952e2p-2);
    r = __builtin_fma(r, z, 0x1.5555555555558p-1);
    // -2 ln u = w ln 2 - 4 s - 2 s^3 R with the two large terms' rounding error kept
    // (w times the first part of ln 2 is exact)
    const double hi = w * 0x1.62e42fefa3800p-1, a = __builtin_fma(-4.0, s0, hi);
    double l = __builtin_fma(-4.0, s0, hi - a);
    l = __builtin_fma(w, 0x1.ef35793c76730p-45, l);
    l = __builtin_fma(-4.0, ds, l);
    l = a + __builtin_fma(-2.0, (s * z) * r, l);
    const double y = double(__builtin_amdgcn_rsqf(float(l)));
    double g = l * y, h = 0.5 * y;
    const double d = __builtin_fma(-g, h, 0.5);
    g = __builtin_fma(g, d, g);
    h = __builtin_fma(h, d, h);
    return __builtin_fma(__builtin_fma(-g, g, l), h, g);
}

// cos(2 pi u) and sin(2 pi u) in FP64 for the same u: the octant comes off the
// integer, leaving X 2^-24 turns with X an odd integer, |X| < 2^21, whose square
// is exact.  Interpolants at Chebyshev nodes in Y = X^2 (errors below 2^-57; at
// most 0.91 ulp over all arguments),
// the powers of 2^-24 folded into the coefficients; 2 pi in two parts.
__device__ __forceinline__ void turn_f64(uint32_t x, double& cs, double& sn) {
    const uint32_t t = x >> 9;
    const uint32_t j = (t + (1u << 20)) >> 21;
    const double X = double(2 * (int(t) - int(j << 21)) + 1);
    const double Y = X * X;
    double p = 0x1.e4a9d9166f052p-311;
    p = __builtin_fma(p, Y, -0x1.e3027dea82bd7p-261);
    p = __builtin_fma(p, Y, 0x1.50783208843ebp-211);
    p = __builtin_fma(p, Y, -0x1.32d2cce500387p-162);
    p = __builtin_fma(p, Y, 0x1.466bc6775a476p-114);
    p = __builtin_fma(p, Y, -0x1.4abbce625be52p-67);
    p = __builtin_fma(p, Y, 0x1.1a62633145c07p-76);
    const double S = __builtin_fma(X, 0x1.921fb54442d18p-22, X * p);
    double c = -0x1.b2f3eb054afcdp-336;
    c = __builtin_fma(c, Y, 0x1.f9ce245cada0bp-286);
    c = __builtin_fma(c, Y, -0x1.a6d1eef479be1p-236);
    c = __builtin_fma(c, Y, 0x1.e1f5068688d5bp-187);
    c = __builtin_fma(c, Y, -0x1.55d3c7e3cb241p-138);
    c = __builtin_fma(c, Y, 0x1.03c1f081b5ac0p-90);
    c = __builtin_fma(c, Y, -0x1.3bd3cc9be45dep-44);
    const double C = __builtin_fma(c, Y, 1.0);
    const double a = (j & 1u) ? S : C, b = (j & 1u) ? C : S;
    cs = ((j + 1u) & 2u) ? -a : a;
    sn = (j & 2u) ? -b : b;
}

// Box-Muller in FP64.  Each function has 2^23 possible arguments, so it carries
// none of the general cases of the device math library's log, sqrt and sincospi:
// about 54 FP64 instructions a pair against 112, 120 vector instructions against 200.
__device__ __forceinline__ void box_muller(uint32_t a, uint32_t b, double& zc, double& zs) {
    const double rad = radius_f64(a);
    double cs, sn;
    turn_f64(b, cs, sn);
    zc = rad * cs;
    zs = rad * sn;
}

// Normals of component j for replicas r0 .. r0+RPT-1 (r0 a multiple of RPT;
// RPT in {1, 2, 4, 8}) at dof i, step n.
template <typename Real, int RPT>
__device__ __forceinline__ void normals(uint32_t k0, uint32_t k1, uint32_t stream, uint32_t i,
                                        uint32_t n, uint32_t j, uint32_t r0, Real* z) {
    if constexpr (RPT >= 4) {
#pragma unroll
        for (int g = 0; g < RPT / 4; ++g) {
            const Block4 b = philox4x32_10(i, n, (j << 16) | ((r0 >> 2) + g), stream, k0, k1);
            box_muller(b.w[0], b.w[1], z[4 * g + 0], z[4 * g + 1]);
            box_muller(b.w[2], b.w[3], z[4 * g + 2], z[4 * g + 3]);
        }
    } else {
        const Block4 b = philox4x32_10(i, n, (j << 16) | (r0 >> 2), stream, k0, k1);
        const bool hi = (r0 & 2u) != 0;
        Real zc, zs;
        box_muller(hi ? b.w[2] : b.w[0], hi ? b.w[3] : b.w[1], zc, zs);
        if constexpr (RPT == 2) {
            z[0] = zc;
            z[1] = zs;
        } else {
            z[0] = (r0 & 1u) ? zs : zc;
        }
    }
}

}  // namespace dev
}  // namespace fth
