// Accurate single-precision sin/cos for the feature kernels (internal header).
#pragma once

#include <hip/hip_runtime.h>

namespace rfsf {
namespace {

// On [-pi/4, pi/4] sin r = r + r^3 P(r^2) and cos r = 1 - r^2/2 + r^4 Q(r^2), P and Q of degree 2 with the least maximal absolute
// error of sine and cosine (1.8e-9 and 1.0e-10: a linear program over 4001 points, then rounded to 32 bits). Evaluated in 32 bits
// the sine is off by 4.0e-8 at most (root mean square 1.1e-8), the cosine by 7.4e-8 (2.5e-8).
constexpr float kSinP[3] = {-1.6666650772e-1f, 8.331975900e-3f, -1.9495293964e-4f};
constexpr float kCosQ[3] = {4.1666645557e-2f, -1.3887364184e-3f, 2.4438091714e-5f};

// sin and cos of x to ~1e-7 absolute for |x| up to 1e5: two-term Cody-Waite reduction by
// pi/2 with fused multiply-adds, then the polynomials above
// and a quadrant swap. The time difference cancels leading digits, so the
// fast hardware approximations are not accurate enough here.
__device__ __forceinline__ void sincos_reduced(float x, float &s, float &c)
{
    const float kf = rintf(x * 0.636619772367581343f);
    float r = fmaf(-kf, 1.57079637050628662109375f, x);
    r = fmaf(-kf, -4.37113900018624283e-8f, r);
    const float r2 = r * r;
    const float ps = fmaf(r2, fmaf(r2, kSinP[2], kSinP[1]), kSinP[0]);
    const float S = fmaf(r * r2, ps, r);
    const float pc = fmaf(r2, fmaf(r2, kCosQ[2], kCosQ[1]), kCosQ[0]);
    const float C = fmaf(r2 * r2, pc, fmaf(-0.5f, r2, 1.0f));
    const int q = (int)kf;
    const float ss = (q & 1) ? C : S;
    const float cc = (q & 1) ? S : C;
    // sin flips sign in quadrants 2, 3; cos in quadrants 1, 2.
    s = __uint_as_float(__float_as_uint(ss) ^ (((unsigned)q & 2u) << 30));
    c = __uint_as_float(__float_as_uint(cc) ^ ((((unsigned)q + 1u) & 2u) << 30));
}

// The same of x (a + b) quarter-turns, a + b the number of them in a unit of x to twice the precision: what rounding x a would cut off
// stays in the reduced argument, so that large angles are no less accurate than x itself. Maximal
// error 4.2e-8 (sine) and 5.8e-8 (cosine), root mean square 1.1e-8 and 1.8e-8 (of sincos_reduced on a reduced argument: 4.0e-8,
// 7.4e-8, 1.1e-8, 2.5e-8). Polynomials in r^2 fitted to least maximal error on [-1/2, 1/2].
//
// Instructions are chosen by what they cost: with 16 wavefronts per CU, multiply-adds, additions and three-operand logic of vector
// registers take 2.6 cycles of a SIMD, the same with a scalar register as an operand 4.35, and so do conversions, roundings, shifts,
// comparisons and selects. So the sine and the cosine are chosen and signed by logic, and all that is constant is in vector registers
// (Quarters, made where the registers are free): 65 cycles instead of 80. Counting quarter-turns by adding 1.5 * 2^23 would spare
// another 6 (1500 x 200 points, 64 to 256 buckets, one to eight channels: none to 2.5 % of the kernel), but the sum's last bits count to 2^22
// only, angles of 6.6e6. As it is, angles of exact products up to 2^23 radians give a level's block to 5e-7, and up to 2^24, where the
// product's rounding takes r past 1/2, to 9e-6, as in the kernel that takes its increments from memory.
struct Quarters {
    float a, b;
    uint32_t top;
    __device__ __forceinline__ Quarters(float a_, float b_) : a(a_), b(b_), top(0x80000000u)
    {
        asm volatile("" : "+v"(a), "+v"(b), "+v"(top));
    }
};
__device__ __forceinline__ void sincos_quarters(float x, const Quarters &turn, float &s, float &c)
{
    const float k = rintf(x * turn.a), r = fmaf(x, turn.b, fmaf(x, turn.a, -k)), r2 = r * r;
    const float rest = r * fmaf(r2, fmaf(r2, fmaf(r2, -4.592289216816425e-3f, 7.967590540647507e-2f), -6.459629535675049e-1f), -6.54208633932285e-8f);
    const uint32_t S = __float_as_uint(fmaf(r, 1.57079637050628662109375f, rest));
    const uint32_t C = __float_as_uint(fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, 9.040216682478786e-4f, -2.086028829216957e-2f), 2.5366923213005066e-1f),
                                                     -1.2337005138397217f), 1.0f));
    const int q = (int)k;
    const uint32_t odd = (uint32_t)__builtin_amdgcn_sbfe(q, 0, 1), signs = (uint32_t)q << 30;
    // odd ? one : the other, then the sign bit: sin flips in quadrants 2, 3; cos in quadrants 1, 2
    const uint32_t ss = __builtin_amdgcn_bitop3_b32(odd, C, S, 0xca), cc = __builtin_amdgcn_bitop3_b32(odd, S, C, 0xca);
    s = __uint_as_float(__builtin_amdgcn_bitop3_b32(ss, signs, turn.top, 0x78));
    c = __uint_as_float(__builtin_amdgcn_bitop3_b32(cc, signs + 0x40000000u, turn.top, 0x78));
}

}  // namespace
}  // namespace rfsf
