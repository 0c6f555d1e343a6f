// Counter-based random numbers of the integrators: Philox4x32-10 (Salmon,
// Moraes, Dror, Shaw, "Parallel random numbers: as easy as 1, 2, 3", SC'11)
// and the Box-Muller map of its words to Gaussians (Section III.C draws the
// random force from Gaussian numbers; this generator replaces the paper's
// Hybrid Taus).
#pragma once

#include <hip/hip_runtime.h>

namespace sop {

// The two products of a round are taken as whole 64-bit ones: one
// instruction each instead of one for either half (the noise of 1e5 particles
// over 1,000 steps: 466 -> 412 us).
__device__ __forceinline__ uint4 philox10(uint4 c, unsigned k0, unsigned k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const unsigned long long p0 = (unsigned long long)0xD2511F53u * c.x;
        const unsigned long long p1 = (unsigned long long)0xCD9E8D57u * c.z;
        c = make_uint4((unsigned)(p1 >> 32) ^ c.y ^ k0, (unsigned)p1, (unsigned)(p0 >> 32) ^ c.w ^ k1, (unsigned)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// Uniform in (0,1) from the top 23 bits: exact in single precision.
__device__ __forceinline__ float unit23(unsigned w)
{
    return (static_cast<float>(w >> 9) + 0.5f) * 0x1p-23f;
}

// sqrt(-2 ln u) for u of unit23, which lies in [2^-24, 1 - 2^-24]: neither the
// logarithm's argument nor the root's is ever below 2^-24, so the general
// functions' scaling of tiny arguments is left out (412 -> 368 us in the case
// above, the same bits).  ln u is log2 u times ln 2 held in two pieces.
__device__ __forceinline__ float radius23(float u)
{
#pragma clang fp contract(off)
    const float l = __builtin_amdgcn_logf(u);
    const float p = l * 0x1.62e42ep-1f;
    const float e = __builtin_fmaf(l, 0x1.efa39ep-25f, __builtin_fmaf(l, 0x1.62e42ep-1f, -p));
    return __builtin_amdgcn_sqrtf(-2.0f * __builtin_fmaf(l, 0x1.62e42ep-1f, e));
}

// Box-Muller: axis 0/1 = radius(u0) * (cos, sin)(2 pi u1), axis 2 =
// radius(u2) * cos(2 pi u3). The logarithm, sine and cosine are the
// hardware ones (the sine and cosine take the angle in turns, so they give
// sin(2 pi u) directly): over all 2^23 uniforms the radius is within 5.7e-7
// and the sine and cosine within 1.3e-7 of FP64, against 5.7e-7 and 5e-8 for
// the library's FP32 functions, at a third of the instructions.
__device__ __forceinline__ float gaussian_axis(const uint4 &w, int axis)
{
    const float ur = unit23(axis < 2 ? w.x : w.z);
    const float ua = unit23(axis < 2 ? w.y : w.w);
    const float rad = radius23(ur);
    return rad * (axis == 1 ? __builtin_amdgcn_sinf(ua) : __builtin_amdgcn_cosf(ua));
}

// Axes 0 and 1 together (one radius, one angle); equal to gaussian_axis.
__device__ __forceinline__ float2 gaussian_pair(const uint4 &w)
{
    const float rad = radius23(unit23(w.x));
    const float ua = unit23(w.y);
    return make_float2(rad * __builtin_amdgcn_cosf(ua), rad * __builtin_amdgcn_sinf(ua));
}

}  // namespace sop
