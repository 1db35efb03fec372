// Device helpers shared by the ahead-of-time kernels of libqaia.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace qaia {

// Counter-based SplitMix64 (Steele, Lea and Flood, OOPSLA 2014): the value
// for counter idx is the (idx+1)-th output of the stream whose state starts
// at seed (state += golden gamma, then the variant-13 finaliser).
__device__ __forceinline__ uint64_t splitmix64_finish(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t idx) {
    return splitmix64_finish(seed + (idx + 1ull) * 0x9e3779b97f4a7c15ull);
}

// Initial soft spin / momentum: 24-bit uniform u, v = 2u - 1 (exact in
// float32), value = float32(amp * v).
__device__ __forceinline__ float init_value(uint64_t seed, uint64_t idx, float amp) {
    uint64_t bits = splitmix64(seed, idx);
    float u = (float)(uint32_t)(bits >> 40) * 0x1p-24f;
    float v = 2.0f * u - 1.0f;
    return amp * v;
}

// Counter of the initial draw of spin i of global replica g (x: 0, y: 1).
__device__ __forceinline__ uint64_t init_counter(uint64_t g, int n, int i, int comp) {
    return ((g * (uint64_t)n + (uint64_t)i) << 1) | (uint64_t)comp;
}

// Standard normal for noise injection (Eq. 10): Box-Muller on two 24-bit
// uniforms of one draw from the keyed stream.  Noise-injected sampling is
// bound by the VALU work of this function, so it is written for its own
// arguments only, with the same values as sqrtf(-2 logf(u1)) cosf(2 pi u2)
// (compared on the device for all 2^24 u1, and for all 2^24 u2):
//  - ln u = log2 u * ln 2 in the steps, and with the two floats of ln 2, of the
//    compiler's own logf (the hardware log2, its product with the high float, that
//    product's remainder, the low float, summed with fused operations), which is
//    what the same values take; u1 is in [2^-24, 1], so there is no denormal or
//    infinity to look for (22 -> 5 operations);
//  - sqrt by one correction of x rsq(x) from its exact residual, x in
//    [0, 33.3]; the bound on rsq makes sqrt(0) = 0 (20 -> 6);
//  - the angle is below 2 pi, which is stated to the compiler: it drops the
//    cosine's reduction of large arguments (132 -> 31), and with it most of
//    the code whose 42 copies (one per spin of a generated kernel) did not fit
//    the instruction cache.
constexpr uint64_t kNoiseKey = 0xd1b54a32d192ed03ull;
// (z: the stream's state at the draw, (seed ^ kNoiseKey) + (idx + 1) * gamma)
__device__ __forceinline__ float noise_from(uint64_t z) {
    const uint64_t bits = splitmix64_finish(z);
    const float u1 = (float)((uint32_t)(bits >> 40) + 1u) * 0x1p-24f;
    const float u2 = (float)(uint32_t)(bits & 0xffffffu) * 0x1p-24f;
    const float l2 = __builtin_amdgcn_logf(u1);
    const float ln2h = 0x1.62e42ep-1f, ln2l = 0x1.efa39ep-25f;  // ln 2 = ln2h + ln2l
    // every fusion is written out: left to the compiler, the last sum's would depend on its flags
    const float ln = fmaf(l2, ln2h, fmaf(l2, ln2l, fmaf(l2, ln2h, -(l2 * ln2h))));
    const float x = -2.0f * ln;
    const float rs = fminf(fabsf(__builtin_amdgcn_rsqf(x)), 0x1p60f);
    const float s0 = x * rs;
    const float radius = fmaf(fmaf(-s0, s0, x), 0.5f * rs, s0);
    const float angle = 6.2831853071795864769f * u2;
    __builtin_assume(__builtin_fabsf(angle) < 131072.0f);  // (fabsf, a call to the front end, would be ignored)
    return radius * cosf(angle);
}
__device__ __forceinline__ float noise_value(uint64_t seed, uint64_t idx) {
    return noise_from((seed ^ kNoiseKey) + (idx + 1ull) * 0x9e3779b97f4a7c15ull);
}

// sgn with sgn(0) = +1 (x is never -0 in these dynamics).
__device__ __forceinline__ float sgn1(float x) { return x >= 0.0f ? 1.0f : -1.0f; }

// Inelastic wall: |x| > 1 -> x = sgn x, y = 0.
__device__ __forceinline__ void wall(float &x, float &y) {
    if (fabsf(x) > 1.0f) {
        x = x > 0.0f ? 1.0f : -1.0f;
        y = 0.0f;
    }
}

}  // namespace qaia
