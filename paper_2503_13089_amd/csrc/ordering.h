// Device helpers of the (norm shell, cosine) ordering key, shared by the ordering machinery (sort.hip) and the cells
// (cells.hip).
#pragma once
#include "common.h"

namespace cc {

// 16-bit norm key: the top half of the fp32 pattern of a non-negative float (monotone, 2^-7 relative steps)
__device__ __forceinline__ uint32_t norm_key(float norm) { return __float_as_uint(norm) >> 16; }

// Shells: 4 norm keys each. `base` places shell 511 at the largest norm any vector can have; everything
// 511 shells (16 octaves) or more below that shares shell 0, anything above shares shell 511.
__device__ __forceinline__ uint32_t shell_base(uint32_t absmax_bits, int d)
{
    const float top = __uint_as_float(absmax_bits) * __builtin_sqrtf(float(d)) * 1.0001f;
    const uint32_t tk = norm_key(top) >> 2;
    return tk > 511u ? tk - 511u : 0u;
}
__device__ __forceinline__ uint32_t shell_of_key(uint32_t nkey, uint32_t base)
{
    const uint32_t s = nkey >> 2;
    return s <= base ? 0u : min(s - base, 511u);
}
// every norm whose key falls in shell s lies in [shell_rlo, shell_rhi)
__device__ __forceinline__ float shell_rlo(uint32_t s, uint32_t base)
{
    return s == 0 ? 0.0f : __uint_as_float(((s + base) << 2) << 16);
}
__device__ __forceinline__ float shell_rhi(uint32_t s, uint32_t base)
{
    return s >= 511u ? INFINITY : __uint_as_float(((s + base + 1) << 2) << 16);
}
__device__ __forceinline__ uint32_t cos_bucket(float t)
{
    const int q = int((t + 1.0f) * 64.0f);
    return uint32_t(max(0, min(q, 127)));
}
// norm, projection on e = (1,..,1)/sqrt(d), and the ordering key of one row
template <int D>
__device__ __forceinline__ uint32_t ordering_key(const float (&x)[D], float norm, uint32_t base, float& proj)
{
    float sum = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) sum += x[j];
    proj = sum * (D == 4 ? 0.5f : (D == 16 ? 0.25f : 0.35355339059327373f));
    const float t = norm > 0.0f ? proj / norm : 0.0f;
    return (shell_of_key(norm_key(norm), base) << 7) | cos_bucket(t);
}

// The ordering keys [klo, khi] of shell `sh` that a candidate with e.c in [plo, phi] can have: its cosine e.c/||c|| with
// ||c|| in [rlo, rhi); 1e-4 of slack for the two divisions (the centroid's own, when its key was made, and the one
// here: 1e-7 each). klo > khi if there is none.
__device__ __forceinline__ void shell_cosine_run(uint32_t sh, uint32_t base, float plo, float phi, uint32_t& klo, uint32_t& khi)
{
    const float rlo = shell_rlo(sh, base), rhi = shell_rhi(sh, base);
    float tlo, thi;
    if (plo >= 0.0f) tlo = rhi < INFINITY ? plo / rhi : 0.0f; else tlo = rlo > 0.0f ? plo / rlo : -1.0f;
    if (phi >= 0.0f) thi = rlo > 0.0f ? phi / rlo : 1.0f; else thi = rhi < INFINITY ? phi / rhi : 0.0f;
    klo = (sh << 7) | cos_bucket(__builtin_fmaxf(tlo - 1e-4f, -1.0f));
    khi = (sh << 7) | cos_bucket(__builtin_fminf(thi + 1e-4f, 1.0f));
}

}  // namespace cc
