// What the kernels that score on the fp16 matrix cores share: the operand layout of the packed codebook and of the
// vectors, and the guard band of a decision (see assign_mfma_f16.hip for the scheme and its error analysis).
#pragma once
#include "common.h"

namespace cc {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));

constexpr float kUnit = 5.9604644775390625e-08f;  // 2^-24
constexpr float kGuardSafety = 1.5f;
constexpr int kAccumUlps = 8;

template <int D>
struct F16Shape {
    static constexpr int kParts = (D == 4) ? 3 : 2;         // fp16 parts per centroid component
    static constexpr bool kNormInK = (D == 4);              // ||c||^2 rides in spare k slots
    static constexpr int kSlots = kParts * D + (kNormInK ? 3 : 0);
    static constexpr int KM = (kSlots + 15) / 16;           // MFMAs per tile
    static constexpr int kTileBytes = 64 * KM * 16 + (kNormInK ? 0 : 128);
};

// The three fp16 parts of a scaled fp32 value.
__device__ __forceinline__ void split3(float v, _Float16 (&h)[3])
{
    h[0] = _Float16(v);
    const float r1 = v - float(h[0]);  // exact
    h[1] = _Float16(r1);
    const float r2 = r1 - float(h[1]);  // exact
    h[2] = _Float16(r2);
}

// sigma*||c||^2 as g0*2^8 + g1*2^-3 + g2*2^-14
__device__ __forceinline__ void split_norm(float v, _Float16 (&g)[3])
{
    g[0] = _Float16(v * 0.00390625f);
    const float r1 = v - float(g[0]) * 256.0f;
    g[1] = _Float16(r1 * 8.0f);
    const float r2 = r1 - float(g[1]) * 0.125f;
    g[2] = _Float16(r2 * 16384.0f);
}

// One centroid at position `pos` of the packed codebook: its scaled components in parts, sigma ||c||^2 (past K: parts 0, norm +inf, which
// never wins). Per 32-centroid tile [64 lanes][KM] x 8 fp16 A-operand values (lane (m, h) holds k slots 16 mi + 8 h .. + 7 of MFMA mi for
// output row m), then, where the norm has no slot, the 32 scaled norms. Output row m of a tile is centroid 32 tile + 16 ((m / 4) % 2) + (m % 4) +
// 4 (m / 8), so that lane half h, accumulator register r is centroid 32 tile + 16 h + r.
template <int D>
__device__ __forceinline__ void put_f16_operand(char* packed, uint32_t pos, const _Float16 (&parts)[D][3], const _Float16 (&g)[3], float scaled_norm)
{
    using S = F16Shape<D>;
    const uint32_t q = pos & 31u, m = 4 * (q >> 4) + (q & 3u) + 8 * ((q & 15u) >> 2);
    char* tile = packed + size_t(pos >> 5) * S::kTileBytes;
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int mi = 0; mi < S::KM; ++mi) {
            f16x8 v;
#pragma unroll
            for (int q8 = 0; q8 < 8; ++q8) {
                const int slot = 16 * mi + 8 * half + q8;
                v[q8] = slot < S::kParts * D ? parts[slot % D][slot / D]
                                             : (S::kNormInK && slot < S::kParts * D + 3 ? g[slot - S::kParts * D] : _Float16(0.0f));
            }
            *reinterpret_cast<f16x8*>(tile + (size_t(half * 32 + m) * S::KM + mi) * 16) = v;
        }
    if (!S::kNormInK) *reinterpret_cast<float*>(tile + 64 * S::KM * 16 + 4 * q) = scaled_norm;
}

// B operands of one vector: lane (n, h) supplies k slots 16 mi + 8 h .. + 7: -2 x_j for the product slots, the fixed
// multipliers for the norm slots, 0 for unused ones.
template <int D>
__device__ __forceinline__ void vector_operand(const float (&x)[D], int h, f16x8 (&b)[F16Shape<D>::KM])
{
    using S = F16Shape<D>;
#pragma unroll
    for (int mi = 0; mi < S::KM; ++mi) {
#pragma unroll
        for (int q8 = 0; q8 < 8; ++q8) {
            _Float16 v[2];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int q = 16 * mi + 8 * half + q8;
                v[half] = _Float16(0.0f);
                constexpr int PD = S::kParts * D;
                if (q < PD) v[half] = _Float16(-2.0f * x[q % D]);
                else if (S::kNormInK && q == PD) v[half] = _Float16(256.0f);
                else if (S::kNormInK && q == PD + 1) v[half] = _Float16(0.125f);
                else if (S::kNormInK && q == PD + 2) v[half] = _Float16(6.103515625e-05f);  // 2^-14
            }
            b[mi][q8] = h ? v[1] : v[0];
        }
    }
}

// How far (in sigma-scaled score units) another group's best score must be above the winner's for the decision to be
// safe; dstar: the winner's direct-form distance. P parts per component, the norm in k slots or as the accumulator's start
// value; ULPS: the bound on the instruction's accumulation in units of 2^-24 of the sum of its terms.
template <int D, int P = F16Shape<D>::kParts, bool NORM_IN_K = F16Shape<D>::kNormInK, int ULPS = kAccumUlps>
__device__ __forceinline__ float f16_guard_band(const float (&x)[D], float dstar, float sigma, float sigma_cmax)
{
    float xn = 0.0f, x1 = 0.0f, xlost = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        xn = __builtin_fmaf(x[j], x[j], xn);
        x1 += __builtin_fabsf(x[j]);
        // what the fp16 operand -2 x_j lost: nonzero only below the fp16 normal range, at most 2^-25, exact in fp32
        const float t = -2.0f * x[j];
        xlost += __builtin_fabsf(t - float(_Float16(t)));
    }
    // accumulation rounding of winner + true nearest (||c||^2 <= 2||x||^2 + 2D for both); what fp16
    // subnormal factors add to the sum of |terms| (with a = 2^-14: each of the P*D product slots at most
    // a |2 x_j| + a |part| + a^2, the parts of one centroid summing to <= 1.002 sigma ||c||_1, and the
    // norm slots at most 2^-6 + 2^-17 + 2^-28); then the split residuals: 2^-25 per component against
    // |2 x_j|, twice, and the norm residual
    constexpr float kA = 6.103515625e-05f;  // 2^-14
    const float inflation = 2.0f * float(P) * kA * x1 + 1.002f * kA * sigma * __builtin_sqrtf(float(D) * (2.0f * xn + 2.0f * dstar)) +
                            float(P * D) * kA * kA + (NORM_IN_K ? 0.015634f : 0.0f);
    // two parts leave a relative residual: |c sigma - h1 - h2| <= 2^-22 |c sigma| per component (each part is a
    // rounding to 11 bits), against |2 x_j|: at most 2^-21 sigma ||x|| ||c|| per score, for the best and for its
    // competitor (three parts leave 2^-33, which the accumulation term dwarfs)
    const float split_rel = P == 2 ? 9.5367431640625e-07f * sigma * __builtin_sqrtf(xn * (2.0f * xn + 2.0f * dstar)) : 0.0f;
    // a lost part of -2 x_j moves every score of this vector by at most |it| * sigma * max|c| * 1.002 (the
    // parts of a centroid component), the best and its competitor in opposite directions at worst
    const float operand_loss = 2.0f * 1.002f * sigma_cmax * xlost;
    return kGuardSafety * 2.0f * float(ULPS) * kUnit * (sigma * (5.0f * xn + 4.0f * dstar) + inflation) +
                        kGuardSafety * (2.0f * kUnit * x1 + 1e-11f + operand_loss + split_rel) + 1e-36f;
}

}  // namespace cc
