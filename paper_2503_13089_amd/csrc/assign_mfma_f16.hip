// E-step on the fp16 matrix cores with fp32-grade scores, for fp16-representable inputs
// (Section 3.1: w_i goes to the centroid minimising ||w_i - c||^2; the paper's tensors are 16-bit).
//
// Same scheme as the fp32 MFMA kernel (scores s = ||c||^2 - 2 x.c, lane = one vector, running
// min / second-min per centroid group, direct-form index recovery, guard band + refinement), but
// the products run on v_mfma_f32_32x32x16_f16, whose rate is 16x that of the fp32 MFMA and which,
// unlike the fp32 MFMA, leaves the vector ALUs free for the min-reduction while it runs.
//
// Exactness: every input x of the fp16 normal range is an fp16 number (checked on the device; otherwise the
// fp32 kernel runs); smaller ones may lose up to 2^-25 in the operand, which the guard band accounts for.
// Each fp32 centroid component, scaled by a power of two sigma so that it fits the fp16 range, is
// split into fp16 parts c*sigma = h1 + h2 (+ h3), each part the fp16 rounding of what is left. An
// fp16 x fp16 product has at most 22 significant bits, so every product h_p * (-2 x) is exact in the
// fp32 accumulator: the only rounding is in the accumulation. d = 4 takes three parts (residual below
// 2^-33 |c*sigma| or the fp16 subnormal step 2^-24): the k = 16 slots of one MFMA hold the 12 products
// and three more slots that add sigma * ||c||^2, itself split into three fp16 parts against the fixed
// multipliers 2^8, 2^-3, 2^-14. d = 8 and 16 take two parts (residual 2^-22 |c*sigma|, which the guard
// band carries as a term of its own - about a quarter on top of the accumulation term): 16 and 32
// slots, one and two MFMAs per tile instead of the two and three that three parts would need, with
// sigma * ||c||^2 as the fp32 C operand.
//
// Guard band: measured on gfx950, the accumulated result differs from the exact sum by at most
// ~3 * 2^-24 * (sum of |terms|), where the matrix core aligns a product by the exponent FIELDS of its
// factors: an fp16 subnormal factor counts as 2^-14 however small it is, so a nonzero product a * b
// weighs max(|a|, 2^-14) * max(|b|, 2^-14) in that sum (a subnormal norm part against the 2^8
// multiplier costs an absolute 2^-6 * 2^-24, for instance). The band assumes kAccumUlps = 8 times
// 2^-24 times that inflated sum, plus the split residual. A vector whose best and second-best group
// scores are closer than the band is re-decided in direct form over all K (refine.hip), exactly as
// for the fp32 kernel.
#include <algorithm>

#include "common.h"
#include "f16_scores.h"
#include "score_sets.h"

namespace cc {

constexpr int kThreads = 256;
// WINDOWED = false: the whole packed codebook in stages of ST tiles. WINDOWED = true: the runs of the
// workgroup's window list (stages of kStageTiles tiles, tiles outside a run skipped).
template <int D, int VT, int ST, int GT, bool WINDOWED>
__global__ __launch_bounds__(kThreads, 2) void assign_mfma_f16_kernel(
    const float* __restrict__ X, uint32_t N, const float* __restrict__ C, uint32_t K, const char* __restrict__ packed,
    uint32_t ntiles, uint32_t* __restrict__ idx, float* __restrict__ dmin, WsHeader* hdr,
    uint32_t* __restrict__ refine_list, uint32_t refine_cap, int gate,
    long long* sums, uint32_t* counts, const uint2* __restrict__ windows, const uint32_t* __restrict__ cperm, int hint_only,
    uint32_t* __restrict__ prev_out, uint32_t* __restrict__ changed)
{
    using S = F16Shape<D>;
    constexpr int KM = S::KM;
    constexpr int TILE_F4 = S::kTileBytes / 16;
    constexpr int STAGE_F4 = ST * TILE_F4;
    constexpr int NPF = (STAGE_F4 + kThreads - 1) / kThreads;
    static_assert(ST % GT == 0, "a tracking group must not straddle LDS stages");
    static_assert(!WINDOWED || ST == int(kStageTiles), "window runs never share a stage of kStageTiles tiles");
    if (!gate_open(hdr, gate)) return;  // uniform over the grid
    __shared__ float4 lds[2][STAGE_F4];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = lane >> 5, n = lane & 31;
    // A windowed launch starts with the last tiles of the norm order: the outer shells have the widest windows, and the
    // workgroups that take longest should not be the ones that start last (cfg3: 2.3 % of the fit; taking tiles from
    // both ends in turn instead costs 5 %).
    const uint32_t wg = WINDOWED ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    const uint32_t vbase = (wg * 4 + wave) * (32 * VT);

    // B operands: lane (n, h) supplies k slots 16*mi + 8h .. +7 of vector n: -2 x_j for the product
    // slots, the fixed multipliers for the norm slots, 0 for unused slots
    f16x8 b[VT][KM];
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
        const uint32_t i = min(vbase + vt * 32 + n, N - 1);
        float x[D];
        load_row<D>(X + size_t(i) * D, x);
        vector_operand<D>(x, h, b[vt]);
    }
    float best[VT], second[VT];
    uint32_t grp[VT];
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
        best[vt] = INFINITY;
        second[vt] = INFINITY;
        grp[vt] = 0;
    }

    const float4* P4 = reinterpret_cast<const float4*>(packed);
    // Stages to score: the whole packed codebook, or the runs of this workgroup's 512-vector tile.
    const uint2* wl = WINDOWED ? windows + size_t((wg * (4 * 32 * VT)) / kWinTile) * kWinStride : nullptr;
    const uint32_t nruns = WINDOWED ? wl[0].x : 1u;
    uint32_t run = 0;
    uint2 cur_run = WINDOWED ? wl[1] : make_uint2(0, ntiles);  // [first tile, end tile)
    uint32_t s = cur_run.x / ST;
    int cur = 0;
#pragma unroll
    for (int p = 0; p < NPF; ++p) {
        const uint32_t j = threadIdx.x + p * kThreads;
        if (NPF * kThreads == STAGE_F4 || j < STAGE_F4) lds[0][j] = P4[size_t(s) * STAGE_F4 + j];
    }
    __syncthreads();

    while (true) {
        // the stage after this one: next in the run, or the first of the next run, or none
        uint32_t sn = s + 1, run_n = run;
        uint2 next_run = cur_run;
        if (sn * ST >= cur_run.y) {
            run_n = run + 1;
            if (WINDOWED && run_n < nruns) {
                next_run = wl[1 + run_n];
                sn = next_run.x / ST;
            }
        }
        // tiles of this stage that belong to the run
        const uint32_t g_lo = cur_run.x > s * ST ? cur_run.x - s * ST : 0u;
        const uint32_t g_hi = min(cur_run.y - s * ST, uint32_t(ST));
        const bool has_next = run_n < nruns;
        if (!has_next) sn = s;  // the last iteration re-reads its own stage; the copy is never used

        float4 pf[NPF];
#pragma unroll
        for (int p = 0; p < NPF; ++p) {
            const uint32_t j = min(threadIdx.x + p * kThreads, uint32_t(STAGE_F4 - 1));
            pf[p] = P4[size_t(sn) * STAGE_F4 + j];
        }

        const char* L = reinterpret_cast<const char*>(lds[cur]);
#pragma unroll 1
        for (uint32_t tt = 0; tt < ST; tt += GT) {
            float m[VT];
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) m[vt] = INFINITY;
            if constexpr (S::kNormInK) {
                static_assert(KM == 1, "d = 4");
                f32x16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    if (WINDOWED && (tt + g < g_lo || tt + g >= g_hi)) continue;  // wave-uniform: tile outside the run
                    const f16x8 a = *reinterpret_cast<const f16x8*>(L + (tt + g) * S::kTileBytes + lane * 16);
#pragma unroll
                    for (int vt = 0; vt < VT; ++vt) {
                        const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b[vt][0], zero, 0, 0, 0);
#pragma unroll
                        for (int q = 0; q < 8; ++q) m[vt] = __builtin_fminf(__builtin_fminf(m[vt], acc[2 * q]), acc[2 * q + 1]);
                    }
                }
            } else {
                // Inside a run the minima of one product are taken while the next one runs: fits of 16 numbers, 5 iterations of 2.8 M vectors,
                // K = 65536, 62.0 to 63.4 -> 59.7 to 61.2 ms (left to the compiler's order 70), layer_compress of 2168 x 549, g = 7, K = 42818 9.0 -> 7.8.
                // At d = 4, two tiles to a group, that is 2 % slower.
                auto operands = [&](int g, f16x8 (&a)[KM], f32x16& cn) {
                    const char* T = L + (tt + g) * S::kTileBytes;
#pragma unroll
                    for (int mi = 0; mi < KM; ++mi) a[mi] = *reinterpret_cast<const f16x8*>(T + (lane * KM + mi) * 16);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 t = *reinterpret_cast<const float4*>(T + 64 * KM * 16 + (16 * h + 4 * q) * 4);
                        cn[4 * q + 0] = t.x; cn[4 * q + 1] = t.y; cn[4 * q + 2] = t.z; cn[4 * q + 3] = t.w;
                    }
                };
                auto product = [&](const f16x8 (&a)[KM], const f32x16& cn, int vt) {
                    f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[vt][0], cn, 0, 0, 0);
#pragma unroll
                    for (int mi = 1; mi < KM; ++mi) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[mi], b[vt][mi], acc, 0, 0, 0);
                    return acc;
                };
                auto minimum = [&](const f32x16& acc, int vt) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) m[vt] = __builtin_fminf(__builtin_fminf(m[vt], acc[2 * q]), acc[2 * q + 1]);
                };
                if (!WINDOWED || (tt >= g_lo && tt + GT <= g_hi)) {
                    f16x8 a[GT][KM];
                    f32x16 cn[GT], acc[2];
#pragma unroll
                    for (int g = 0; g < GT; ++g) operands(g, a[g], cn[g]);
                    acc[0] = product(a[0], cn[0], 0);
#pragma unroll
                    for (int i = 0; i < GT * VT; ++i) {
                        if (i + 1 < GT * VT) acc[(i + 1) & 1] = product(a[(i + 1) / VT], cn[(i + 1) / VT], (i + 1) % VT);
                        minimum(acc[i & 1], i % VT);
                    }
                    __builtin_amdgcn_sched_group_barrier(8, KM, 0);
#pragma unroll
                    for (int i = 0; i < GT * VT; ++i) {   // a product, the eight instructions of the minimum before it, the next product ...
                        __builtin_amdgcn_sched_group_barrier(8, KM, 0);
                        __builtin_amdgcn_sched_group_barrier(2, 8, 0);
                    }
                } else {
#pragma unroll
                    for (int g = 0; g < GT; ++g) {
                        if (WINDOWED && (tt + g < g_lo || tt + g >= g_hi)) continue;  // wave-uniform: tile outside the run
                        f16x8 a[KM];
                        f32x16 cn;
                        operands(g, a, cn);
#pragma unroll
                        for (int vt = 0; vt < VT; ++vt) minimum(product(a, cn, vt), vt);
                    }
                }
            }
            const uint32_t gid = (s * ST + tt) / GT;
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) {
                second[vt] = __builtin_amdgcn_fmed3f(best[vt], second[vt], m[vt]);
                grp[vt] = m[vt] < best[vt] ? gid : grp[vt];
                // plain v_min_f32: both operands come from v_min3/v_med3 results, which are already canonical,
                // so the canonicalising v_max the compiler would put in front of fminf is not needed
                asm("v_min_f32 %0, %1, %2" : "=v"(best[vt]) : "v"(best[vt]), "v"(m[vt]));
            }
        }

#pragma unroll
        for (int p = 0; p < NPF; ++p) {
            const uint32_t j = threadIdx.x + p * kThreads;
            if (NPF * kThreads == STAGE_F4 || j < STAGE_F4) lds[cur ^ 1][j] = pf[p];
        }
        __syncthreads();
        if (!has_next) break;
        s = sn;
        run = run_n;
        cur_run = next_run;
        cur ^= 1;
    }

    // ---- epilogue: index recovery in direct form, merge of the two half-waves, guard-band test.
    // Scores are in sigma-scaled units; the band is scaled to match.
    // read once: the header's cache line is the target of the refine-list atomics below, and a reload per vector
    // (which the compiler would emit, since those atomics may alias it) costs a trip to memory each time
    const uint32_t cmax_bits = hdr->cmax_bits;
    const float sigma = __builtin_ldexpf(1.0f, centroid_scale_log2(cmax_bits, D));
    const float sigma_cmax = sigma * __uint_as_float(cmax_bits);
    const int sum_exp = sums != nullptr ? fixed_point_exp(hdr->absmax_bits, N) : 0;
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
        const uint32_t i_raw = vbase + vt * 32 + n;
        const uint32_t i = min(i_raw, N - 1);
        float x[D];
        load_row<D>(X + size_t(i) * D, x);
        // The overall best group sits in one of the two lanes that share this vector; both lanes split its
        // tiles. The other lane's best group, like every other group, only matters through `second`.
        static_assert(GT % 2 == 0, "the two lanes of a vector split the tiles of the winning group");
        const float ob = __shfl_xor(best[vt], 32, 64);
        const float os = __shfl_xor(second[vt], 32, 64);
        const uint32_t og = uint32_t(__shfl_xor(int(grp[vt]), 32, 64));
        const bool mine = best[vt] < ob || (best[vt] == ob && h == 0);
        const int wh = mine ? h : 1 - h;
        const uint32_t wgrp = mine ? grp[vt] : og;
        const float bstar = __builtin_fminf(best[vt], ob);
        const float sstar = __builtin_fminf(__builtin_fminf(second[vt], os), __builtin_fmaxf(best[vt], ob));
        float bd;
        uint32_t bk;
        recover_group<D, GT, (D == 16 && WINDOWED ? 2 : 4)>(x, C, cperm, K, wgrp, wh, h * (GT / 2), (h + 1) * (GT / 2), bd, bk);
        const float od = __shfl_xor(bd, 32, 64);
        const uint32_t ok = uint32_t(__shfl_xor(int(bk), 32, 64));
        const bool take = od < bd || (od == bd && ok < bk);
        const float dstar = take ? od : bd;
        const uint32_t kstar = take ? ok : bk;
        if (hint_only) {  // bootstrap pass: the code is only an upper bound for the next pass's windows
            if (h == 0 && i_raw < N) idx[i] = kstar;
            continue;
        }
        const float delta = f16_guard_band<D>(x, dstar, sigma, sigma_cmax);
        const bool safe = (sstar - bstar) > delta;  // false for NaN as well
        bool moved = false;
        if (h == 0 && i_raw < N) {
            if (changed != nullptr) {
                // the code this vector had so far, kept wherever the M-step will have to look at it again: the
                // code differs, or the refinement may still change it
                const uint32_t old = idx[i];
                moved = old != kstar || !safe;
                if (moved) prev_out[i] = old;
            }
            idx[i] = kstar;
            dmin[i] = dstar;
            if (sums != nullptr) accumulate_vector<D>(x, kstar, sums, counts, sum_exp, +1);
            if (!safe) {
                const uint32_t pos = atomicAdd(&hdr->refine_count, 1u);
                if (pos < refine_cap) refine_list[pos] = i;
            }
        }
        if (changed != nullptr) {  // uniform over the wave; lanes 0..31 hold the 32 consecutive vectors of this tile
            const unsigned long long m = __ballot(moved);
            if (lane == 0 && vbase + vt * 32 < N) changed[(vbase + vt * 32) >> 5] = uint32_t(m);
        }
    }
}

// The same for few vectors: a workgroup of 8 waves takes 32 VT of them, the waves take turns at the tiles.
constexpr int kFewWaves = 8;
template <int D, int VT, bool WINDOWED>
__global__ __launch_bounds__(64 * kFewWaves, VT <= 2 || (VT == 4 && D <= 8) ? 4 : 2) void assign_few_f16_kernel(
    const float* __restrict__ X, uint32_t N, const float* __restrict__ C, uint32_t K, const char* __restrict__ packed, uint32_t* __restrict__ idx,
    float* __restrict__ dmin, WsHeader* hdr, uint32_t* __restrict__ refine_list, uint32_t refine_cap, int gate, long long* sums, uint32_t* counts,
    const uint2* __restrict__ windows, const uint32_t* __restrict__ cperm, int hint_only, uint32_t* __restrict__ prev_out, uint32_t* __restrict__ changed)
{
    if (!gate_open(hdr, gate)) return;  // uniform over the grid
    constexpr int kLds = kFewWaves * VT * 64;
    __shared__ float x_best[kLds], x_second[kLds];
    __shared__ uint32_t x_grp[kLds];
    __shared__ __attribute__((aligned(16))) float norms[kFewWaves * 32 * kSetGroup];
    const int sum_exp = sums != nullptr ? fixed_point_exp(hdr->absmax_bits, N) : 0;
    score_sets<D, VT, kFewWaves, WINDOWED>(
        X, C, cperm, N, K, packed, (K + 31) / 32, windows, kWinTile, uint32_t(kWinStride), hdr->cmax_bits, x_best, x_second, x_grp, norms,
        [&](uint32_t i, bool mine, const float (&x)[D], uint32_t k, float distance, bool safe) {
            bool moved = false;
            if (mine) {
                if (hint_only) {
                    idx[i] = k;
                    return;
                }
                if (changed != nullptr) {   // as in assign_mfma_f16_kernel
                    const uint32_t old = idx[i];
                    moved = old != k || !safe;
                    if (moved) prev_out[i] = old;
                }
                idx[i] = k;
                dmin[i] = distance;
                if (sums != nullptr) accumulate_vector<D>(x, k, sums, counts, sum_exp, +1);
                if (!safe) {
                    const uint32_t pos = atomicAdd(&hdr->refine_count, 1u);
                    if (pos < refine_cap) refine_list[pos] = i;
                }
            }
            if (changed != nullptr && !hint_only) {   // lanes 0..31 hold 32 consecutive vectors
                const unsigned long long m = __ballot(moved);
                if ((threadIdx.x & 63) == 0 && i < N) changed[i >> 5] = uint32_t(m);
            }
        });
}

template <int D, int VT>
static hipError_t launch_few(const EStep& e, const Workspace& w, hipStream_t s)
{
    constexpr bool kWindowed = VT > 1;   // up to 8192 vectors: never
    const auto kernel = kWindowed && e.windows != nullptr ? assign_few_f16_kernel<D, VT, kWindowed> : assign_few_f16_kernel<D, VT, false>;
    ProfileScope scope(e.profile, kProfEstepF16, s);
    hipLaunchKernelGGL(kernel, dim3((e.N + 32 * VT - 1) / (32 * VT)), dim3(64 * kFewWaves), 0, s, e.X, e.N, e.rows, e.K,
                       static_cast<const char*>(e.packed), e.idx, w.dmin, w.hdr, w.refine_list, w.refine_cap, e.gate,
                       e.accumulate ? w.sums : nullptr, e.accumulate ? w.counts : nullptr, e.windows, e.row_ids, e.hint_only ? 1 : 0, e.prev_out, e.changed);
    return hipGetLastError();
}

// Up to how many vectors. A workgroup of the kernel above takes 512 through the codebook one stage of LDS after the other: 130000 vectors are one
// workgroup per compute unit, and 17000 are 33 in all. Fits of 10 iterations, us, that kernel / 64 to a workgroup (VT = 2) / 128 (4) / 256 (8), d, K, N:
// 4, 2600, 17000 696 / 341 / 420 / 419, 90000 807 / 593 / 571 / 642, 450000 1937 / 1668 / 1633 / 1724; 4, 20000 (windows), 200000 1594 / 1288 /
// 1120 / 1192, 450000 1750 / 2004 / 1622 / 1774, 800000 1999 / 2992 / 2306 / 2558; 8, 2600, 90000 1166 / 843 / 867 / 929, 800000 (windows) 3099 / 3364 / 2923 /
// 2941; 8, 20000, 200000 2872 / 2426 / 2212 / 2244, 1.6 M 12126 / 14428 / 12472 / 12509; 16, 2600, 17000 1422 / 581 / 640 / 666, 450000 5626 / 4786 / 5088 /
// 4935, 1.6 M (windows) 10241 / 9803 / 10797 / 8781; 16, 20000, 90000 4102 / 2387 / 2680 / 2447, 450000 8312 / 8190 / 9375 / 7359, 1.6 M 22308 / 25825 / 24050 /
// 21851. 32 to a workgroup: never better from 17000 on. (d = 16, 64 to a workgroup: with index recovery four rows at once; two take 522 instead of 609 at K = 2600,
// 17000 and 2309 instead of 2635 at K = 20000, 90000.) The lines between 64 and 256 to a workgroup at d = 16 with that, an E-step, 64 / 256: by windows K = 9811, 183000 277 / 266, K = 32070,
// 168000 512 / 476; K = 1787, 233000 122 / 113, K = 889, 353000 173 / 163. At d = 8, 128 to a workgroup, fewer waves per SIMD instead of 40 to 60 bytes of
// scratch a lane: K = 1137, 322000 129 instead of 108, K = 12705, 377000 350 instead of 300.
// Whole codebook, 2 iterations, us, that kernel / this one: 4, 4096, 1 M 656 / 664, 4.2 M 2074 / 2324; 8, 1000, 1 M 786 / 690, 8000, 4 M 4898 / 4698; 16, 8000, 2 M
// 5373 / 4258.
constexpr uint32_t few_most(int d, bool windowed)
{
    if (windowed) return d == 4 ? 1u << 19 : (d == 8 ? 1u << 20 : 1u << 21);
    return d == 4 ? 1u << 20 : (d == 8 ? 1u << 23 : 1u << 22);
}

template <int D, int VT, int ST>
static hipError_t launch_t(const EStep& e, const Workspace& w, hipStream_t s)
{
    // Tiles per tracking group: the epilogue re-evaluates the winning group in direct form, 8 * GT centroids per
    // lane. Over the whole codebook that is noise and a wide group keeps the hot loop lean; a windowed launch
    // scores only a few per cent of the codebook, the epilogue is then a third of the kernel, so groups are narrower.
    // From 32768 centroids on, 8-tile groups pay over the whole codebook (19.0 -> 18.75 ms at K = 65536, N = 11.3 M);
    // at K = 4096 the doubled epilogue would cost more than the loop saves.
    // At d = 8 and 16 a window still holds most of the codebook (the bands narrow like K^(-1/d)), the loop dominates again
    // and 4-tile groups pay (8192 x 28672, d = 8, K = 65536: 10 iterations in 531 instead of 545 ms).
    constexpr int GT = 4, GT_WIDE = ST >= 8 ? 8 : 4, GT_WINDOWED = D >= 8 ? 4 : 2;
    if (e.N <= few_most(D, e.windows != nullptr)) {
        if (e.N <= 8192u && e.windows == nullptr) return launch_few<D, 1>(e, w, s);
        if (e.N <= (D == 4 ? 49152u : (D == 8 ? 98304u : (e.windows != nullptr ? 131072u : 229376u)))) return launch_few<D, 2>(e, w, s);
        return launch_few<D, (D == 16 ? 8 : 4)>(e, w, s);
    }
    // a windowed workgroup scores the vectors of one window list (or a part of them)
    constexpr int VTW = VT * 128 > int(kWinTile) ? int(kWinTile) / 128 : VT;
    const uint32_t per_block = 4 * 32 * (e.windows != nullptr ? VTW : VT);
    const auto kernel = e.windows != nullptr ? assign_mfma_f16_kernel<D, VTW, int(kStageTiles), GT_WINDOWED, true>
                        : (e.K >= 32768  ? assign_mfma_f16_kernel<D, VT, ST, GT_WIDE, false>
                                         : assign_mfma_f16_kernel<D, VT, ST, GT, false>);
    {
        ProfileScope scope(e.profile, kProfEstepF16, s);
        hipLaunchKernelGGL(kernel, dim3((e.N + per_block - 1) / per_block), dim3(kThreads),
                           0, s, e.X, e.N, e.rows, e.K, static_cast<const char*>(e.packed), e.packed_tiles, e.idx, w.dmin, w.hdr,
                           w.refine_list, w.refine_cap, e.gate, e.accumulate ? w.sums : nullptr,
                           e.accumulate ? w.counts : nullptr, e.windows, e.row_ids, e.hint_only ? 1 : 0,
                           e.prev_out, e.changed);
    }
    return hipGetLastError();
}

hipError_t launch_assign_mfma_f16(const EStep& e, uint32_t d, const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: return launch_t<4, 4, 8>(e, w, s);
        case 8: return launch_t<8, 4, 4>(e, w, s);
        case 16: return launch_t<16, 4, 4>(e, w, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cc
