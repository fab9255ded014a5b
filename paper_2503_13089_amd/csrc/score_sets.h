// Few vectors against a codebook or windows of it on the fp16 matrix cores (see assign_mfma_f16.hip for the scheme and its error
// analysis): a workgroup takes 32 VT vectors, its W waves take turns at the tiles and load operands straight from the packed codebook. Shared by
// the far vectors of a fit by cells (cells.hip) and the E-steps of calls with too few vectors to fill the chip with 512 to a workgroup
// (assign_mfma_f16.hip).
#pragma once
#include "common.h"
#include "f16_scores.h"

namespace cc {

constexpr int kSetGroup = 2;   // tiles of 32 centroids that are scored together: the tracking group

// Between what lanes of one wave write to LDS and what other lanes of it read: its LDS accesses are served in order, so there is
// nothing to wait for, but the compiler has to keep them in order.
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// One running best / second best: `w` into (best, second)
__device__ __forceinline__ void take_score(float& best, float& second, float w)
{
    second = __builtin_amdgcn_fmed3f(best, second, w);
    asm("v_min_f32 %0, %1, %2" : "=v"(best) : "v"(best), "v"(w));
}

// win_tile vectors (a multiple of those of a workgroup) share a window, those of two begin win_stride entries apart.
// finish(i, mine, x, k, distance, safe), by whole waves: the decision for vector i, in the lane with `mine` set; the vectors of lanes n are
// neighbours from a multiple of 32 on. LDS: x_best, x_second, x_grp of W * VT * 64, lds_norms (16-byte aligned) of W * 32 * kSetGroup entries.
template <int D, int VT, int W, bool WINDOWED, typename Finish>
__device__ __forceinline__ void score_sets(const float* __restrict__ X, const float* __restrict__ rows, const uint32_t* __restrict__ cperm,
                                           uint32_t N, uint32_t K, const char* __restrict__ packed, uint32_t ntiles, const uint2* __restrict__ windows,
                                           uint32_t win_tile, uint32_t win_stride,
                                           uint32_t cmax_bits, float* x_best, float* x_second, uint32_t* x_grp, float* lds_norms, Finish finish)
{
    using S = F16Shape<D>;
    constexpr int GT = kSetGroup, KM = S::KM;
    constexpr uint32_t kSet = 32 * VT;
    static_assert(GT == 2, "a lane of each half to a tile's norms");
    static_assert(kWinSlots <= 64 && kFarWinSlots <= 64, "a lane to a run");
    static_assert((!WINDOWED || kWinTile % kSet == 0) && VT <= W, "a set has one window, a wave finishes a tile");
    const int lane = threadIdx.x & 63, h = lane >> 5, n = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    float* const norms = lds_norms + wave * (32 * GT);
    const uint32_t sets = (N + kSet - 1) / kSet;
    for (uint32_t set = blockIdx.x; set < sets; set += gridDim.x) {
        const uint32_t i0 = (sets - 1 - set) * kSet;  // the widest windows first
        f16x8 b[VT][KM];
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) {
            float x[D];
            load_row<D>(X + size_t(min(i0 + vt * 32 + n, N - 1)) * D, x);
            vector_operand<D>(x, h, b[vt]);
        }
        float best_of[VT], second_of[VT];
        uint32_t grp_of[VT];
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) {
            best_of[vt] = second_of[vt] = INFINITY;
            grp_of[vt] = 0;
        }
        // The window's groups of GT tiles in one sequence (runs share none), the waves taking every W-th: lane r holds where
        // run r ends in it and what turns a place in the sequence into a group. Tiles of a group beside the run are scored with it.
        uint32_t run_end = 0, shift = 0, total = (ntiles + GT - 1) / GT, r = 0;
        if constexpr (WINDOWED) {
            const uint2* wl = windows + size_t(i0 / win_tile) * win_stride;
            uint32_t g0 = 0, count = 0;
            if (uint32_t(lane) < wl[0].x) {
                const uint2 run = wl[1 + lane];
                g0 = run.x / GT;
                count = (run.y + GT - 1) / GT - g0;
            }
            run_end = count;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t before = uint32_t(__shfl_up(int(run_end), off, 64));
                if (lane >= off) run_end += before;
            }
            shift = g0 - (run_end - count);
            total = uint32_t(__builtin_amdgcn_readlane(int(run_end), 63));
        }
        auto group_at = [&](uint32_t at) {   // ascending places; past the end the last one
            const uint32_t f = min(at, total - 1);
            if constexpr (!WINDOWED) return f;
            while (f >= uint32_t(__builtin_amdgcn_readlane(int(run_end), int(r)))) ++r;
            return f + uint32_t(__builtin_amdgcn_readlane(int(shift), int(r)));
        };
        float norm = 0.0f;   // d = 8 and 16: lane (u, row) loads the norm of a row of tile u, a group ahead
        auto load = [&](uint32_t group, f16x8 (&to)[GT][KM]) {   // a scalar base and one offset per lane
            const char* tiles = packed + size_t(group) * (GT * S::kTileBytes);
#pragma unroll
            for (int u = 0; u < GT; ++u)
#pragma unroll
                for (int mi = 0; mi < KM; ++mi)
                    to[u][mi] = *reinterpret_cast<const f16x8*>(tiles + ((uint32_t(lane) * KM + mi) * 16 + u * S::kTileBytes));
            if constexpr (!S::kNormInK) norm = *reinterpret_cast<const float*>(tiles + (uint32_t(h) * S::kTileBytes + 1024 * KM + 4 * n));
        };
        f16x8 from[GT][KM], to[GT][KM];
        uint32_t at = uint32_t(wave), g = 0;
        if (at < total) {
            g = group_at(at);
            load(g, from);
        }
        for (; at < total; at += W) {
            f32x16 cn[S::kNormInK ? 1 : GT];
            if constexpr (S::kNormInK) {
#pragma unroll
                for (int q = 0; q < 16; ++q) cn[0][q] = 0.0f;
            } else {   // rows 16 h .. 16 h + 15 of every tile
                wave_order();   // what the group before had there has been read
                norms[lane] = norm;
                wave_order();
#pragma unroll
                for (int u = 0; u < GT; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 v = reinterpret_cast<const float4*>(norms + 32 * u + 16 * h)[q];
                        cn[u][4 * q] = v.x; cn[u][4 * q + 1] = v.y; cn[u][4 * q + 2] = v.z; cn[u][4 * q + 3] = v.w;
                    }
            }
            const uint32_t next = group_at(at + W);
            load(next, to);
            __builtin_amdgcn_sched_barrier(0);   // else the compiler would put the loads behind the products
            // the products of one tile run while the minima of the one before it are taken
            float m[VT];
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) m[vt] = INFINITY;
            f32x16 acc[2];
            auto product = [&](int i) {
                acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(from[i / VT][0], b[i % VT][0], cn[S::kNormInK ? 0 : i / VT], 0, 0, 0);
#pragma unroll
                for (int mi = 1; mi < KM; ++mi) acc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(from[i / VT][mi], b[i % VT][mi], acc[i & 1], 0, 0, 0);
            };
            product(0);
#pragma unroll
            for (int i = 0; i < GT * VT; ++i) {
                if (i + 1 < GT * VT) product(i + 1);
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    m[i % VT] = __builtin_fminf(__builtin_fminf(m[i % VT], acc[i & 1][2 * q]), acc[i & 1][2 * q + 1]);
            }
            __builtin_amdgcn_sched_group_barrier(8, KM, 0);
#pragma unroll
            for (int i = 0; i < GT * VT; ++i) {   // a product, the eight instructions of the minimum before it, the next product ...
                __builtin_amdgcn_sched_group_barrier(8, KM, 0);
                __builtin_amdgcn_sched_group_barrier(2, 8, 0);
            }
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) {
                grp_of[vt] = m[vt] < best_of[vt] ? g : grp_of[vt];
                take_score(best_of[vt], second_of[vt], m[vt]);
            }
            g = next;
#pragma unroll
            for (int u = 0; u < GT; ++u)
#pragma unroll
                for (int mi = 0; mi < KM; ++mi) from[u][mi] = to[u][mi];
        }
        auto exchange = [&](int w, int vt) { return (w * VT + vt) * 64 + lane; };
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) {
            x_best[exchange(wave, vt)] = best_of[vt];
            x_second[exchange(wave, vt)] = second_of[vt];
            x_grp[exchange(wave, vt)] = grp_of[vt];
        }
        __syncthreads();
        if (wave < VT) {  // wave w finishes tile w: index recovery and guard band as in assign_mfma_f16.hip
            float best = INFINITY, second = INFINITY;
            uint32_t grp = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float ob = x_best[exchange(w, wave)], os = x_second[exchange(w, wave)];
                if (ob < best) grp = x_grp[exchange(w, wave)];
                second = __builtin_fminf(__builtin_fminf(second, os), __builtin_fmaxf(best, ob));
                best = __builtin_fminf(best, ob);
            }
            const uint32_t i_raw = i0 + wave * 32 + n, i = min(i_raw, N - 1);
            float x[D];
            load_row<D>(X + size_t(i) * D, x);
            const float ob = __shfl_xor(best, 32, 64), os = __shfl_xor(second, 32, 64);
            const uint32_t og = uint32_t(__shfl_xor(int(grp), 32, 64));
            const bool mine = best < ob || (best == ob && h == 0);
            const float bstar = __builtin_fminf(best, ob);
            const float sstar = __builtin_fminf(__builtin_fminf(second, os), __builtin_fmaxf(best, ob));
            float bd;
            uint32_t bk;
            recover_group<D, GT, (D == 16 && VT <= 2 ? 2 : 4)>(x, rows, cperm, K, mine ? grp : og, mine ? h : 1 - h, h, h + 1, bd, bk);
            const float od = __shfl_xor(bd, 32, 64);
            const uint32_t ok = uint32_t(__shfl_xor(int(bk), 32, 64));
            const bool take = od < bd || (od == bd && ok < bk);
            const float dstar = take ? od : bd;
            const float sigma = __builtin_ldexpf(1.0f, centroid_scale_log2(cmax_bits, D));
            const bool safe = (sstar - bstar) > f16_guard_band<D>(x, dstar, sigma, sigma * __uint_as_float(cmax_bits));
            finish(i_raw, h == 0 && i_raw < N, x, take ? ok : bk, dstar, safe);
        }
        __syncthreads();  // the exchange buffers have been read
    }
}

}  // namespace cc
