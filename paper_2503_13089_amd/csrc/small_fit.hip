// Lloyd iterations of small problems (Section 3.1) in two launches each: E-step on the vector ALUs with the codebook in
// LDS and the cluster sums taken in the same kernel, then one kernel that adds the workgroups' sums and divides.
//
// A matrix-core E-step of a small problem leaves most of the chip idle (N = 65536: 128 workgroups of 512 vectors), spends its time in the latency of its stages and
// of the index recovery, and an iteration with it is eleven launches of 2 us each, most of them gated off.
//
// A workgroup of 8 waves holds the codebook (K rows and their norms, fp32) and the accumulators (64-bit fixed-point sums and counts) in
// LDS. A lane scores V vectors, ||c||^2 / 2 - x.c (the rows are staged as -c: a vector of which
// twice is no finite number is scored, and added, as it is), four centroids at a time: d multiply-adds a pair, two minima, a compare, a select and best and second
// best for four of them. The best four are then compared in direct form; a vector whose second best comes within the guard band of the
// fp32 matrix cores, which do the same chain of multiply-adds (assign_mfma.hip), is decided in direct form over the codebook. Bound: multiply-adds issue in 2 clocks and
// the rest in 4, so a pair takes 2 d + 6 clocks, and LDS takes 8 to give all lanes 16 bytes: 2 d + 2 a centroid and wave, which four vectors per lane share. Direct form
// for every pair, a vector to a lane, took 4 d + 18 of the ALUs and as much of LDS as now four times the vectors.
// Its waves split the codebook S ways when there are too few vectors to give every lane some of its own; the S
// partial minima of a vector meet in LDS. The sums are
// the same integers as in the other formulations of the M-step, so the centroids are the same bits.
// Measured (fit of 10 iterations, N = 65536, K = 256, d = 4): 871 us on the matrix cores, 141 in direct form, 124 now; 4.2 M,
// K = 140 1708 (direct form) / 1006, 11 M, K = 250 7570 / 4151, 4 M of 8, K = 390 7211 / 3784, 1 M of 16, K = 250 2276 / 1530.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace cc {

namespace {

constexpr int kThreads = 512;
constexpr uint32_t kMaxBlocks = 512;      // two workgroups per compute unit
constexpr uint32_t kMaxLds = 76 * 1024;   // of rows, sums and counts

// What decides whether a problem is small: rows, sums [D][K] and counts [K]
size_t state_bytes(uint32_t d, uint32_t K) { return size_t(K) * (d * 4 + d * 8 + 4); }

constexpr uint32_t kFour = 4;             // centroids scored together
uint32_t whole_fours(uint32_t K) { return (K + kFour - 1) / kFour * kFour; }
// LDS of one workgroup: rows and norms of whole fours, sums and counts, and (S > 1) what the waves exchange of 64 V vectors each: best, second best and four
size_t lds_bytes(uint32_t d, uint32_t K, int V, int S, bool sums)
{
    return size_t(whole_fours(K)) * (d * 4 + 4) + (sums ? size_t(K) * (d * 8 + 4) : 0) + 16 + (S > 1 ? size_t(kThreads) * V * 12 : 0);
}

// bytes of one workgroup's partial sums: [D][K] int64, then [K] counts, rounded to whole 64-bit words
size_t partial_bytes(uint32_t d, uint32_t K) { return (size_t(K) * (d * 8 + 4) + 7) & ~size_t(7); }

template <int D>
__device__ __forceinline__ void load_opposite(const float* row, float (&c)[D])
{
    load_row<D>(row, c);
#pragma unroll
    for (int j = 0; j < D; ++j) c[j] = -c[j];
}

// The decision for a lane's vector x from the best four of its scores (`four`: the first of them), by whole waves; `on`: there is a vector. rows: the centroids' opposites.
// Where a score that matters could have overflowed, or missed the start value, the band has: a centroid no farther than bd has partial sums of at most
// 3 (||x||^2 + bd), and the sum that the band is made of is 18 times that bracket or more.
template <int D, bool SPLIT>
__device__ __forceinline__ void decide_small(const float (&x)[D], bool on, float best, float second, uint32_t four, const float* rows, uint32_t K,
                                             float& bd, uint32_t& bk)
{
    float d[kFour];
#pragma unroll
    for (uint32_t u = 0; u < kFour; ++u) {
        float c[D];
        load_opposite<D>(rows + size_t(four + u) * D, c);
        d[u] = direct_sqdist<D>(x, c);   // NaN past K
    }
    bd = __builtin_fminf(__builtin_fminf(__builtin_fminf(d[0], d[1]), d[2]), d[3]);
    bk = four;
#pragma unroll
    for (int u = int(kFour) - 1; u >= 0; --u) bk = d[u] == bd ? four + u : bk;
    float xn = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) xn = __builtin_fmaf(x[j], x[j], xn);
    const float band = 1.5f * 5.9604644775390625e-08f * (float(5 * D + 2) * xn + float(4 * D + 2) * bd) + 1e-36f;
    unsigned long long todo = __ballot(on && !(second - best > band));   // NaN too
    // One by one, or the whole wave at once where that takes less: among vectors of few different values, whose centroids have doubles or lie equally near, scores decide
    // little. Fits of 10 iterations of numbers of 2 bits, us, direct form for every pair / scores, one by one / now: (65536, 4, 256) 141 / 554 / 212, (4.2 M, 4, 140)
    // 1822 / 8272 / 3008, (4 M, 8, 390) 7105 / 7590 / 7288, (1 M, 16, 250) 2217 / 1772 / 1654. (Scores left out where most vectors of the iteration before were undecided:
    // 192, 2216, 7364, 2361, but 0.3 to 3 % more for everybody else.)
    // On its own a vector takes as much as so many centroids of a whole wave; more where few of the waves decide, and hide less of each other's waits.
    const uint32_t alone = SPLIT ? 16 + K / 24 : 8 + K / 48;
    if (__builtin_expect(uint32_t(__popcll(todo)) * alone > K, 0)) {
        todo = 0;
        bd = INFINITY;
        bk = 0;
#pragma unroll 32 / D
        for (uint32_t k = 0; k < K; ++k) {
            float c[D];
            load_opposite<D>(rows + size_t(k) * D, c);
            const float dist = direct_sqdist<D>(x, c);
            bk = dist < bd ? k : bk;
            bd = dist < bd ? dist : bd;
        }
    }
    const uint32_t lane = threadIdx.x & 63;
    while (todo != 0) {
        const int src = __ffsll(static_cast<long long>(todo)) - 1;
        todo &= todo - 1;
        float y[D];
#pragma unroll
        for (int j = 0; j < D; ++j) y[j] = __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(__float_as_uint(x[j])), src)));
        unsigned long long key = (0x7f800000ull << 32) | 0u;   // no distance is less than infinity: the first centroid
        for (uint32_t k = lane; k < K; k += 64) {
            float c[D];
            load_opposite<D>(rows + size_t(k) * D, c);
            const float dist = direct_sqdist<D>(y, c);
            const unsigned long long v = (static_cast<unsigned long long>(__float_as_uint(dist)) << 32) | k;
            key = dist < INFINITY && v < key ? v : key;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long v = __shfl_xor(key, off, 64);
            key = v < key ? v : key;
        }
        if (lane == uint32_t(src)) {
            bk = uint32_t(key & 0xffffffffull);
            bd = __uint_as_float(uint32_t(key >> 32));
        }
    }
}

template <int D, int V, uint32_t S, bool DIRECT, bool SUMS>
__global__ __launch_bounds__(kThreads, 4) void small_iter_kernel(const float* __restrict__ X, uint32_t N, const float* __restrict__ C,
                                                                 uint32_t K, uint32_t per_block, uint32_t* __restrict__ idx,
                                                                 float* __restrict__ dmin, char* __restrict__ partials,
                                                                 uint32_t partial_stride, WsHeader* __restrict__ hdr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t padded = (K + kFour - 1) / kFour * kFour;
    float* rows = reinterpret_cast<float*>(smem);                                                    // [padded][D], opposites unless DIRECT, NaN past K
    float* norms = rows + size_t(padded) * D;                                                        // [padded], halves
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(norms + padded);                // [D][K]
    uint32_t* counts = reinterpret_cast<uint32_t*>(sums + (SUMS ? size_t(K) * D : 0));               // [K]
    float2* met = reinterpret_cast<float2*>((reinterpret_cast<uintptr_t>(counts + (SUMS ? K : 0)) + 15) & ~uintptr_t(15));   // [kThreads V]
    uint32_t* met_four = reinterpret_cast<uint32_t*>(met + kThreads * V);                            // [kThreads V]
    const int e = SUMS ? fixed_point_exp(hdr->absmax_bits, N) : 0;
    const uint32_t lane = threadIdx.x & 63, wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    constexpr uint32_t VW = V * 64;                             // vectors of a wave
    const uint32_t VS = kThreads / S * V;                       // of one step
    const uint32_t slice = wave % S, part = wave / S;
    const uint32_t most = DIRECT ? K : padded, k_per = !DIRECT ? (padded / kFour + S - 1) / S * kFour : (K + S - 1) / S;
    const uint32_t k_lo = min(slice * k_per, most), k_hi = min(k_lo + k_per, most);
    const uint32_t lo = blockIdx.x * per_block, hi = min(lo + per_block, N);
    // S > 1: the first step's vectors are on their way while the codebook is staged, those a thread scores and the one it decides
    constexpr bool kEarly = S > 1 && D * V <= 16;   // else the registers are wanted while it is scored
    float x[V][D], y[D];
    auto load_vectors = [&](uint32_t v0) {
#pragma unroll
        for (int v = 0; v < V; ++v) load_row<D>(X + size_t(min(v0 + part * VW + v * 64 + lane, N - 1)) * D, x[v]);
        if constexpr (kEarly)
            if (threadIdx.x < VS) load_row<D>(X + size_t(min(v0 + threadIdx.x, N - 1)) * D, y);
    };
    for (uint32_t k = threadIdx.x, first = 1; first || k < padded; k += kThreads, first = 0) {
        float c[D];
#pragma unroll
        for (int j = 0; j < D; ++j) c[j] = __uint_as_float(0x7fc00000u);
        if (k < K) load_row<D>(C + size_t(k) * D, c);
        if (first) {   // requested after the codebook, whose wait then does not include them
            if constexpr (S > 1) load_vectors(lo);
            if constexpr (SUMS) {
                for (uint32_t t = threadIdx.x; t < K * D; t += kThreads) sums[t] = 0;
                for (uint32_t t = threadIdx.x; t < K; t += kThreads) counts[t] = 0;
            }
        }
        if (k >= padded) break;
        if constexpr (!DIRECT) {
            double norm = 0.0;
#pragma unroll
            for (int j = 0; j < D; ++j) {
                norm += double(c[j]) * double(c[j]);
                c[j] = -c[j];
            }
            norms[k] = float(0.5 * norm);
        }
#pragma unroll
        for (int q = 0; q < D / 4; ++q)
            reinterpret_cast<float4*>(rows)[k * (D / 4) + q] = make_float4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
    }
    auto finish = [&](const float (&x)[D], uint32_t i, float best, float second, uint32_t at) {
        float bd = best;
        uint32_t bk = at;
        if constexpr (!DIRECT) decide_small<D, (S > 1)>(x, i < hi, best, second, at, rows, K, bd, bk);
        if (i >= hi) return;
        if constexpr (SUMS) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const long long f = fixed_point_term(x[j], e);
                if (f != 0) atomicAdd(&sums[j * K + bk], static_cast<unsigned long long>(f));
            }
            atomicAdd(&counts[bk], 1u);
        }
        if (idx != nullptr) idx[i] = bk;
        if (dmin != nullptr) dmin[i] = bd;
    };
    __syncthreads();
    for (uint32_t v0 = lo; v0 < hi; v0 += VS) {
        if (S == 1 || v0 != lo) load_vectors(v0);
        if constexpr (DIRECT) {   // distances in direct form, nothing to decide
            float bd[V];
            uint32_t bk[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                bd[v] = INFINITY;
                bk[v] = min(k_lo, K - 1);
            }
#pragma unroll 4
            for (uint32_t k = k_lo; k < k_hi; ++k) {
                float c[D];
                load_row<D>(rows + size_t(k) * D, c);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const float dist = direct_sqdist<D>(x[v], c);
                    bk[v] = dist < bd[v] ? k : bk[v];
                    bd[v] = dist < bd[v] ? dist : bd[v];
                }
            }
            if constexpr (S == 1) {
#pragma unroll
                for (int v = 0; v < V; ++v) finish(x[v], v0 + part * VW + v * 64 + lane, bd[v], 0.0f, bk[v]);
                continue;
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < V; ++v) met[wave * VW + v * 64 + lane] = make_float2(bd[v], __uint_as_float(bk[v]));
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < VS; t += kThreads) {   // whole waves
                const uint32_t from = t / VW * S * VW + t % VW, i = v0 + t;
                if (!kEarly || t >= uint32_t(kThreads)) load_row<D>(X + size_t(min(i, N - 1)) * D, y);
                float2 b = met[from];
#pragma unroll
                for (uint32_t o = 1; o < S; ++o) {   // ascending slices: a strict "<" keeps the lowest index
                    const float2 other = met[from + o * VW];
                    b.y = other.x < b.x ? other.y : b.y;
                    b.x = other.x < b.x ? other.x : b.x;
                }
                finish(y, i, b.x, 0.0f, __float_as_uint(b.y));
            }
        } else {
        float best[V], second[V];
        uint32_t four[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            best[v] = second[v] = 3e38f;
            four[v] = min(k_lo, padded - kFour);
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): else the loop has a wait for each vector
        for (uint32_t k = k_lo; k < k_hi; k += kFour) {
            const float4 n4 = *reinterpret_cast<const float4*>(norms + k);
            const float n[kFour] = {n4.x, n4.y, n4.z, n4.w};
            float c[kFour][D];
#pragma unroll
            for (uint32_t u = 0; u < kFour; ++u) load_row<D>(rows + size_t(k + u) * D, c[u]);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                float s[kFour];
#pragma unroll
                for (uint32_t u = 0; u < kFour; ++u) {
                    s[u] = n[u];
#pragma unroll
                    for (int j = 0; j < D; ++j) s[u] = __builtin_fmaf(x[v][j], c[u][j], s[u]);
                }
                const float m = __builtin_fminf(__builtin_fminf(__builtin_fminf(s[0], s[1]), s[2]), s[3]);
                four[v] = m < best[v] ? k : four[v];
                second[v] = __builtin_amdgcn_fmed3f(best[v], second[v], m);
                best[v] = __builtin_fminf(best[v], m);
            }
        }
        if constexpr (S == 1) {
#pragma unroll
            for (int v = 0; v < V; ++v) finish(x[v], v0 + part * VW + v * 64 + lane, best[v], second[v], four[v]);
        } else {
        __syncthreads();   // the exchange buffers of the step before have been read
#pragma unroll
        for (int v = 0; v < V; ++v) {
            met[wave * VW + v * 64 + lane] = make_float2(best[v], second[v]);
            met_four[wave * VW + v * 64 + lane] = four[v];
        }
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < VS; t += kThreads) {   // whole waves
            const uint32_t from = t / VW * S * VW + t % VW, i = v0 + t;
            if (!kEarly || t >= uint32_t(kThreads)) load_row<D>(X + size_t(min(i, N - 1)) * D, y);
            float2 b = met[from];
            uint32_t f = met_four[from];
#pragma unroll
            for (uint32_t o = 1; o < S; ++o) {
                const float2 other = met[from + o * VW];
                f = other.x < b.x ? met_four[from + o * VW] : f;
                b.y = __builtin_fminf(__builtin_fminf(b.y, other.y), __builtin_fmaxf(b.x, other.x));
                b.x = __builtin_fminf(b.x, other.x);
            }
            finish(y, i, b.x, b.y, f);
        }
        }
        }
    }
    if constexpr (SUMS) {
        __syncthreads();
        unsigned long long* ps = reinterpret_cast<unsigned long long*>(partials + size_t(blockIdx.x) * partial_stride);
        uint32_t* pc = reinterpret_cast<uint32_t*>(ps + size_t(K) * D);
        for (uint32_t t = threadIdx.x; t < K * D; t += kThreads) ps[t] = sums[t];
        for (uint32_t t = threadIdx.x; t < K; t += kThreads) pc[t] = counts[t];
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
        hdr->assign_calls += 1;
    }
}

// Sixteen (component, cluster) entries per workgroup, sixteen threads each over the workgroups' partial sums.
constexpr int kFinThreads = 256;
template <int D>
__global__ __launch_bounds__(kFinThreads) void small_means_kernel(const char* __restrict__ partials, uint32_t partial_stride,
                                                                  uint32_t blocks, float* C, uint32_t* __restrict__ counts_out,
                                                                  uint32_t K, uint32_t N, WsHeader* hdr)
{
    __shared__ long long red_s[kFinThreads];
    __shared__ uint32_t red_n[kFinThreads];
    const uint32_t t = blockIdx.x * 16 + (threadIdx.x & 15), group = threadIdx.x >> 4;
    const bool live = t < K * D;
    const uint32_t k = live ? t % K : 0u, j = live ? t / K : 0u;   // clusters vary fastest, as in the partial sums
    long long s = 0;
    uint32_t n = 0;
    auto batch = [&](uint32_t first, auto most, auto all) {   // requests under way together; past the last block too: one at a time the rest took a trip to memory each
        constexpr uint32_t n_of = decltype(most)::value;
        unsigned long long part[n_of];
        uint32_t members[n_of];
#pragma unroll
        for (uint32_t u = 0; u < n_of; ++u) {
            const uint32_t b = first + group + 16 * u;
            const unsigned long long* ps = reinterpret_cast<const unsigned long long*>(partials + size_t(decltype(all)::value || b < blocks ? b : 0u) * partial_stride);
            part[u] = ps[j * K + k];
            members[u] = reinterpret_cast<const uint32_t*>(ps + size_t(K) * D)[k];
        }
#pragma unroll
        for (uint32_t u = 0; u < n_of; ++u) {
            const bool in = decltype(all)::value || first + group + 16 * u < blocks;
            s += in ? static_cast<long long>(part[u]) : 0;
            n += in ? members[u] : 0u;
        }
    };
    uint32_t first = 0;
    for (; first + 16 * 8 <= blocks; first += 16 * 8) batch(first, std::integral_constant<uint32_t, 8>{}, std::true_type{});
    const uint32_t rest = blocks - first;
    if (rest > 16 * 4) batch(first, std::integral_constant<uint32_t, 8>{}, std::false_type{});
    else if (rest > 16 * 2) batch(first, std::integral_constant<uint32_t, 4>{}, std::false_type{});
    else if (rest > 16) batch(first, std::integral_constant<uint32_t, 2>{}, std::false_type{});
    else if (rest > 0) batch(first, std::integral_constant<uint32_t, 1>{}, std::false_type{});
    red_s[threadIdx.x] = s;
    red_n[threadIdx.x] = n;
    __syncthreads();
    const int e = fixed_point_exp(hdr->absmax_bits, N);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        hdr->fixed_point_exp = e;
        hdr->assign_calls += 1;
    }
    if (group != 0 || !live) return;
    for (int g = 1; g < 16; ++g) {
        s += red_s[threadIdx.x + 16 * g];
        n += red_n[threadIdx.x + 16 * g];
    }
    if (n > 0) C[size_t(k) * D + j] = float(ldexp(double(s), -e) / double(n));  // an empty cluster keeps its centroid
    if (counts_out != nullptr && j == 0) counts_out[k] = n;
}

// Up to so many centroids for eight waves, every distance in direct form: what scores save is less than exchange and decision of their candidates take. Fits of 10
// iterations, us, direct / scores: N = 65536, d = 4, K = 64 96.7 / 98.7, 110 111.1 / 110.8, 170 126.4 / 122.0; 32768, d = 8, K = 80 106.6 / 107.5, 140 125.4 / 122.8;
// 65536, d = 8, K = 100 135.0 / 137.6, 200 168.3 / 163.1; 19200, d = 16, K = 90 138.6 / 141.5, 190 178.8 / 175.0.
constexpr uint32_t kDirectMost = 112;
// Workgroups of `per` groups of 64 vectors
SmallCut cut_by(uint32_t groups, uint32_t per)
{
    SmallCut c{};
    c.per_block = per * 64;
    c.blocks = (groups + per - 1) / per;
    return c;
}

// Least that a workgroup takes: at most kMaxBlocks of them
uint32_t least_per_block(uint32_t groups) { return (groups + kMaxBlocks - 1) / kMaxBlocks; }

// us of an iteration: scores, exchange and decisions on the vector ALUs (a compute unit with one workgroup issues four fifths of what one with two does),
// and the workgroups' sums out and in again at 4.5 TB/s.
double cost_of(const SmallCut& c, uint32_t d, uint32_t K, bool sums)
{
    const uint32_t at_once = 8 / uint32_t(c.slices) * c.lane, steps = (c.per_block / 64 + at_once - 1) / at_once;   // groups of 64 vectors
    const double alu = c.lane * (c.direct ? 4.0 * d + 18.0 : 2.0 * d + 7.0), lds = 4.0 * (c.direct ? 2.0 * d : 2.0 * d + 2.0);   // a centroid and wave; four SIMDs share LDS
    const double scores = double((K + c.slices - 1) / c.slices) * (std::max(alu, lds) + 0.25 * std::min(alu, lds));   // clocks of a wave and step
    const double decisions = (c.direct ? 0.0 : (c.slices == 1 ? c.lane : (at_once + 7) / 8) * (24.0 * d + 420.0)) + (c.slices > 1 ? 1000.0 : 0.0);
    const uint32_t rounds = (c.blocks + 255) / 256;
    const bool side_by_side = rounds > 1 && lds_bytes(d, K, c.lane, c.slices, sums) <= 80 * 1024;
    const double idle = c.blocks < 256 ? 0.25 * (256 - c.blocks) / 256 : 0.0;   // fewer share what all wait for
    const double us = 2.0 * rounds * (side_by_side ? 1.0 : 1.25) * (1.0 + idle) * steps * (scores + decisions) / 2200;
    if (!sums) return us;
    const double meet = double(rounds) * (c.per_block / 64) * (d + 1) * 200.0 / K / 2200;   // additions of a wave that wait for each other: 3 clocks each for 64 / K of them
    return us + meet + double(c.blocks) * 2 * double(partial_bytes(d, K)) / 4.5e6;
}

template <int D, bool SUMS>
hipError_t launch_iter_t(const float* X, uint32_t N, const float* C, uint32_t K, const SmallCut& c, uint32_t* idx, float* dmin, const Workspace& w,
                         hipStream_t s)
{
    const uint32_t lds = uint32_t(lds_bytes(D, K, c.lane, c.slices, SUMS)), stride = uint32_t(partial_bytes(D, K));
    auto launch = [&](auto kernel) {
        if (lds > 48 * 1024) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3(c.blocks), dim3(kThreads), lds, s, X, N, C, K, c.per_block, idx, dmin, w.small_partials, stride, w.hdr);
        return hipGetLastError();
    };
    if (c.lane == 1) return launch(small_iter_kernel<D, 1, 8, true, SUMS>);
    if (c.lane == 2) {
        if (c.direct) return c.slices == 1 ? launch(small_iter_kernel<D, 2, 1, true, SUMS>) : launch(small_iter_kernel<D, 2, 8, true, SUMS>);
        switch (c.slices) {
            case 1:
                if constexpr (D != 8) return launch(small_iter_kernel<D, 2, 1, false, SUMS>);
                return hipErrorInvalidValue;
            case 2:
                if constexpr (D == 16) return launch(small_iter_kernel<D, 2, 2, false, SUMS>);
                return hipErrorInvalidValue;
            case 4: return launch(small_iter_kernel<D, 2, 4, false, SUMS>);
            default: return launch(small_iter_kernel<D, 2, 8, false, SUMS>);
        }
    }
    if constexpr (D < 16) {
        if (c.lane == 3) return launch(small_iter_kernel<D, 3, 8, false, SUMS>);
        if (c.direct) return c.slices == 1 ? launch(small_iter_kernel<D, 4, 1, true, SUMS>) : launch(small_iter_kernel<D, 4, 8, true, SUMS>);
        switch (c.slices) {
            case 1: return launch(small_iter_kernel<D, 4, 1, false, SUMS>);
            case 2: return launch(small_iter_kernel<D, 4, 2, false, SUMS>);
            case 4: return launch(small_iter_kernel<D, 4, 4, false, SUMS>);
            default: return launch(small_iter_kernel<D, 4, 8, false, SUMS>);
        }
    }
    return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_small_iter_t(const float* X, uint32_t N, float* C, uint32_t K, const SmallCut& c, uint32_t* idx, float* dmin, uint32_t* counts,
                               const Workspace& w, hipStream_t s)
{
    if (hipError_t e = launch_iter_t<D, true>(X, N, C, K, c, idx, dmin, w, s); e != hipSuccess) return e;
    hipLaunchKernelGGL(small_means_kernel<D>, dim3((K * D + 15) / 16), dim3(kFinThreads), 0, s, w.small_partials,
                       uint32_t(partial_bytes(D, K)), c.blocks, C, counts, K, N, w.hdr);
    return hipGetLastError();
}

}  // namespace

// Where this form is the fastest: rows and accumulators fit LDS, and the scores cost less on the vector ALUs than what the matrix-core form pays in launches,
// latency and the M-step. Below 128 centroids the E-step is in direct form anyway. Fits of 10 iterations, us, matrix-core form (its own choice of
// windows) / this one, inputs that are fp16 numbers (others, which go through the fp32 matrix cores there, gain more): d = 4: (N, K) = (262144, 620) 538 / 397, (500000, 700)
// 778 / 669, (300000, 700) 588 / 529, (270000, 800) 586 / 506, (400000, 800) 720 / 693, (131072, 900) 421 / 331, (140000, 1000) 454 / 427, (180000, 1000) 481 / 482, (500000,
// 1000) 812 / 877, (90000, 1200) 402 / 370, (65536, 1300) 366 / 344, (131072, 1300) 440 / 486, (66000, 1490) 412 / 409; d = 8: (4 M, 450) 5936 / 4267, (4 M, 520) 6031 / 4838,
// (1 M, 560) 1762 / 1436, (300000, 560) 774 / 682, (262144, 620) 706 / 616, (500000, 620) 1044 / 967, (140000, 700) 573 / 480, (200000, 700) 667 / 648, (300000, 700) 784 /
// 795, (400000, 660) 928 / 945, (90000, 745) 517 / 398. d = 16, every codebook that fits: (20000, 390) 598 / 277, (400000, 390) 1545 / 1185, (8 M, 390)
// 22863 / 15195 (others 20405 / 15591), (1 M, 300) 2920 / 1760, (4 M, 250) 9796 / 5380, (4 M, 130) 9803 / 3381; and d = 8: (8 M, 570) 11907 / 10364.
// An E-step alone, fp16 numbers, others: d = 8: (4 M, 390) 516 / 387, 506 / 424, (800000, 400) 137 / 118, 167 / 152, (300000, 500) 83 / 76, 117 / 100, (4 M, 570) 529 / 534,
// 624 / 581; d = 4: (4 M, 280) 230 / 172, 284 / 202, (400000, 700) 75 / 71, 103 / 91, (130000, 900) 44 / 33, 59 / 39: the same lines.
bool small_problem(uint64_t N, uint32_t d, uint32_t K)
{
    if (state_bytes(d, K) > kMaxLds || N >= (1ull << 31)) return false;
    if (d == 4) return K <= 288 || N * K <= (K <= 720 ? 360000000ull : (K <= 832 ? 320000000ull : (K <= 1024 ? 180000000ull : 100000000ull)));
    if (d == 8) return K <= 576 || N * K <= (K <= 640 ? 310000000ull : 140000000ull);
    return true;
}

// How the vectors are dealt out: the cheapest of as many workgroups as there may be, or fewer, of 2, 3 or 4 vectors to a lane and 8, 4, 2 or 1 ways to split the
// codebook that a kernel exists for. A codebook that is not split goes in direct form where that costs less, up to 20 to 30 centroids: what a decision takes beside its
// scores is 24 d + 420 clocks. With few of them the additions to the sums meet, and the fullest compute unit is what a call waits for. Fits of 10
// iterations, us, scores alone and meetings not counted / now: (376704, 16, 4) 281 / 200, (590848, 8, 4) 251 / 190, (2.6 M, 8, 2) 770 / 610, (2.1 M, 8, 10) 428 / 368, (3.3 M, 4,
// 3) 455 / 400, (417152, 8, 20) 194 / 171. Few groups to a workgroup leave none of the larger steps whole; steps that are split 8 ways fit any number.
SmallCut small_cut(uint32_t N, uint32_t d, uint32_t K, bool sums)
{
    const uint32_t groups = (N + 63) / 64, least = least_per_block(groups);
    SmallCut best{};
    double best_cost = 1e300;
    for (uint32_t per = least; per <= 2 * least + 1; per += std::max(1u, least / 16)) {
        SmallCut c = cut_by(groups, per);
        for (int lane = d == 16 ? 2 : 4; lane >= 1; --lane) {
            if ((lane == 1) != (per == 1)) continue;
            for (int slices = 8; slices >= (lane == 1 || lane == 3 ? 8 : 1); slices /= 2) {
                if (lane == 2 && slices == 2 && d != 16) continue;   // no size takes these
                c.lane = lane;
                c.slices = slices;
                for (int form = 0; form < 2; ++form) {
                    c.direct = lane == 1 || (slices == 8 && lane != 3 && K <= kDirectMost) || form == 1;
                    if (form == 1 && slices != 1) break;   // not split: whichever costs less
                    if (lane == 2 && d == 8 && slices == 1 && !c.direct) continue;   // no size
                    const double cost = cost_of(c, d, K, sums);
                    if (cost < best_cost) {
                        best_cost = cost;
                        best = c;
                    }
                }
            }
        }
    }
    return best;
}

size_t small_partials_bytes(uint64_t N, uint32_t d, uint32_t K)
{
    if (!small_problem(N, d, K)) return 0;
    const uint32_t groups = uint32_t((N + 63) / 64);
    return size_t(cut_by(groups, least_per_block(groups)).blocks) * partial_bytes(d, K);
}

hipError_t launch_small_iter(const float* X, uint32_t N, uint32_t d, float* C, uint32_t K, const SmallCut& cut, uint32_t* idx, float* dmin,
                             uint32_t* counts, const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: return launch_small_iter_t<4>(X, N, C, K, cut, idx, dmin, counts, w, s);
        case 8: return launch_small_iter_t<8>(X, N, C, K, cut, idx, dmin, counts, w, s);
        case 16: return launch_small_iter_t<16>(X, N, C, K, cut, idx, dmin, counts, w, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_small_assign(const float* X, uint32_t N, uint32_t d, const float* C, uint32_t K, uint32_t* idx, float* dmin,
                               const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: return launch_iter_t<4, false>(X, N, C, K, small_cut(N, d, K, false), idx, dmin, w, s);
        case 8: return launch_iter_t<8, false>(X, N, C, K, small_cut(N, d, K, false), idx, dmin, w, s);
        case 16: return launch_iter_t<16, false>(X, N, C, K, small_cut(N, d, K, false), idx, dmin, w, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cc
