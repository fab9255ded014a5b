// Lloyd iterations of small problems (Section 3.1) in two launches each: E-step in direct form with the codebook in
// LDS and the cluster sums taken in the same kernel, then one kernel that adds the workgroups' sums and divides.
//
// What bounds a small fit is not arithmetic: at N = 65536, K = 256, d = 4 the matrix-core E-step fills half of the chip
// (128 workgroups of 512 vectors) and spends its time in the latency of its stages and of the index recovery (57 us for
// 17 M distances), and an iteration is eleven launches of 2 us each, most of them gated off. In direct form every
// distance is final - no guard band, no refinement, no recovery - and costs 2 d + 3 vector instructions: 5 us of
// vector-ALU time for that E-step.
//
// A workgroup of 8 waves holds the codebook (K rows, fp32) and the accumulators (64-bit fixed-point sums and counts) in
// LDS. Its waves split the codebook S ways when there are too few vectors to give every lane one of its own; the S
// partial minima of a vector meet in LDS, and the lower index wins among equal distances as everywhere. The sums are
// the same integers as in the other formulations of the M-step, so the centroids are the same bits.
// Measured (fit of 10 iterations, N = 65536, K = 256, d = 4): 871 -> 155 us.
#include <algorithm>

#include "common.h"

namespace cc {

namespace {

constexpr int kThreads = 512;
constexpr uint32_t kMaxBlocks = 512;      // two workgroups per compute unit
constexpr uint32_t kMaxLds = 76 * 1024;   // two workgroups per compute unit next to the exchange buffers

// LDS of one workgroup: codebook rows, sums [D][K], counts [K]
size_t lds_bytes(uint32_t d, uint32_t K) { return size_t(K) * (d * 4 + d * 8 + 4); }

// bytes of one workgroup's partial sums: [D][K] int64, then [K] counts, rounded to whole 64-bit words
size_t partial_bytes(uint32_t d, uint32_t K) { return (size_t(K) * (d * 8 + 4) + 7) & ~size_t(7); }

template <int D, int S, bool SUMS>
__global__ __launch_bounds__(kThreads) void small_iter_kernel(const float* __restrict__ X, uint32_t N, const float* __restrict__ C,
                                                              uint32_t K, uint32_t per_block, uint32_t* __restrict__ idx,
                                                              float* __restrict__ dmin, char* __restrict__ partials,
                                                              uint32_t partial_stride, WsHeader* __restrict__ hdr)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* rows = reinterpret_cast<float*>(smem);                                                    // [K][D]
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(smem + size_t(K) * D * 4);      // [D][K]
    uint32_t* counts = reinterpret_cast<uint32_t*>(smem + size_t(K) * D * 12);                       // [K]
    __shared__ float best_d[S > 1 ? kThreads : 1];
    __shared__ uint32_t best_k[S > 1 ? kThreads : 1];
    for (uint32_t t = threadIdx.x; t < K * (D / 4); t += kThreads)
        reinterpret_cast<float4*>(rows)[t] = reinterpret_cast<const float4*>(C)[t];
    if constexpr (SUMS) {
        for (uint32_t t = threadIdx.x; t < K * D; t += kThreads) sums[t] = 0;
        for (uint32_t t = threadIdx.x; t < K; t += kThreads) counts[t] = 0;
    }
    __syncthreads();
    const int e = SUMS ? fixed_point_exp(hdr->absmax_bits, N) : 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr uint32_t VS = kThreads / S;                       // vectors of one step
    const uint32_t slice = uint32_t(wave) % S, local = (uint32_t(wave) / S) * 64 + lane;
    const uint32_t k_per = (K + S - 1) / S;
    const uint32_t k_lo = min(slice * k_per, K), k_hi = min(k_lo + k_per, K);
    const uint32_t lo = blockIdx.x * per_block, hi = min(lo + per_block, N);
    for (uint32_t v0 = lo; v0 < hi; v0 += VS) {
        const uint32_t i = v0 + local;
        float x[D];
        load_row<D>(X + size_t(min(i, N - 1)) * D, x);
        float bd = INFINITY;
        uint32_t bk = k_lo;
#pragma unroll 4
        for (uint32_t k = k_lo; k < k_hi; ++k) {
            float c[D];
            load_row<D>(rows + size_t(k) * D, c);
            const float dist = direct_sqdist<D>(x, c);
            if (dist < bd) {
                bd = dist;
                bk = k;
            }
        }
        if constexpr (S > 1) {
            __syncthreads();   // the exchange buffers of the step before have been read
            best_d[threadIdx.x] = bd;
            best_k[threadIdx.x] = bk;
            __syncthreads();
            if (slice != 0) continue;
#pragma unroll
            for (int o = 1; o < S; ++o) {   // ascending slices: a strict "<" keeps the lowest index
                const float od = best_d[threadIdx.x + 64 * o];
                if (od < bd) {
                    bd = od;
                    bk = best_k[threadIdx.x + 64 * o];
                }
            }
        }
        if (i < hi) {
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
#pragma unroll 8
    for (uint32_t b = group; b < blocks; b += 16) {
        const unsigned long long* ps = reinterpret_cast<const unsigned long long*>(partials + size_t(b) * partial_stride);
        s += static_cast<long long>(ps[j * K + k]);
        n += reinterpret_cast<const uint32_t*>(ps + size_t(K) * D)[k];
    }
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

struct Cut {
    uint32_t blocks, per_block;
    int slices;
};

// Workgroups of at least 64 vectors, at most `most`; with fewer vectors per workgroup than threads the waves split
// the codebook (8, 4 or 2 ways) instead of idling.
Cut cut_into(uint32_t N, uint32_t most)
{
    Cut c;
    const uint32_t groups = (N + 63) / 64;
    const uint32_t per = (groups + most - 1) / most;   // groups of 64 vectors per workgroup
    c.per_block = per * 64;
    c.blocks = (groups + per - 1) / per;
    c.slices = per >= 8 ? 1 : (per >= 4 ? 2 : (per >= 2 ? 4 : 8));
    return c;
}

// us of an iteration: distances on the vector ALUs (2.7 clocks per instruction with two workgroups on a compute unit, 3.5 with one), and
// the workgroups' sums out and in again at 3 TB/s.
double cost_of(const Cut& c, uint32_t d, uint32_t K)
{
    const uint32_t at_once = 8 / uint32_t(c.slices), groups = c.per_block / 64;   // groups of 64 vectors
    const double instructions = double(c.blocks) * 8 / 1024 * ((groups + at_once - 1) / at_once) * ((K + c.slices - 1) / c.slices) * (2 * d + 4);
    return instructions * (c.blocks <= 256 ? 3.5 : 2.7) / 2200 + double(c.blocks) * 2 * double(partial_bytes(d, K)) / 3e6;
}

// One or two workgroups per compute unit: two hide each other's latencies, one leaves half as many partial sums to add. Fits of 10
// iterations, us, two / one: N = 65536, K = 256, d = 4 168 / 153; N = 32768, K = 300, d = 16 334 / 290; N = 512000, K = 100, d = 4 301 / 333;
// N = 76800, K = 1000, d = 4 520 / 566.
Cut cut_of(uint32_t N, uint32_t d, uint32_t K)
{
    const Cut two = cut_into(N, kMaxBlocks), one = cut_into(N, kMaxBlocks / 2);
    return cost_of(one, d, K) < cost_of(two, d, K) ? one : two;
}

template <int D, bool SUMS>
hipError_t launch_iter_t(const float* X, uint32_t N, const float* C, uint32_t K, uint32_t* idx, float* dmin, const Workspace& w,
                         hipStream_t s)
{
    const Cut c = SUMS ? cut_of(N, D, K) : cut_into(N, kMaxBlocks);
    const uint32_t lds = uint32_t(SUMS ? lds_bytes(D, K) : size_t(K) * D * 4), stride = uint32_t(partial_bytes(D, K));
#define CC_SMALL(S)                                                                                                       \
    do {                                                                                                                  \
        if (lds > 48 * 1024) {                                                                                            \
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&small_iter_kernel<D, S, SUMS>),       \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(kMaxLds));           \
            if (e != hipSuccess) return e;                                                                                \
        }                                                                                                                 \
        hipLaunchKernelGGL((small_iter_kernel<D, S, SUMS>), dim3(c.blocks), dim3(kThreads), lds, s, X, N, C, K, c.per_block, idx, \
                           dmin, w.small_partials, stride, w.hdr);                                                        \
    } while (0)
    switch (c.slices) {
        case 1: CC_SMALL(1); break;
        case 2: CC_SMALL(2); break;
        case 4: CC_SMALL(4); break;
        default: CC_SMALL(8); break;
    }
#undef CC_SMALL
    return hipGetLastError();
}

template <int D>
hipError_t launch_small_iter_t(const float* X, uint32_t N, float* C, uint32_t K, uint32_t* idx, float* dmin, uint32_t* counts,
                               const Workspace& w, hipStream_t s)
{
    if (hipError_t e = launch_iter_t<D, true>(X, N, C, K, idx, dmin, w, s); e != hipSuccess) return e;
    hipLaunchKernelGGL(small_means_kernel<D>, dim3((K * D + 15) / 16), dim3(kFinThreads), 0, s, w.small_partials,
                       uint32_t(partial_bytes(D, K)), cut_of(N, D, K).blocks, C, counts, K, N, w.hdr);
    return hipGetLastError();
}

}  // namespace

// Where this form is the fastest: the accumulators fit LDS, and the distances cost less in direct form than what the
// matrix-core form pays in launches, latency and the M-step. Below 128 centroids the E-step is in direct form anyway. Fits of 10
// iterations, us, matrix-core form (its own choice of windows) / this one, inputs that are fp16 numbers: d = 4: K = 140: N = 260000 515 / 236, 10 M 6766 / 4023;
// K = 250: 10 M 8997 / 6899; K = 500: 260000 570 / 509, 520000 863 / 852; d = 8: K = 140: 4 M 5596 / 2853; K = 390: 4.5 M 9297 / 8250; K = 500: 260000 852 / 779;
// d = 16: K = 250: 2.5 M 9608 / 5412; K = 300: 430000 2072 / 1424. From 512 centroids on what counts is how N falls into groups of 64 for 512
// workgroups, and the kind of the inputs, which nobody knows here: those that are no fp16 numbers go through the fp32 matrix cores. fp16 numbers / others: d = 4:
// K = 513: 131072 396 / 331, 529 / 338, 230000 512 / 501, 615 / 511; K = 600: 131072 399 / 376, 530 / 382, 131200 428 / 530, 587 / 536, 230000 514 / 571,
// 613 / 581; K = 800: 131072 405 / 444, 561 / 452; K = 900: 60000 367 / 326, 548 / 329, 131072 408 / 503, 563 / 509; K = 1000: 60000 365 / 357, 547 / 359; d = 8:
// K = 513: 131072 510 / 505, 694 / 519, 160000 571 / 770, 842 / 791; K = 600: 110000 505 / 554, 685 / 563; K = 700: 55000 439 / 398, 672 / 402, 131072 518 / 622,
// 703 / 637.
bool small_problem(uint64_t N, uint32_t d, uint32_t K)
{
    if (lds_bytes(d, K) > kMaxLds || N >= (1ull << 31)) return false;
    if (K < (d == 4 ? 256u : 400u)) return true;
    if (K <= (d == 4 ? 560u : 512u)) return N * K <= (d == 4 ? 1ull << 28 : 1ull << 27);
    return (N <= (1u << 16) && N * K <= (1ull << 26)) || (N <= (1u << 17) && K <= (d == 4 ? 832u : 608u));
}

// An E-step alone (matrix cores / this form, us, fp16 numbers, others): d = 8, K = 340: 4 M 688 / 556, 578 / 595; K = 370: 720 / 604, 584 / 644; K = 399: 731 / 648,
// 587 / 690. Lines that would cost the first more than they give the others are not drawn: d = 4, K = 240: 4 M 332 / 253, 263 / 279; d = 16, K = 340: 280000 169 / 147,
// 152 / 175, 420000 217 / 146, 187 / 175.
bool small_assign_pays(uint64_t N, uint32_t d, uint32_t K) { return d != 8 || K <= 368 || N * K <= (1ull << 27); }

size_t small_partials_bytes(uint64_t N, uint32_t d, uint32_t K)
{
    return small_problem(N, d, K) ? size_t(cut_into(uint32_t(N), kMaxBlocks).blocks) * partial_bytes(d, K) : 0;
}

hipError_t launch_small_iter(const float* X, uint32_t N, uint32_t d, float* C, uint32_t K, uint32_t* idx, float* dmin,
                             uint32_t* counts, const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: return launch_small_iter_t<4>(X, N, C, K, idx, dmin, counts, w, s);
        case 8: return launch_small_iter_t<8>(X, N, C, K, idx, dmin, counts, w, s);
        case 16: return launch_small_iter_t<16>(X, N, C, K, idx, dmin, counts, w, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_small_assign(const float* X, uint32_t N, uint32_t d, const float* C, uint32_t K, uint32_t* idx, float* dmin,
                               const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: return launch_iter_t<4, false>(X, N, C, K, idx, dmin, w, s);
        case 8: return launch_iter_t<8, false>(X, N, C, K, idx, dmin, w, s);
        case 16: return launch_iter_t<16, false>(X, N, C, K, idx, dmin, w, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cc
