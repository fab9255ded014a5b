// Incremental M-step inside a fit (Section 3.1: c_k <- mean of its vectors): the cluster sums are integers, so they can be kept up to
// date instead of recomputed. From the third iteration on (the second of a fit by cells) only the vectors whose code changed since the
// previous one (18 % of them in the second iteration of the 4-bit benchmark, 2 % in the twentieth) are looked at, each twice: plus for
// the new cluster, minus for the old one. Bit-identical to a recomputation. The E-step that produced the codes leaves a bitmap of the
// vectors that may have changed, and their previous codes.
//
// Two launches. One workgroup per 16384 vectors packs the flagged ones into a list and sorts their two entries (offset within the chunk,
// sign, cluster) by slice, 512 slices of the clusters at most; then one workgroup per slice goes through the runs of its slice in all
// chunks, fetches the rows, adds them in LDS to the slice's sums, and those to what the workspace holds, and writes the means. Slices are
// taken over the centroids' position in the norm order (cinv), which neighbouring vectors share.
//
// Bound: latency (four dependent reads in the first kernel, five in the second), and at d = 4 a line per fetched row, twice per changed
// vector. The former way - count, two scans, copy into records by bucket, sums, for few clusters the means - took six launches. An
// iteration's M-step, before / now, us: 11.3 M vectors of 4, K = 65536 87 / 52 (18 + 34), 4.2 M of 4, K = 4096 57 / 26, 2.8 M of 6, K = 65500 52 / 23. 512
// threads per slice: with 256 the first of these fits takes 14.17 ms instead of 14.10, with 1024 the second 5.46 instead of 5.38.
#include "common.h"

namespace cc {

namespace {

constexpr int kCollectThreads = 1024, kSumThreads = 512;
constexpr uint32_t kMostSlices = 512, kOffsetBits = 14;
constexpr uint32_t kRound = 2048;        // chunks whose runs a workgroup holds in LDS at once
constexpr uint32_t kSliceClusters = 65536 / kMostSlices;   // at most
static_assert(kDeltaChunk == 1u << kOffsetBits && kDeltaChunk == 16 * kCollectThreads, "offset bits; half a bitmap word per thread");

// log2 of the clusters per slice: as many slices as there may be, of at least 4 clusters
uint32_t slice_bits(uint32_t K)
{
    uint32_t bits = 2;
    while (((K - 1) >> bits) + 1 > kMostSlices) ++bits;
    return bits;
}

// Exclusive prefix sum over the workgroup of one value per thread; `total` receives the sum.
template <int THREADS>
__device__ __forceinline__ uint32_t exclusive_scan(uint32_t v, uint32_t* wave_sum, uint32_t& total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = uint32_t(__shfl_up(int(incl), off, 64));
        if (lane >= off) incl += t;
    }
    __syncthreads();  // wave_sum may still be read from an earlier call
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - v;
    total = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        before += w < wave ? wave_sum[w] : 0u;
        total += wave_sum[w];
    }
    return before;
}

// An entry: offset in the chunk, 1 bit minus, cluster within the slice.
__global__ __launch_bounds__(kCollectThreads) void delta_collect_kernel(const uint32_t* __restrict__ idx, const uint32_t* __restrict__ prev,
                                                                        const uint32_t* __restrict__ changed, uint32_t N, uint32_t K,
                                                                        const uint32_t* __restrict__ cinv, uint32_t slices, uint32_t bits,
                                                                        uint32_t* __restrict__ runs, uint32_t* __restrict__ entries)
{
    __shared__ uint16_t flagged[kDeltaChunk];
    __shared__ uint32_t cursor[kMostSlices];
    __shared__ uint32_t wave_sum[kCollectThreads / 64];
    const uint32_t lo = blockIdx.x * kDeltaChunk;
    if (threadIdx.x < kMostSlices) cursor[threadIdx.x] = 0;
    // the flagged offsets, packed: half a word of the bitmap each (bits beyond N are never set)
    const uint32_t first = 16 * threadIdx.x;
    uint32_t word = lo + first < N ? (changed[(lo + first) >> 5] >> (first & 31)) & 0xffffu : 0u, total;
    uint32_t pos = exclusive_scan<kCollectThreads>(uint32_t(__popc(word)), wave_sum, total);
    for (; word != 0; word &= word - 1) flagged[pos++] = uint16_t(first + uint32_t(__ffs(int(word)) - 1));
    __syncthreads();
    struct Change {
        uint32_t at, plus, minus;   // positions of the clusters; plus == minus: none
    };
    auto look = [&](uint32_t e) {
        const uint32_t at = flagged[e], k = idx[lo + at], kp = prev[lo + at];
        const bool moved = k != kp && k < K && kp < K;
        const uint32_t a = moved ? k : 0u, b = moved ? kp : 0u;
        return Change{at, cinv != nullptr ? cinv[a] : a, cinv != nullptr ? cinv[b] : b};
    };
    auto count = [&](const Change& c) {
        if (c.plus == c.minus) return;
        atomicAdd(&cursor[c.plus >> bits], 1u);
        atomicAdd(&cursor[c.minus >> bits], 1u);
    };
    // the first of a thread are kept for the second pass
    constexpr int kKept = 2;
    Change kept[kKept];
#pragma unroll
    for (int q = 0; q < kKept; ++q) {
        const uint32_t e = q * kCollectThreads + threadIdx.x;
        kept[q] = e < total ? look(e) : Change{0u, 0u, 0u};
    }
#pragma unroll
    for (int q = 0; q < kKept; ++q) count(kept[q]);
    for (uint32_t e = kKept * kCollectThreads + threadIdx.x; e < total; e += kCollectThreads) count(look(e));
    __syncthreads();
    uint32_t all;
    const uint32_t n = threadIdx.x < slices ? cursor[threadIdx.x] : 0u, begin = exclusive_scan<kCollectThreads>(n, wave_sum, all);
    if (threadIdx.x < slices) {
        runs[size_t(blockIdx.x) * slices + threadIdx.x] = begin | n << 16;   // both at most 32768
        cursor[threadIdx.x] = begin;
    }
    __syncthreads();
    uint32_t* out = entries + size_t(lo) * 2;
    auto place = [&](const Change& c) {
        if (c.plus == c.minus) return;
        const uint32_t mask = (1u << bits) - 1;
        out[atomicAdd(&cursor[c.plus >> bits], 1u)] = c.at | (c.plus & mask) << (kOffsetBits + 1);
        out[atomicAdd(&cursor[c.minus >> bits], 1u)] = c.at | 1u << kOffsetBits | (c.minus & mask) << (kOffsetBits + 1);
    };
#pragma unroll
    for (int q = 0; q < kKept; ++q) place(kept[q]);
    for (uint32_t e = kKept * kCollectThreads + threadIdx.x; e < total; e += kCollectThreads) place(look(e));
}

// One workgroup per slice. Every thread takes a stretch of the slice's entries: where the vectors lie ordered by cluster, neighbouring
// entries add to one accumulator.
template <int D>
__global__ __launch_bounds__(kSumThreads) void delta_sum_kernel(const float* __restrict__ X, uint32_t N, uint32_t K, const uint32_t* __restrict__ cperm,
                                                                uint32_t chunks, uint32_t slices, uint32_t bits, const uint32_t* __restrict__ runs,
                                                                const uint32_t* __restrict__ entries, const float* prev, float* out,
                                                                uint32_t* counts_out, WsHeader* hdr, long long* __restrict__ sums_ws,
                                                                uint32_t* __restrict__ counts_ws)
{
    __shared__ unsigned long long sum[D][kSliceClusters + 1];
    __shared__ uint32_t cnt[kSliceClusters];
    __shared__ uint32_t before[kRound + 1];   // entries in the runs before this one
    __shared__ uint16_t at[kRound];           // where the run begins in its chunk
    __shared__ uint32_t wave_sum[kSumThreads / 64];
    const uint32_t clusters = 1u << bits, p0 = blockIdx.x << bits;
    for (uint32_t t = threadIdx.x; t < (kSliceClusters + 1) * D; t += kSumThreads) (&sum[0][0])[t] = 0;
    if (threadIdx.x < kSliceClusters) cnt[threadIdx.x] = 0;
    const int e = fixed_point_exp(hdr->absmax_bits, N);
    for (uint32_t c0 = 0; c0 < chunks; c0 += kRound) {
        constexpr uint32_t kEach = kRound / kSumThreads;
        uint32_t run[kEach], mine = 0;
#pragma unroll
        for (uint32_t q = 0; q < kEach; ++q) {
            const uint32_t c = c0 + threadIdx.x * kEach + q;
            run[q] = c < chunks ? runs[size_t(c) * slices + blockIdx.x] : 0u;
        }
#pragma unroll
        for (uint32_t q = 0; q < kEach; ++q) mine += run[q] >> 16;
        uint32_t total;
        uint32_t upto = exclusive_scan<kSumThreads>(mine, wave_sum, total);   // begins with a barrier: `before` is read no more
#pragma unroll
        for (uint32_t q = 0; q < kEach; ++q) {
            before[threadIdx.x * kEach + q] = upto;
            at[threadIdx.x * kEach + q] = uint16_t(run[q] & 0xffffu);
            upto += run[q] >> 16;
        }
        if (threadIdx.x == kSumThreads - 1) before[kRound] = total;
        __syncthreads();
        const uint32_t per = (total + kSumThreads - 1) / kSumThreads;
        const uint32_t first = min(threadIdx.x * per, total), last = min(first + per, total);
        uint32_t r = 0;   // the run of entry `first`
        for (uint32_t step = kRound / 2; step > 0; step /= 2) r += before[r + step] <= first ? step : 0u;
        constexpr int U = D == 16 ? 2 : 4;
        for (uint32_t i = first; i < last; i += U) {
            uint32_t where[U], chunk[U], entry[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t j = min(i + u, last - 1);
                while (before[r + 1] <= j) ++r;
                chunk[u] = c0 + r;
                where[u] = at[r] + (j - before[r]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) entry[u] = entries[size_t(chunk[u]) * (2 * kDeltaChunk) + where[u]];
            float x[U][D];
#pragma unroll
            for (int u = 0; u < U; ++u) load_row<D>(X + (size_t(chunk[u]) * kDeltaChunk + (entry[u] & (kDeltaChunk - 1))) * D, x[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i + u >= last) continue;
                const uint32_t local = entry[u] >> (kOffsetBits + 1);
                const bool minus = (entry[u] >> kOffsetBits) & 1;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const long long v = fixed_point_term(x[u][j], e);
                    atomicAdd(&sum[j][local], static_cast<unsigned long long>(minus ? -v : v));   // two's complement: wraps like int64
                }
                atomicAdd(&cnt[local], minus ? 0xffffffffu : 1u);
            }
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) hdr->fixed_point_exp = e;
    for (uint32_t t = threadIdx.x; t < clusters * D; t += kSumThreads) {
        const uint32_t local = t / D, j = t % D;
        if (p0 + local >= K) continue;
        const uint32_t k = cperm != nullptr ? cperm[p0 + local] : p0 + local;
        const size_t o = size_t(k) * D + j;
        const uint32_t n = counts_ws[k] + cnt[local];
        const long long isum = sums_ws[o] + static_cast<long long>(sum[j][local]);
        sums_ws[o] = isum;
        const double whole = ldexp(double(isum), -e);
        out[o] = n > 0 ? float(whole / double(n)) : prev[o];   // one fp64 division, one rounding; an empty cluster keeps its centroid
    }
    __syncthreads();   // every count has been read
    for (uint32_t local = threadIdx.x; local < clusters; local += kSumThreads) {
        if (p0 + local >= K) continue;
        const uint32_t k = cperm != nullptr ? cperm[p0 + local] : p0 + local, n = counts_ws[k] + cnt[local];
        counts_ws[k] = n;
        if (counts_out != nullptr) counts_out[k] = n;
    }
}

template <int D>
hipError_t update_delta_t(const float* X, uint32_t N, const uint32_t* idx, const float* prev, uint32_t K, float* out, uint32_t* counts_out,
                          const Workspace& w, hipStream_t s)
{
    const uint32_t chunks = (N + kDeltaChunk - 1) / kDeltaChunk, bits = slice_bits(K), slices = ((K - 1) >> bits) + 1;
    uint32_t* entries = reinterpret_cast<uint32_t*>(w.records);
    uint32_t* runs = reinterpret_cast<uint32_t*>(w.records + align256(size_t(N) * 8));
    hipLaunchKernelGGL(delta_collect_kernel, dim3(chunks), dim3(kCollectThreads), 0, s, idx, w.idx_prev, w.changed, N, K, w.cinv, slices, bits, runs, entries);
    hipLaunchKernelGGL(delta_sum_kernel<D>, dim3(slices), dim3(kSumThreads), 0, s, X, N, K, w.cperm, chunks, slices, bits, runs, entries, prev, out,
                       counts_out, w.hdr, w.sums, w.counts);
    return hipGetLastError();
}

}  // namespace

// Room for entries and runs in the record buffer (2 N records); a few thousand vectors of many clusters have none.
bool update_delta_applies(uint32_t N, uint32_t d, uint32_t K, const Workspace& w)
{
    if (!w.bucket_ok || w.records == nullptr) return false;
    const uint32_t slices = ((K - 1) >> slice_bits(K)) + 1;
    return align256(size_t(N) * 8) + size_t((N + kDeltaChunk - 1) / kDeltaChunk) * slices * 4 <= size_t(N) * 2 * (4 * d + 16);
}

hipError_t launch_update_delta(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, const float* prev, uint32_t K, float* out,
                               uint32_t* counts_out, const Workspace& w, hipStream_t s)
{
    if (!update_delta_applies(N, d, K, w)) return hipErrorInvalidValue;
    switch (d) {
        case 4: return update_delta_t<4>(X, N, idx, prev, K, out, counts_out, w, s);
        case 8: return update_delta_t<8>(X, N, idx, prev, K, out, counts_out, w, s);
        case 16: return update_delta_t<16>(X, N, idx, prev, K, out, counts_out, w, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cc
