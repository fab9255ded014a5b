// M-step by cluster slices (Section 3.1: c_k <- mean of the vectors assigned to cluster k), for many vectors and
// K <= 65536: two passes over the codes, no copy of the vectors.
//
// The K x (d sums + count) accumulators do not fit one workgroup's LDS, but a slice of them does (4096 clusters at
// d = 4, 2048 at d = 8, 1024 at d = 16: 64-bit fixed-point sums, about 144 KB). So the clusters are cut into slices and
// the vectors into chunks of 7168. A first kernel sorts the codes of every chunk by slice, as 32-bit entries (position
// within the chunk, cluster within the slice), and on the way looks for the largest magnitude, which fixes the exponent of
// the sums; then workgroup (slice s, range r of chunks) reads its entries, fetches their rows and adds them into its LDS
// accumulators with integer atomics. The per-workgroup results go to the workspace and a third kernel adds the ranges of
// every cluster and divides. One slice needs no entries.
//
// Every row is read once by each of the first two kernels; what is written is 4 bytes per vector and the partial sums
// (37 MB at K = 65536, d = 4). Workgroups are numbered so that one XCD (they are dealt to the 8 XCDs in turn) owns whole
// ranges: its L2 then serves the cache lines whose rows belong to several slices. The sums are the same 64-bit integers as
// in the other formulations of the M-step, so the result is the same bits, whatever the scheduling.
//
// The same kernels serve the gradient of a layer's codebook (Sections 3.2-3.3: the sum of the weight gradient over the
// entries rebuilt from each codebook entry): there the rows are 16-bit numbers and the codes the layer's stored 16-bit
// codes, both read in place and converted as they are fetched (SRC below).
//
// Bound: with many slices, one 8/16/32/64-byte row fetch per vector from a different cache line each - the L1 fill rate
// (about 0.35 lines per clock and compute unit); with few, the two passes over the rows (5 TB/s). The former form had every
// slice look at every code, with packed positions in an LDS queue, after a reset, a scan and an fp64 conversion per number.
// Before and after, a whole call: 11.3 M vectors of 4 at K = 65536 159 -> 134 us (53 chunks, 68 sums, 10 means); 28 M of 8
// 845 -> 484; 1.1 M of 4 at K = 300 106 -> 26; 6 M of 16 at K = 3000 206 -> 181; bf16 gradient of a 4096x11008 layer
// 142 -> 108. 28 M of 8 at K = 6000 pay for writing and reading the entries: 420 -> 435.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace cc {

namespace {

constexpr int kThreads = 1024;            // 16 waves: what hides the latency of the row fetches
constexpr int kWaves = kThreads / 64;
constexpr uint32_t kWorkgroups = 256;
constexpr uint32_t kLeast = 32768;        // vectors; below, few memory-side atomics take no longer (20000 of 16 numbers: 33 and 36 us)
constexpr int kChunkThreads = 512;        // for a chunk: finer grains than 1024, 4 M vectors are 585 chunks
constexpr uint32_t kChunk = 7168;         // vectors sorted together
constexpr uint32_t kPosBits = 13;
constexpr uint32_t kCounters = 512;       // of a chunk: slices x 8 groups of positions x what is left for the lanes, so that
constexpr uint32_t kGroups = 8;           // few of them take turns at one counter

// Where rows and codes come from: 0 = fp32 rows and 32-bit codes (the clustering), 1 = fp16 and 2 = bf16 rows with
// 16-bit codes (a layer's gradient): the numbering of cc_dtype.
// A row comes in pieces of at most 16 bytes, one per lane: neighbouring lanes take neighbouring pieces of one row, which
// costs one cache lookup per row instead of one per load (d = 16: 146 -> 93 us for 8 M rows).
template <int D, int SRC>
struct Piece {
    static constexpr int kNumbers = SRC == 0 ? 4 : (D < 8 ? D : 8);
    static constexpr int kLanes = D / kNumbers;
};

template <int D, int SRC>
__device__ __forceinline__ void fetch_piece(const void* __restrict__ X, size_t row, uint32_t piece, float (&v)[Piece<D, SRC>::kNumbers])
{
    constexpr int n = Piece<D, SRC>::kNumbers;
    if constexpr (SRC == 0) {
        const float4 t = *reinterpret_cast<const float4*>(static_cast<const float*>(X) + row * D + piece * n);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
        uint32_t w[n / 2];  // two numbers per word, the lower-addressed one in the low half
        const uint16_t* from = static_cast<const uint16_t*>(X) + row * D + piece * n;
        if constexpr (n == 4) {
            const uint2 t = *reinterpret_cast<const uint2*>(from);
            w[0] = t.x; w[1] = t.y;
        } else {
            const uint4 t = *reinterpret_cast<const uint4*>(from);
            w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
        }
#pragma unroll
        for (int p = 0; p < n / 2; ++p) {
            if constexpr (SRC == 2) {
                v[2 * p] = __uint_as_float(w[p] << 16);
                v[2 * p + 1] = __uint_as_float(w[p] & 0xffff0000u);
            } else {
                const uint16_t lo = uint16_t(w[p] & 0xffffu), hi = uint16_t(w[p] >> 16);
                v[2 * p] = float(__builtin_bit_cast(_Float16, lo));
                v[2 * p + 1] = float(__builtin_bit_cast(_Float16, hi));
            }
        }
    }
}

template <int SRC>
__device__ __forceinline__ uint32_t code_at(const void* idx, size_t i)
{
    if constexpr (SRC == 0) return static_cast<const uint32_t*>(idx)[i];
    else return static_cast<const uint16_t*>(idx)[i];
}

// As many clusters as LDS holds, one workgroup per compute unit.
template <int D>
struct Slice {
    static constexpr uint32_t kBits = D == 4 ? 12u : (D == 8 ? 11u : 10u);
    static constexpr uint32_t kClusters = 1u << kBits;
    // sums of one component lie side by side; the two extra keep the lanes that share a row off one bank
    static constexpr uint32_t kPitch = kClusters + 2;
    static constexpr uint32_t kSumBytes = kPitch * D * 8;
    static constexpr uint32_t kLdsBytes = kSumBytes + kClusters * 4;
    static_assert((65536u >> kBits) <= 64u && kBits + kPosBits <= 32u, "a lane per slice; an entry in 32 bits");
};

// What the input scan found in one chunk, and its codes >= K.
struct ScanPart {
    uint32_t absmax, flags, skipped, pad;   // flags: bit 0 = not fit for the fp16 kernels, bit 1 = a non-finite input
};

struct Cut {
    bool listed;
    uint32_t slices, chunks, ranges;
    uint32_t sharers;   // waves that share a chunk's entries
    size_t sum_bytes, part_bytes, entry_bytes, start_bytes;
};

// The record buffer (2 N records) holds it all; ranges = 0: not even one range of partial sums fits.
template <int D>
Cut cut_of(uint32_t N, uint32_t K)
{
    const size_t have = size_t(N) * 2 * (4 * D + 16);
    Cut c;
    c.listed = !update_one_slice(D, K);
    static_assert(Slice<D>::kClusters == 16384 / D);
    c.slices = (K + Slice<D>::kClusters - 1) / Slice<D>::kClusters;
    c.chunks = uint32_t((uint64_t(N) + kChunk - 1) / kChunk);
    c.part_bytes = align256(size_t(c.chunks) * sizeof(ScanPart));
    c.entry_bytes = c.listed ? align256(size_t(c.chunks) * kChunk * 4) : 0;
    c.start_bytes = c.listed ? align256(size_t(c.chunks) * (c.slices + 1) * 4) : 0;
    const size_t taken = c.part_bytes + c.entry_bytes + c.start_bytes + 256, per_range = size_t(c.slices) * Slice<D>::kLdsBytes;
    const uint32_t fit = uint32_t(have > taken ? std::min<size_t>((have - taken) / per_range, kWorkgroups) : 0);
    c.ranges = std::min({std::max(kWorkgroups / c.slices, 1u), c.chunks, fit});
    c.sharers = 1;
    while (c.sharers < uint32_t(kWaves) && c.sharers * 128 < kChunk / c.slices) c.sharers *= 2;
    c.sum_bytes = align256(per_range * c.ranges);
    return c;
}

// A number as the input scan sees it: the largest finite magnitude (fp32 bits) and flags. SRC 1, 2: the bits of a 16-bit
// number; magnitudes of one 16-bit format order like their bits.
template <int SRC>
struct Scan {
    uint32_t m = 0, flags = 0;
    __device__ __forceinline__ void look(uint32_t w)
    {
        if constexpr (SRC == 0) {   // as scan_inputs_kernel
            const uint32_t a = w & 0x7fffffffu;
            const bool finite = a < 0x7f800000u;
            m = finite ? max(m, a) : m;
            const float v = __uint_as_float(w), back = float(_Float16(v));
            flags |= uint32_t((back != v && a >= 0x38800000u) || (a >= 0x47000000u)) | (finite ? 0u : 2u);
        } else {
            constexpr uint32_t kInf = SRC == 1 ? 0x7c00u : 0x7f80u;
            const uint32_t lo = w & 0x7fffu, hi = (w >> 16) & 0x7fffu;
            m = lo < kInf ? max(m, lo) : m;
            m = hi < kInf ? max(m, hi) : m;
            flags |= (lo < kInf && hi < kInf) ? 0u : 2u;
        }
    }
    __device__ __forceinline__ uint32_t absmax() const
    {
        if constexpr (SRC == 0) return m;
        else return __float_as_uint(SRC == 1 ? float(__builtin_bit_cast(_Float16, uint16_t(m))) : __uint_as_float(m << 16));
    }
};

// One chunk. FRESH: the input scan of its rows and codes. LISTED: its entries by slice, entries[chunk][..], the slices'
// starts within it in starts[chunk][slices + 1]; the order within a slice depends on scheduling, the sums do not. Codes >= K
// belong to no slice.
template <int D, int SRC, bool FRESH, bool LISTED>
__global__ __launch_bounds__(kChunkThreads) void slice_chunk_kernel(const void* __restrict__ X, const void* __restrict__ idx, uint32_t N, uint32_t K,
                                                               uint32_t slices, WsHeader* hdr, ScanPart* __restrict__ parts,
                                                               uint32_t* __restrict__ entries, uint32_t* __restrict__ starts)
{
    using S = Slice<D>;
    constexpr int U = kChunk / kChunkThreads;
    static_assert(kChunk % kChunkThreads == 0, "whole rounds");
    __shared__ uint32_t count[kCounters];
    __shared__ uint32_t sorted[LISTED ? kChunk : 1];
    __shared__ uint32_t total, red[3];
    const uint32_t first = blockIdx.x * kChunk, n = min(kChunk, N - first);
    // Counter of a code: by slice, then position, then lane; kGroups groups of positions, so that slices that work side by
    // side find each other's cache lines. While a 128-byte line holds more rows than there are slices (at most four of them:
    // the counters), the order of the rows is kept - a count per 64 positions, ranks by ballot: neighbours of a slice share
    // cache lines, and summing 20 M vectors of 4 numbers at K = 8192 takes 92 instead of 109 us, 28 M of 8 at K = 6000 232
    // instead of 265; the chunks take 5 more. With a row to a line it gives 2 us for those 5.
    const bool keep_order = slices <= 4 && slices * (D * (SRC == 0 ? 4 : 2)) < 128;
    const uint32_t log_lanes = keep_order ? 4u : 6 - (32 - __clz(slices - 1)), sub = threadIdx.x & ((1u << log_lanes) - 1);
    const uint32_t wave = threadIdx.x >> 6;
    static_assert(kCounters / kGroups == 64 && kGroups == 8, "slices x lanes");
    static_assert(kChunk / 64 <= kCounters / 4, "a count per 64 positions");
    auto counter = [&](uint32_t code, int u) {
        const uint32_t slice = code >> S::kBits;
        return keep_order ? (slice << 7) | (u * (kChunkThreads / 64) + wave) : (((slice << 3) | (u * kGroups / U)) << log_lanes) | sub;
    };
    uint32_t code[U], rank[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t p = u * kChunkThreads + threadIdx.x;
        code[u] = p < n ? code_at<SRC>(idx, size_t(first) + p) : 0xffffffffu;
    }
    for (uint32_t t = threadIdx.x; t < kCounters; t += kChunkThreads) count[t] = 0;
    if (threadIdx.x < 3) red[threadIdx.x] = 0;
    Scan<SRC> scan;
    if constexpr (FRESH) {
        // 16 bytes a load (8 where a 16-bit row has no more), a row's worth per code
        constexpr int W = D * (SRC == 0 ? 4 : 2) / 8;   // 8-byte pieces per row
        const uint2* rows = static_cast<const uint2*>(X) + size_t(first) * W;
        const uint32_t pieces = n * W;
        constexpr int V = 4;
        for (uint32_t i0 = 2 * threadIdx.x; i0 < pieces; i0 += 2 * V * kChunkThreads) {
            uint4 t[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const uint32_t i = i0 + 2 * v * kChunkThreads;
                t[v] = make_uint4(0u, 0u, 0u, 0u);
                if (i + 1 < pieces) {
                    t[v] = *reinterpret_cast<const uint4*>(rows + i);
                } else if (i < pieces) {
                    const uint2 last = rows[i];
                    t[v] = make_uint4(last.x, last.y, 0u, 0u);
                }
            }
#pragma unroll
            for (int v = 0; v < V; ++v) {
                scan.look(t[v].x);
                scan.look(t[v].y);
                scan.look(t[v].z);
                scan.look(t[v].w);
            }
        }
    }
    __syncthreads();
    uint32_t bad = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        rank[u] = 0;
        if (LISTED && keep_order) {
            const uint32_t slice = code[u] >> S::kBits;
            const unsigned long long valid = __ballot(code[u] < K), odd = __ballot(slice & 1), high = __ballot(slice & 2);
            auto members = [&](uint32_t q) { return valid & (q & 1 ? odd : ~odd) & (q & 2 ? high : ~high); };
            const unsigned long long of = members(slice);
            rank[u] = __builtin_amdgcn_mbcnt_hi(uint32_t(of >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(of), 0u));
            if ((threadIdx.x & 63) < slices)
                count[((threadIdx.x & 63) << 7) | (u * (kChunkThreads / 64) + wave)] = uint32_t(__popcll(members(threadIdx.x & 63)));
        } else if (LISTED && code[u] < K) {
            rank[u] = atomicAdd(&count[counter(code[u], u)], 1u);
        }
        if (code[u] >= K && u * kChunkThreads + threadIdx.x < n) ++bad;
    }
    if (bad) {
        if (FRESH) atomicAdd(&red[2], bad);
        else atomicAdd(&hdr->skipped_vectors, static_cast<unsigned long long>(bad));
    }
    if constexpr (FRESH) {
        uint32_t m = scan.m, flags = scan.flags;
        for (int off = 32; off > 0; off >>= 1) {
            m = max(m, uint32_t(__shfl_xor(int(m), off, 64)));
            flags |= uint32_t(__shfl_xor(int(flags), off, 64));
        }
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&red[0], m);
            if (flags) atomicOr(&red[1], flags);
        }
    }
    __syncthreads();
    if (FRESH && threadIdx.x == 0) {
        scan.m = red[0];
        parts[blockIdx.x] = ScanPart{scan.absmax(), red[1], red[2], 0u};
    }
    if constexpr (LISTED) {
        if (threadIdx.x < 64) {   // counts to places, eight counters per lane
            constexpr uint32_t kEach = kCounters / 64;
            uint32_t c[kEach], sum = 0;
#pragma unroll
            for (uint32_t q = 0; q < kEach; ++q) {
                c[q] = count[threadIdx.x * kEach + q];
                sum += c[q];
            }
            uint32_t upto = sum;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = uint32_t(__shfl_up(int(upto), off, 64));
                if (int(threadIdx.x) >= off) upto += o;
            }
            uint32_t at = upto - sum;
            if (threadIdx.x == 63) total = upto;
#pragma unroll
            for (uint32_t q = 0; q < kEach; ++q) {
                count[threadIdx.x * kEach + q] = at;
                at += c[q];
            }
        }
        __syncthreads();
        if (threadIdx.x <= slices)
            starts[size_t(blockIdx.x) * (slices + 1) + threadIdx.x] = threadIdx.x < slices ? count[(threadIdx.x * kGroups) << log_lanes] : total;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (code[u] < K)
                sorted[count[counter(code[u], u)] + rank[u]] =
                    ((code[u] & (S::kClusters - 1)) << kPosBits) | (u * kChunkThreads + threadIdx.x);
        }
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < total; t += kChunkThreads) entries[size_t(first) + t] = sorted[t];
    }
}

// (slice, range) of a workgroup. Workgroups are dealt to the 8 XCDs in turn; XCD q takes the q-th contiguous share of
// the jobs in range-major order, i.e. all slices of a few ranges: the workgroups that scan the same codes and fetch
// rows from the same cache lines (a 128-byte line holds rows of several slices) then share one L2, so every line
// comes from memory once instead of once per slice.
__device__ __forceinline__ bool job_of_workgroup(uint32_t slices, uint32_t ranges, uint32_t& slice, uint32_t& range)
{
    const uint32_t jobs = slices * ranges, per_xcd = (jobs + 7) / 8;
    const uint32_t job = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    slice = job % slices;
    range = job / slices;
    return job < jobs && blockIdx.x / 8 < per_xcd;
}

// LISTED: by entry lists; otherwise (one slice) the codes themselves, in their order.
template <int D, int SRC, bool LISTED>
__global__ __launch_bounds__(kThreads) void sliced_accumulate_kernel(const void* __restrict__ X, uint32_t N, const void* __restrict__ idx,
                                                                     uint32_t K, uint32_t slices, uint32_t chunks, uint32_t ranges,
                                                                     uint32_t sharers, WsHeader* hdr, const ScanPart* __restrict__ parts,
                                                                     const uint32_t* __restrict__ entries,
                                                                     const uint32_t* __restrict__ starts,
                                                                     unsigned long long* __restrict__ part_sums,
                                                                     uint32_t* __restrict__ part_counts)
{
    using S = Slice<D>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned long long* sum = reinterpret_cast<unsigned long long*>(smem);              // [D][kPitch]
    uint32_t* cnt = reinterpret_cast<uint32_t*>(smem + S::kSumBytes);                   // [kClusters]
    __shared__ uint32_t found[3];
    uint32_t slice, range;
    if (!job_of_workgroup(slices, ranges, slice, range)) return;  // uniform over the workgroup
    for (uint32_t t = threadIdx.x; t < S::kPitch * D; t += kThreads) sum[t] = 0;
    for (uint32_t t = threadIdx.x; t < S::kClusters; t += kThreads) cnt[t] = 0;
    if (threadIdx.x < 3) found[threadIdx.x] = 0;
    __syncthreads();

    const uint32_t k_n = min(S::kClusters, K - slice * S::kClusters);   // clusters of this slice
    uint32_t absmax, flags;
    if (parts != nullptr) {   // what the chunks found; the first workgroup leaves the call's bookkeeping
        uint32_t m = 0, f = 0, skipped = 0;
        for (uint32_t t = threadIdx.x; t < chunks; t += kThreads) {
            m = max(m, parts[t].absmax);
            f |= parts[t].flags;
            skipped += parts[t].skipped;
        }
        for (int off = 32; off > 0; off >>= 1) {
            m = max(m, uint32_t(__shfl_xor(int(m), off, 64)));
            f |= uint32_t(__shfl_xor(int(f), off, 64));
            skipped += uint32_t(__shfl_xor(int(skipped), off, 64));
        }
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&found[0], m);
            if (f) atomicOr(&found[1], f);
            if (skipped) atomicAdd(&found[2], skipped);
        }
        __syncthreads();
        absmax = found[0];
        flags = found[1];
        if (slice == 0 && range == 0 && threadIdx.x == 0) {
            WsHeader h{};
            h.absmax_bits = absmax;
            h.x_not_f16 = flags & 1u;
            h.x_nonfinite = flags >> 1;
            h.skipped_vectors = found[2];
            *hdr = h;
        }
    } else {
        absmax = hdr->absmax_bits;
        flags = hdr->x_nonfinite << 1;
    }
    const int e = fixed_point_exp(absmax, N);
    const bool finite = (flags & 2u) == 0;   // otherwise every number is looked at
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t bad = 0;
    constexpr int n = Piece<D, SRC>::kNumbers, P = Piece<D, SRC>::kLanes;
    constexpr int U = SRC == 0 && (D >= 8 || !LISTED) ? 2 : 1;   // rows a lane has under way: what measured better
    const uint32_t piece = lane % P, which = lane / P;   // this lane's part of a row, its row within a batch of 64 / P
    unsigned long long* mine = sum + piece * (n * S::kPitch);
    auto add = [&](const float (&x)[n], uint32_t c) {
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const long long v = finite ? fixed_point_finite(x[j], e) : fixed_point_term(x[j], e);
            atomicAdd(&mine[j * S::kPitch + c], static_cast<unsigned long long>(v));
        }
        if (piece == 0) atomicAdd(&cnt[c], 1u);
    };
    // Range r takes every ranges-th chunk, from the last one down - what the previous kernel read last is still in the
    // memory-side cache - kWaves / sharers of them at a time: the workgroups of all slices of a range then work within a
    // window of X that their L2 holds. The entries of a wave's next batch are requested before the rows of this one, and
    // those before the ones of the last are added.
    uint32_t done = range + ranges * (wave / sharers), first = 0, i0 = 0, end = 0;   // chunks above the current one
    const uint32_t step = ranges * (kWaves / sharers);
    auto open = [&]() {   // first batch at or after `done`
        for (; done < chunks; done += step) {
            const uint32_t chunk = chunks - 1 - done;
            const uint32_t* at = starts + size_t(chunk) * (slices + 1) + slice;
            first = chunk * kChunk;
            end = LISTED ? at[1] : min(kChunk, N - first);
            i0 = (LISTED ? at[0] : 0u) + wave % sharers * (U * 64 / P);
            if (i0 < end) return;
        }
    };
    auto load_entries = [&](uint32_t (&ent)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = min(i0 + u * (64 / P) + which, end - 1);
            ent[u] = LISTED ? entries[size_t(first) + i] : (min(code_at<SRC>(idx, size_t(first) + i), K) << kPosBits) | i;
        }
    };
    float pending[U][n];
    uint32_t cluster[U], ent[U];
    bool active[U];
#pragma unroll
    for (int u = 0; u < U; ++u) active[u] = false;
    open();
    if (done < chunks) load_entries(ent);
    auto commit = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (active[u]) add(pending[u], cluster[u]);
    };
    while (done < chunks) {
        size_t row[U];
        uint32_t c[U];
        bool on[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            row[u] = size_t(first) + (ent[u] & ((1u << kPosBits) - 1));
            c[u] = ent[u] >> kPosBits;
            on[u] = i0 + u * (64 / P) + which < end;
            if (!LISTED && on[u] && c[u] >= k_n) {
                on[u] = false;
                if (piece == 0) ++bad;
            }
        }
        i0 += sharers * (U * 64 / P);
        if (i0 >= end) {
            done += step;
            open();
        }
        if (done < chunks) load_entries(ent);
        float x[U][n];
#pragma unroll
        for (int u = 0; u < U; ++u) fetch_piece<D, SRC>(X, row[u], piece, x[u]);
        commit();
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int j = 0; j < n; ++j) pending[u][j] = x[u][j];
            cluster[u] = c[u];
            active[u] = on[u];
        }
    }
    commit();
    if (bad && parts == nullptr) atomicAdd(&hdr->skipped_vectors, static_cast<unsigned long long>(bad));
    __syncthreads();
    const size_t job = size_t(slice) * ranges + range;
    unsigned long long* ps = part_sums + job * (S::kPitch * D);
    uint32_t* pc = part_counts + job * S::kClusters;
#pragma unroll
    for (int j = 0; j < D; ++j)
        for (uint32_t t = threadIdx.x; t < k_n; t += kThreads) ps[j * S::kPitch + t] = sum[j * S::kPitch + t];
    for (uint32_t t = threadIdx.x; t < k_n; t += kThreads) pc[t] = cnt[t];
}

// Adds the ranges of every cluster (integers: any order gives the same bits; this one is fixed anyway), leaves the
// totals in the workspace and writes the means (or, mean = 0, the plain sums). An empty cluster keeps prev. A workgroup
// finishes 64 neighbouring clusters of one component, its waves take turns at the ranges (one thread per cluster and
// component waited 75 us for 256 ranges at K = 1024).
template <int D, int W>
__global__ __launch_bounds__(64 * W) void sliced_finalize_kernel(const unsigned long long* __restrict__ part_sums,
                                                                   const uint32_t* __restrict__ part_counts, uint32_t ranges,
                                                                   const float* prev, float* out, uint32_t* counts_out, uint32_t K,
                                                                   uint32_t N, WsHeader* hdr, int mean, long long* __restrict__ sums_ws,
                                                                   uint32_t* __restrict__ counts_ws)
{
    using S = Slice<D>;
    __shared__ long long red_sum[W][64];
    __shared__ uint32_t red_count[W][64];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, groups = (K + 63) / 64;
    const uint32_t j = blockIdx.x / groups, k = (blockIdx.x % groups) * 64 + lane;
    const int e = fixed_point_exp(hdr->absmax_bits, N);
    if (blockIdx.x == 0 && threadIdx.x == 0) hdr->fixed_point_exp = e;
    const uint32_t slice = k / S::kClusters, local = k % S::kClusters;
    long long isum = 0;
    uint32_t n = 0;
    if (k < K) {
#pragma unroll 4
        for (uint32_t r = wave; r < ranges; r += W) {
            const size_t job = size_t(slice) * ranges + r;
            isum += static_cast<long long>(part_sums[job * (S::kPitch * D) + j * S::kPitch + local]);
            n += part_counts[job * S::kClusters + local];
        }
    }
    red_sum[wave][lane] = isum;
    red_count[wave][lane] = n;
    __syncthreads();
    if (wave != 0 || k >= K) return;
#pragma unroll
    for (int v = 1; v < W; ++v) {
        isum += red_sum[v][lane];
        n += red_count[v][lane];
    }
    const size_t o = size_t(k) * D + j;
    sums_ws[o] = isum;
    if (j == 0) {
        counts_ws[k] = n;
        if (counts_out != nullptr) counts_out[k] = n;
    }
    const double total = ldexp(double(isum), -e);
    out[o] = !mean ? float(total) : (n > 0 ? float(total / double(n)) : prev[o]);
}

template <int D, int SRC, bool LISTED>
hipError_t launch_t(const Cut& c, const void* X, uint32_t N, const void* idx, const float* prev, uint32_t K, float* out,
                    uint32_t* counts_out, const Workspace& w, bool mean, bool fresh, hipStream_t s)
{
    using S = Slice<D>;
    const uint32_t jobs = c.slices * c.ranges;
    unsigned long long* part_sums = reinterpret_cast<unsigned long long*>(w.records);
    uint32_t* part_counts = reinterpret_cast<uint32_t*>(w.records + size_t(jobs) * S::kSumBytes);
    ScanPart* parts = reinterpret_cast<ScanPart*>(w.records + c.sum_bytes);
    uint32_t* entries = reinterpret_cast<uint32_t*>(w.records + c.sum_bytes + c.part_bytes);
    uint32_t* starts = reinterpret_cast<uint32_t*>(w.records + c.sum_bytes + c.part_bytes + c.entry_bytes);
    // per call: the attribute belongs to the current device
    if (const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sliced_accumulate_kernel<D, SRC, LISTED>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(S::kLdsBytes)); e != hipSuccess)
        return e;
    if (fresh)
        hipLaunchKernelGGL((slice_chunk_kernel<D, SRC, true, LISTED>), dim3(c.chunks), dim3(kChunkThreads), 0, s, X, idx, N, K, c.slices, w.hdr,
                           parts, entries, starts);
    else if constexpr (LISTED && SRC == 0)
        hipLaunchKernelGGL((slice_chunk_kernel<D, SRC, false, true>), dim3(c.chunks), dim3(kChunkThreads), 0, s, X, idx, N, K, c.slices, w.hdr,
                           parts, entries, starts);
    hipLaunchKernelGGL((sliced_accumulate_kernel<D, SRC, LISTED>), dim3(8 * ((jobs + 7) / 8)), dim3(kThreads), S::kLdsBytes, s, X, N, idx,
                       K, c.slices, c.chunks, c.ranges, c.sharers, w.hdr, fresh ? parts : nullptr, entries, starts, part_sums, part_counts);
    const dim3 done((K + 63) / 64 * D);
    if (c.ranges > 32)
        hipLaunchKernelGGL((sliced_finalize_kernel<D, 16>), done, dim3(1024), 0, s, part_sums, part_counts, c.ranges, prev, out,
                           counts_out, K, N, w.hdr, mean ? 1 : 0, w.sums, w.counts);
    else
        hipLaunchKernelGGL((sliced_finalize_kernel<D, 4>), done, dim3(256), 0, s, part_sums, part_counts, c.ranges, prev, out,
                           counts_out, K, N, w.hdr, mean ? 1 : 0, w.sums, w.counts);
    return hipGetLastError();
}

template <int D, int SRC>
hipError_t update_sliced_t(const void* X, uint32_t N, const void* idx, const float* prev, uint32_t K, float* out,
                           uint32_t* counts_out, const Workspace& w, bool mean, bool fresh, hipStream_t s)
{
    const Cut c = cut_of<D>(N, K);
    return c.listed ? launch_t<D, SRC, true>(c, X, N, idx, prev, K, out, counts_out, w, mean, fresh, s)
                    : launch_t<D, SRC, false>(c, X, N, idx, prev, K, out, counts_out, w, mean, fresh, s);
}

}  // namespace

// Whether the M-step by slices applies: not to so few vectors that three launches with a workgroup per 7168 of them take
// longer than atomics, nor where the record buffer does not hold one range of partial sums (far fewer vectors than centroids).
bool update_sliced_applies(uint32_t N, uint32_t d, uint32_t K, const Workspace& w)
{
    if (!w.bucket_ok || w.records == nullptr || N < kLeast) return false;
    return (d == 4 ? cut_of<4>(N, K).ranges : (d == 8 ? cut_of<8>(N, K).ranges : cut_of<16>(N, K).ranges)) > 0;
}

// `out` may alias `prev`; `out` must not alias X. Sums and counts are left in w.sums / w.counts. fresh: no input scan has run
// since the call began; this one leaves the header as a reset and a scan would.
hipError_t launch_update_sliced(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, const float* prev, uint32_t K,
                                float* out, uint32_t* counts_out, const Workspace& w, bool mean, bool fresh, hipStream_t s)
{
    if (!update_sliced_applies(N, d, K, w)) return hipErrorInvalidValue;
    switch (d) {
        case 4: return update_sliced_t<4, 0>(X, N, idx, prev, K, out, counts_out, w, mean, fresh, s);
        case 8: return update_sliced_t<8, 0>(X, N, idx, prev, K, out, counts_out, w, mean, fresh, s);
        case 16: return update_sliced_t<16, 0>(X, N, idx, prev, K, out, counts_out, w, mean, fresh, s);
        default: return hipErrorInvalidValue;
    }
}

// The sums (not the means) of 16-bit rows by 16-bit code, read in place: rows [N * d] fp16 (dtype 1) or bf16 (2),
// 16-byte aligned; codes [N], 4-byte aligned. Leaves the header as a reset and a
// scan of the rows would. Same fixed-point sums as launch_update on the converted rows: same bits.
hipError_t launch_sum_rows16_sliced(const void* rows, int dtype, uint32_t N, uint32_t d, const uint16_t* codes, uint32_t K,
                                    float* out, const Workspace& w, hipStream_t s)
{
    if (!update_sliced_applies(N, d, K, w) || (dtype != 1 && dtype != 2)) return hipErrorInvalidValue;
    const bool bf = dtype == 2;
    switch (d) {
        case 4: return bf ? update_sliced_t<4, 2>(rows, N, codes, nullptr, K, out, nullptr, w, false, true, s)
                          : update_sliced_t<4, 1>(rows, N, codes, nullptr, K, out, nullptr, w, false, true, s);
        case 8: return bf ? update_sliced_t<8, 2>(rows, N, codes, nullptr, K, out, nullptr, w, false, true, s)
                          : update_sliced_t<8, 1>(rows, N, codes, nullptr, K, out, nullptr, w, false, true, s);
        case 16: return bf ? update_sliced_t<16, 2>(rows, N, codes, nullptr, K, out, nullptr, w, false, true, s)
                           : update_sliced_t<16, 1>(rows, N, codes, nullptr, K, out, nullptr, w, false, true, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cc
