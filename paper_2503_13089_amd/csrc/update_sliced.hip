// M-step by cluster slices (Section 3.1: c_k <- mean of the vectors assigned to cluster k), for many vectors and
// K <= 65536: two passes over the codes; no copy of the vectors but the 16-bit one below.
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
// Rows of 8 to 32 bytes go along (record_chunk_kernel): what a chunk leaves for a slice are its rows as 16-bit numbers, read back in
// sequence, instead of entries that name rows to be fetched from a line each. Taken for 16-bit gradients (records_pay says which) and for fp32 vectors of 4
// whose chunk holds fp16 or bf16 numbers only (a compressed model's weights do); a chunk of other numbers leaves entries. fp32 vectors
// of 8 and 16 keep the entries: at 32 bytes a row the second read costs less than writing the rows (28 M of 8 500 us with entries, 526
// with rows).
//
// Bound, rows along: the passes over memory (chunk kernel 5.6 TB/s, 40 us for the gradient of 4096x11008, 55 for 11.3 M vectors of 4), then
// the records from memory (25 us) beside the LDS atomics (11 clocks a wave, 14 us). A number's fixed-point term took 14 vector instructions (26 us); numbers of 16 bits have
// at most 30 bits above a unit that nearly all share, which takes 6 (a wave's step that has another takes the 14): with that and the records of two steps under way
// 11.3 M vectors of 4 99.7 -> 96.2 us a call, the gradient 77.1 -> 74.9. By entries, where rows come a line each, that was no faster. Slices of 2048 clusters at d = 4 then, half the partial sums of 4096. By entries: one row fetch per
// vector from a different cache line each - the L1 fill rate - or, with few slices, the two passes over the rows.
// By entries / rows along, us a call, fp32 vectors of 4; numbers of fp16 or bf16 / of neither: 2 M, K = 12000 46 / 39 / 38; 11.3 M, K = 65536 126 / 105 / 120;
// 20 M, K = 8192 182 / 154 / 188, K = 65536 231 / 159 / 226. 16-bit gradients through an fp32 copy / rows along: 4096x11008 g = 6 344 / 143, g = 9 458 / 187.
// By entries only: 28 M of 8 at K = 65536 500 us, 6 M of 16 at K = 3000 189; one slice: 11.5 M of 4 at K = 300 106.
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
// Vectors sorted together. Records hold 10 (d = 4) to 34 bytes each in LDS, and this leaves room for two to four chunks on a compute unit.
template <int D, int RECORDS>
constexpr uint32_t kChunkOf = RECORDS ? (D == 16 ? 1792 : 3584) : 7168;
template <int D, int RECORDS>
constexpr int kChunkThreadsOf = RECORDS ? int(kChunkOf<D, 1> / 7) : kChunkThreads;
constexpr uint32_t kPosBits = 13;
constexpr uint32_t kKindShift = 16, kStartMask = 0xffffu;   // where a slice starts in a chunk, and above it what the chunk left
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
template <int D, int RECORDS = 0>
struct Slice {
    static constexpr uint32_t kBits = D == 4 ? (RECORDS == 1 ? 11u : 12u) : (D == 8 ? 11u : 10u);
    static constexpr uint32_t kClusters = 1u << kBits;
    // sums of one component lie side by side; the two extra keep the lanes that share a row off one bank
    static constexpr uint32_t kPitch = kClusters + 2;
    static constexpr uint32_t kSumBytes = kPitch * D * 8;
    static constexpr uint32_t kLdsBytes = kSumBytes + kClusters * 4;
    static_assert((65536u >> kBits) <= 64u && kBits + kPosBits <= 32u, "a lane per slice; an entry in 32 bits");
};

// What the input scan found in one chunk, and its codes >= K.
struct ScanPart {
    uint32_t absmax, flags, skipped, pad;   // flags: bit 0 = not fit for the fp16 kernels, bit 1 = a non-finite input, kLeftEntries
};
constexpr uint32_t kLeftEntries = 4;   // the rows of this chunk could not go along
// What lies in a chunk's part of the entry buffer, told beside where its slices start: entries (32 bits each), or the rows themselves as fp16
// or bf16 numbers by slice, followed by their clusters within the slice (16 bits).
enum Kind : uint32_t { kEntries = 0, kRowsF16 = 1, kRowsBf16 = 2 };
template <int D>
constexpr uint32_t kRecordBytes = 2 * D + 2;
template <int D>
constexpr int kRecordRows = 2;   // a lane has under way twice
template <int D>
constexpr uint32_t kRecordStep = kRecordRows<D> * (D == 16 ? 32 : 64);   // rows of a wave at once

struct Cut {
    bool listed;
    uint32_t slices, chunks, ranges;
    uint32_t sharers;         // waves that share a chunk's entries, or rows
    uint32_t entry_sharers;   // entries of a chunk whose rows could not go along
    size_t sum_bytes, part_bytes, entry_bytes, start_bytes;
};

// The record buffer (2 N records) holds it all; ranges = 0: not even one range of partial sums fits.
template <int D, int RECORDS = 0>
Cut cut_of(uint32_t N, uint32_t K)
{
    constexpr uint32_t kChunk = kChunkOf<D, RECORDS>;
    const size_t have = size_t(N) * 2 * (4 * D + 16);
    Cut c;
    c.listed = RECORDS || !update_one_slice(D, K);
    using S = Slice<D, RECORDS>;
    static_assert(Slice<D>::kClusters == 16384 / D);
    c.slices = (K + S::kClusters - 1) / S::kClusters;
    c.chunks = uint32_t((uint64_t(N) + kChunk - 1) / kChunk);
    c.part_bytes = align256(size_t(c.chunks) * sizeof(ScanPart));
    c.entry_bytes = c.listed ? align256(size_t(c.chunks) * kChunk * (RECORDS ? kRecordBytes<D> : 4)) : 0;
    c.start_bytes = c.listed ? align256(size_t(c.chunks) * (c.slices + 1) * 4) : 0;
    const size_t taken = c.part_bytes + c.entry_bytes + c.start_bytes + 256, per_range = size_t(c.slices) * S::kLdsBytes;
    const uint32_t fit = uint32_t(have > taken ? std::min<size_t>((have - taken) / per_range, kWorkgroups) : 0);
    c.ranges = std::min({std::max(kWorkgroups / c.slices, 1u), c.chunks, fit});
    c.sharers = 1;
    while (c.sharers < uint32_t(kWaves) && c.sharers * (RECORDS ? kRecordStep<D> : 128u) < kChunk / c.slices) c.sharers *= 2;
    // With as many waves to the entries of these shorter chunks as to their rows each had one batch of 64, and waited for where they begin as often as
    // for them (11.3 M vectors, K = 12000: the sums 65 us instead of 55).
    c.entry_sharers = RECORDS ? 1 : c.sharers;
    while (RECORDS && c.entry_sharers < uint32_t(kWaves) && c.entry_sharers * 512 < kChunk / c.slices) c.entry_sharers *= 2;
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

// The same in fewer instructions, of numbers that are all finite: otherwise flag 1 is set and Scan has to look again. fp32 numbers
// come with their fp16 neighbour; flag 2: one is no fp16 number, flag 3: one is no bf16 number.
template <int SRC>
struct RowScan {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    uint32_t m = 0, strange = 0, bits = 0;   // largest magnitude, that of those that are no fp16 numbers, the OR of all
    __device__ __forceinline__ void look(uint32_t w, float back)
    {
        if constexpr (SRC == 0) {
            const uint32_t a = w & 0x7fffffffu;
            m = max(m, a);
            strange = max(strange, back != __uint_as_float(w) ? a : 0u);
            bits |= w;
        } else {   // both halves at once
            const uint32_t a = w & 0x7fff7fffu;
            m = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m), __builtin_bit_cast(u16x2, a)));
        }
    }
    __device__ __forceinline__ uint32_t largest() const { return SRC == 0 ? m : max(m & 0xffffu, m >> 16); }
    __device__ __forceinline__ uint32_t flags() const
    {
        if constexpr (SRC != 0) return largest() < (SRC == 1 ? 0x7c00u : 0x7f80u) ? 0u : 2u;
        return uint32_t(strange >= 0x38800000u || m >= 0x47000000u) | (m < 0x7f800000u ? 0u : 2u) | (strange != 0 ? 4u : 0u) |
               ((bits & 0xffffu) != 0 ? 8u : 0u);
    }
};

// Counts to places, by one wave, eight counters per lane.
__device__ __forceinline__ void counts_to_places(uint32_t* count, uint32_t& total)
{
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

// One chunk. FRESH: the input scan of its rows and codes. LISTED: its entries by slice, entries[chunk][..], the slices'
// starts within it in starts[chunk][slices + 1]; the order within a slice depends on scheduling, the sums do not. Codes >= K
// belong to no slice.
template <int D, int SRC, bool FRESH, bool LISTED>
__global__ __launch_bounds__(kChunkThreads) void slice_chunk_kernel(const void* __restrict__ X, const void* __restrict__ idx, uint32_t N, uint32_t K,
                                                               uint32_t slices, WsHeader* hdr, ScanPart* __restrict__ parts,
                                                               uint32_t* __restrict__ entries, uint32_t* __restrict__ starts)
{
    using S = Slice<D>;
    constexpr uint32_t kChunk = kChunkOf<D, false>;
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
        if (threadIdx.x < 64) counts_to_places(count, total);
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

// Where the rows of a layer's gradient lie: row v = (r, c) of codes [in][per_row] at r * out_features + c * g, the last of every
// r less `padding` numbers. per_row = 0: whole rows of D numbers side by side.
struct RowPlace {
    uint32_t per_row, g, padding;
};

// One chunk whose rows go along: as slice_chunk_kernel<FRESH, LISTED>, but what it leaves for a slice are the rows themselves,
// 16-bit numbers, and their clusters. fp32 rows (SRC 0) do where all numbers of the chunk are fp16 numbers, or all of them bf16 ones;
// a chunk of others leaves entries. The rows are read once, coalesced, and held in registers until their places are known.
template <int D, int SRC, bool WHOLE, int RECORDS>
__global__ __launch_bounds__((kChunkThreadsOf<D, 1>), (D == 8 ? 4 : 1)) void record_chunk_kernel(const void* __restrict__ X, const void* __restrict__ idx, uint32_t N,
                                                                                uint32_t K, uint32_t slices, RowPlace place,
                                                                                ScanPart* __restrict__ parts, char* __restrict__ records,
                                                                                uint32_t* __restrict__ starts)
{
    using S = Slice<D, RECORDS>;
    constexpr uint32_t kChunk = kChunkOf<D, 1>, T = kChunkThreadsOf<D, 1>;
    constexpr int U = kChunk / T;
    static_assert(kChunk % T == 0 && (SRC != 0 || (WHOLE && D == 4)), "whole rounds");
    typedef uint32_t Words __attribute__((ext_vector_type(D == 4 ? 2 : 4)));   // a piece of a record
    constexpr int kPieces = D == 16 ? 2 : 1;
    __shared__ uint32_t count[kCounters];
    __shared__ __attribute__((aligned(16))) char sorted[kChunk * kRecordBytes<D>];
    __shared__ uint32_t total, red[3];
    const uint32_t first = blockIdx.x * kChunk, n = min(kChunk, N - first);
    const uint32_t log_lanes = slices == 1 ? 6u : 6 - (32 - __clz(slices - 1)), sub = threadIdx.x & ((1u << log_lanes) - 1);
    uint32_t some = 0;   // the numbers of four rows, a lane each
    if constexpr (SRC == 0) {
        const uint32_t q = (threadIdx.x & 63) / 4 % 4;
        some = static_cast<const uint32_t*>(X)[size_t(uint64_t(N) * q / 4) * D + (threadIdx.x & 3)];
    }
    constexpr int kWords = SRC == 0 ? D : D / 2;
    uint32_t code[U], rank[U], raw[U][kWords];   // the numbers as they are
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t p = u * T + threadIdx.x;
        code[u] = p < n ? code_at<SRC>(idx, size_t(first) + p) : 0xffffffffu;
    }
    for (uint32_t t = threadIdx.x; t < kCounters; t += T) count[t] = 0;
    if (threadIdx.x < 3) red[threadIdx.x] = 0;
    // past the end the last row once more, which finds nothing new and belongs to no slice
    auto row_at = [&](int u) { return size_t(first) + min(uint32_t(u * T + threadIdx.x), n - 1); };
    RowScan<SRC> scan;
    if constexpr (SRC == 0) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        auto rows = [&](auto load) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < D / 4; ++q) {
                    const u32x4 t = load(static_cast<const u32x4*>(X) + row_at(u) * (D / 4) + q);
#pragma unroll
                    for (int j = 0; j < 4; ++j) raw[u][4 * q + j] = t[j];
                }
        };
        // Rows that go along are read past the caches, which leaves those to the records (11.3 M vectors from memory 131 us a call, otherwise 160); rows of other numbers
        // are read again soon (from the caches 119, otherwise 140). Which it will be, a few numbers tell well enough, the same for every workgroup.
        const bool sixteen = __all(float(_Float16(__uint_as_float(some))) == __uint_as_float(some) || (some & 0xffffu) == 0);
        if (sixteen) {
            asm volatile("");   // else the compiler makes one plain load of the two
            rows([](const u32x4* p) { return __builtin_nontemporal_load(p); });
            asm volatile("");
        } else {
            rows([](const u32x4* p) { return *p; });
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < D; ++j) scan.look(raw[u][j], float(_Float16(__uint_as_float(raw[u][j]))));
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (WHOLE) {
                constexpr int A = D * 2 < 16 ? D * 2 : 16;
                __builtin_memcpy(raw[u], __builtin_assume_aligned(static_cast<const uint32_t*>(X) + row_at(u) * (D / 2), A), D * 2);
            } else {
                const uint32_t v = uint32_t(row_at(u)), r = v / place.per_row;
                const uint32_t keep = v - r * place.per_row == place.per_row - 1 ? place.g - place.padding : place.g;
                const uint16_t* from = static_cast<const uint16_t*>(X) + (size_t(v) * place.g - size_t(r) * place.padding);
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const uint32_t half = uint32_t(j) < place.g ? from[min(uint32_t(j), keep - 1)] : 0u;
                    const uint32_t kept = uint32_t(j) < keep ? half : 0u;
                    raw[u][j / 2] = j & 1 ? raw[u][j / 2] | kept << 16 : kept;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < D / 2; ++q) scan.look(raw[u][q], 0.0f);
    }
    __syncthreads();   // counters and reductions are clear
    uint32_t m = scan.largest(), flags = scan.flags();
    if (flags & 2u) {   // what is not finite has no magnitude
        Scan<SRC> again;
        if constexpr (SRC == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < D; ++j) again.look(raw[u][j]);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < D / 2; ++q) {
                    again.look(raw[u][q]);
                    constexpr uint32_t kInf = SRC == 1 ? 0x7c00u : 0x7f80u;   // such numbers add nothing
                    raw[u][q] &= ((raw[u][q] & kInf) == kInf ? 0u : 0xffffu) | (((raw[u][q] >> 16) & kInf) == kInf ? 0u : 0xffff0000u);
                }
        }
        m = again.m;
        flags |= again.flags;
    }
    for (int off = 32; off > 0; off >>= 1) {
        m = max(m, uint32_t(__shfl_xor(int(m), off, 64)));
        flags |= uint32_t(__shfl_xor(int(flags), off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&red[0], m);
        if (flags) atomicOr(&red[1], flags);
    }
    __syncthreads();
    const uint32_t found = red[1];
    const uint32_t kind = SRC != 0 ? uint32_t(SRC) : ((found & 2u) ? kEntries : (!(found & 4u) ? kRowsF16 : (!(found & 8u) ? kRowsBf16 : kEntries)));
    // As in slice_chunk_kernel the entries of few slices stay in the order of the rows.
    const bool keep_order = SRC == 0 && kind == kEntries && slices <= 8;
    static_assert(SRC != 0 || (kChunk / 64 <= 64 && kCounters == 8 * 64), "a count per slice and 64 positions");
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto counter = [&](uint32_t code, int u) {
        const uint32_t slice = code >> S::kBits;
        return keep_order ? (slice << 6) | (u * (T / 64) + wave) : (((slice << 3) | (u * kGroups / U)) << log_lanes) | sub;
    };
    uint32_t bad = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        rank[u] = 0;
        if (keep_order) {
            const uint32_t slice = code[u] >> S::kBits;
            const unsigned long long valid = __ballot(code[u] < K), b0 = __ballot(slice & 1), b1 = __ballot(slice & 2), b2 = __ballot(slice & 4);
            auto members = [&](uint32_t q) { return valid & (q & 1 ? b0 : ~b0) & (q & 2 ? b1 : ~b1) & (q & 4 ? b2 : ~b2); };
            const unsigned long long same = members(slice);
            rank[u] = __builtin_amdgcn_mbcnt_hi(uint32_t(same >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(same), 0u));
            if (lane < 8) count[(lane << 6) | (u * (T / 64) + wave)] = uint32_t(__popcll(members(lane)));
        } else if (code[u] < K) {
            rank[u] = atomicAdd(&count[counter(code[u], u)], 1u);
        }
        if (code[u] >= K && u * T + threadIdx.x < n) ++bad;
    }
    if (bad) atomicAdd(&red[2], bad);
    __syncthreads();
    if (threadIdx.x == 0) {
        Scan<SRC> whole;
        whole.m = red[0];
        parts[blockIdx.x] = ScanPart{whole.absmax(), (found & 3u) | (kind == kEntries ? kLeftEntries : 0u), red[2], 0u};
    }
    if (threadIdx.x < 64) counts_to_places(count, total);
    __syncthreads();
    const uint32_t members = total;
    if (threadIdx.x <= slices)   // the first counter of a slice
        starts[size_t(blockIdx.x) * (slices + 1) + threadIdx.x] =
            (threadIdx.x < slices ? count[keep_order ? threadIdx.x << 6 : (threadIdx.x * kGroups) << log_lanes] : members) | kind << kKindShift;
    char* out = records + size_t(blockIdx.x) * (kChunk * kRecordBytes<D>);
    uint16_t* clusters = reinterpret_cast<uint16_t*>(sorted + kChunk * (2 * D));
    if (SRC == 0 && kind == kEntries) {
        uint32_t* at = reinterpret_cast<uint32_t*>(sorted);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (code[u] < K) at[count[counter(code[u], u)] + rank[u]] = ((code[u] & (S::kClusters - 1)) << kPosBits) | (u * T + threadIdx.x);
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < members; t += T) reinterpret_cast<uint32_t*>(out)[t] = at[t];
        return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (code[u] >= K) continue;
        const uint32_t at = count[counter(code[u], u)] + rank[u];
        uint32_t row[D / 2];
#pragma unroll
        for (int q = 0; q < D / 2; ++q) {
            if constexpr (SRC != 0) {
                row[q] = raw[u][q];
            } else if (kind == kRowsBf16) {
                row[q] = (raw[u][2 * q] >> 16) | (raw[u][2 * q + 1] & 0xffff0000u);
            } else {
                const _Float16 lo = _Float16(__uint_as_float(raw[u][2 * q])), hi = _Float16(__uint_as_float(raw[u][2 * q + 1]));
                row[q] = uint32_t(__builtin_bit_cast(uint16_t, lo)) | uint32_t(__builtin_bit_cast(uint16_t, hi)) << 16;
            }
        }
        __builtin_memcpy(__builtin_assume_aligned(sorted + at * (2 * D), D == 4 ? 8 : 16), row, 2 * D);
        clusters[at] = uint16_t(code[u] & (S::kClusters - 1));
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < members * kPieces; t += T)
        __builtin_nontemporal_store(reinterpret_cast<const Words*>(sorted)[t], reinterpret_cast<Words*>(out) + t);   // 112 MB, 20 M vectors 190 -> 179 us
    for (uint32_t t = threadIdx.x; t < (members + 1) / 2; t += T)   // the last one may bring a number that nobody reads
        reinterpret_cast<uint32_t*>(out + kChunk * (2 * D))[t] = reinterpret_cast<const uint32_t*>(clusters)[t];
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

// The records of a slice in the chunks of a range, added into the accumulators. A unit of a wave is its share of one chunk's run;
// where the runs begin is loaded for 64 units at once, a lane each, and the records of the next step (kStep rows) before those of
// this one are added.
template <int D, int SRC, int RECORDS>
__device__ __forceinline__ void add_records(unsigned long long* sum, uint32_t* cnt, int e, ShortTerms st, uint32_t slice, uint32_t slices,
                                            uint32_t range, uint32_t ranges, uint32_t chunks, uint32_t sharers,
                                            const char* __restrict__ records, const uint32_t* __restrict__ starts)
{
    using S = Slice<D, RECORDS>;
    constexpr uint32_t kChunk = kChunkOf<D, 1>;
    constexpr int n = D < 8 ? D : 8, P = D / n, U = kRecordRows<D>;   // numbers of a lane, lanes of a row, rows of a lane
    constexpr uint32_t R = 64 / P, kStep = U * R;
    static_assert(kStep == kRecordStep<D>);
    typedef uint32_t Words __attribute__((ext_vector_type(n / 2)));
    const uint32_t lane = threadIdx.x & 63, wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    const uint32_t piece = lane % P, which = lane / P;
    unsigned long long* mine = sum + piece * (n * S::kPitch);
    const uint32_t share = wave % sharers, per_round = ranges * (kWaves / sharers);   // chunks that all waves take in one round
    uint32_t upto = range + ranges * (wave / sharers);   // chunks above the current one
    // the runs of the next 64 chunks of this wave, a lane each
    uint32_t run_begin = 0, run_end = 0, run_kind = 0, left = 64;
    auto look_ahead = [&]() {
        const uint64_t mine_done = uint64_t(upto) + uint64_t(per_round) * lane;
        run_begin = run_end = 0;
        if (mine_done < chunks) {
            const uint32_t chunk = chunks - 1 - uint32_t(mine_done);
            const uint32_t* at = starts + size_t(chunk) * (slices + 1) + slice;
            const uint32_t from = at[0], to = at[1];
            run_kind = from >> kKindShift;
            run_begin = from & kStartMask;
            run_end = run_kind == kEntries ? run_begin : to & kStartMask;
        }
    };
    look_ahead();
    uint32_t at = 0, end = 0, kind = 0, chunk = 0;   // the next rows of this wave's share: at, at + sharers kStep, ..
    uint32_t last_at = 0, last_end = 0;
    auto next = [&]() {   // false: no rows left
        last_at = at;
        last_end = end;
        at += sharers * kStep;
        while (at >= end) {
            if (left == 0) {
                look_ahead();
                left = 64;
            }
            if (upto >= chunks) {   // the rows of before stay the ones to look at
                at = last_at;
                end = last_end;
                return false;
            }
            const int l = int(64 - left);
            chunk = uint32_t(__builtin_amdgcn_readfirstlane(int(chunks - 1 - upto)));
            at = uint32_t(__builtin_amdgcn_readlane(int(run_begin), l)) + share * kStep;
            end = uint32_t(__builtin_amdgcn_readlane(int(run_end), l));
            kind = uint32_t(__builtin_amdgcn_readlane(int(run_kind), l));
            --left;
            upto = chunks - upto > per_round ? upto + per_round : chunks;
        }
        return true;
    };
    struct Step {
        Words w[U];
        uint32_t cluster[U], rows, kind;
    };
    // Always four (2 U) requests, of the last rows once more where none are left: the counts of the waits then hold on every path.
    auto load = [&](Step& s, bool more) {
        const char* base = records + size_t(chunk) * (kChunk * kRecordBytes<D>);
        s.rows = more ? min(end - at, kStep) : 0u;
        s.kind = kind;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = min(at + u * R + which, end - 1);
            s.w[u] = reinterpret_cast<const Words*>(base)[i * P + piece];
            s.cluster[u] = reinterpret_cast<const uint16_t*>(base + kChunk * (2 * D))[i];
        }
    };
    auto add_kind = [&](const Step& s, auto bf16) {
        float x[U][n], t[U][n];
        uint32_t fractions = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < n; ++j) {
                const uint32_t w = s.w[u][j / 2];
                x[u][j] = decltype(bf16)::value ? __uint_as_float(j & 1 ? w & 0xffff0000u : w << 16)
                                                : float(__builtin_bit_cast(_Float16, uint16_t(j & 1 ? w >> 16 : w)));
                t[u][j] = x[u][j] * st.scale;
                fractions |= not_whole(t[u][j]);
            }
        auto put = [&](auto shorts) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u * R + which >= s.rows) continue;
#pragma unroll
                for (int j = 0; j < n; ++j)
                    atomicAdd(&mine[j * S::kPitch + s.cluster[u]],
                              decltype(shorts)::value ? short_term(t[u][j], st.k) : static_cast<unsigned long long>(fixed_point_finite(x[u][j], e)));
                if (SRC == 0 && piece == 0) atomicAdd(&cnt[s.cluster[u]], 1u);
            }
        };
        if (__any(fractions != 0)) put(std::false_type{});
        else put(std::true_type{});
    };
    auto add = [&](const Step& s) {
        if (s.rows == 0) return;   // nor a wait for its requests
        if (SRC == 2 || (SRC == 0 && s.kind == kRowsBf16)) add_kind(s, std::true_type{});
        else add_kind(s, std::false_type{});
    };
    end = 0;
    at = 0u - sharers * kStep;   // next() begins with a step
    if (!next()) return;
    Step a, b;
    load(a, true);
    // Two steps ahead; a wave of one step asks for no other. Calls whose waves have a few steps, us, all steps asked for and added / now: 99468 vectors of 4, K = 10680 20.4 / 19.4,
    // 250245, K = 4179 21.8 / 21.3, 16-bit gradient of 512 x 512 at K = 8000 15.9 / 15.3.
    Step c;
    bool more = next();
    if (!more) {
        add(a);
        return;
    }
    load(b, true);
    do {
        more = more && next();
        load(c, more);
        add(a);
        more = more && next();
        load(a, more);
        add(b);
        more = more && next();
        load(b, more);
        add(c);
    } while (more);
    add(a);
    add(b);
}

// LISTED: by entry lists; otherwise (one slice) the codes themselves, in their order. RECORDS: by what record_chunk_kernel left (2: in wide slices).
template <int D, int SRC, bool LISTED, int RECORDS>
__global__ __launch_bounds__(kThreads) void sliced_accumulate_kernel(const void* __restrict__ X, uint32_t N, const void* __restrict__ idx,
                                                                     uint32_t K, uint32_t slices, uint32_t chunks, uint32_t ranges,
                                                                     uint32_t sharers, uint32_t entry_sharers, WsHeader* hdr,
                                                                     const ScanPart* __restrict__ parts, const uint32_t* __restrict__ entries,
                                                                     const uint32_t* __restrict__ starts,
                                                                     unsigned long long* __restrict__ part_sums,
                                                                     uint32_t* __restrict__ part_counts)
{
    using S = Slice<D, RECORDS>;
    constexpr uint32_t kChunk = kChunkOf<D, RECORDS>;
    constexpr bool kCounted = SRC == 0;   // the gradient's sums need no numbers of members
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
            h.x_nonfinite = flags >> 1 & 1u;
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
    if constexpr (RECORDS)
        add_records<D, SRC, RECORDS>(sum, cnt, e, short_terms(absmax, e), slice, slices, range, ranges, chunks, sharers,
                            reinterpret_cast<const char*>(entries), starts);
    uint32_t bad = 0;
    auto add_entries = [&](auto all_finite) {
    constexpr int n = Piece<D, SRC>::kNumbers, P = Piece<D, SRC>::kLanes;
    constexpr int U = SRC == 0 && (D >= 8 || !LISTED) ? 2 : 1;   // rows a lane has under way: what measured better
    const uint32_t piece = lane % P, which = lane / P;   // this lane's part of a row, its row within a batch of 64 / P
    unsigned long long* mine = sum + piece * (n * S::kPitch);
    auto add = [&](const float (&x)[n], uint32_t c) {
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const long long v = decltype(all_finite)::value ? fixed_point_finite(x[j], e) : fixed_point_term(x[j], e);
            atomicAdd(&mine[j * S::kPitch + c], static_cast<unsigned long long>(v));
        }
        if (kCounted && piece == 0) atomicAdd(&cnt[c], 1u);
    };
    // Range r takes every ranges-th chunk, from the last one down - what the previous kernel read last is still in the
    // memory-side cache - kWaves / entry_sharers of them at a time: the workgroups of all slices of a range then work within a
    // window of X that their L2 holds. The entries of a wave's next batch are requested before the rows of this one, and
    // those before the ones of the last are added.
    uint32_t done = range + ranges * (wave / entry_sharers), first = 0, i0 = 0, end = 0;   // chunks above the current one
    size_t entries_at = 0;
    constexpr uint32_t kEntryPitch = RECORDS ? kChunk * kRecordBytes<D> / 4 : kChunk;
    const uint32_t step = ranges * (kWaves / entry_sharers);
    auto open = [&]() {   // first batch at or after `done`
        for (; done < chunks; done += step) {
            const uint32_t chunk = chunks - 1 - done;
            const uint32_t* at = starts + size_t(chunk) * (slices + 1) + slice;
            first = chunk * kChunk;
            entries_at = size_t(chunk) * kEntryPitch;
            end = LISTED ? at[1] : min(kChunk, N - first);
            i0 = LISTED ? at[0] : 0u;
            if (RECORDS && i0 >> kKindShift != kEntries) continue;
            i0 += wave % entry_sharers * (U * 64 / P);
            if (i0 < end) return;
        }
    };
    auto load_entries = [&](uint32_t (&ent)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = min(i0 + u * (64 / P) + which, end - 1);
            ent[u] = LISTED ? entries[entries_at + i] : (min(code_at<SRC>(idx, size_t(first) + i), K) << kPosBits) | i;
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
        i0 += entry_sharers * (U * 64 / P);
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
    };
    // Where no chunk left entries none is asked for them, which is a chain of 25 loads a wave (11.3 M vectors, K = 65536: a call 108.7 -> 105.3 us, 20 M 169 -> 159).
    if constexpr (!RECORDS || SRC == 0) {
        const bool any = !RECORDS || (flags & kLeftEntries) != 0;
        if (any && finite) add_entries(std::true_type{});   // a branch per number otherwise
        else if (any) add_entries(std::false_type{});
    }
    if (bad && parts == nullptr) atomicAdd(&hdr->skipped_vectors, static_cast<unsigned long long>(bad));
    __syncthreads();
    const size_t job = size_t(slice) * ranges + range;
    unsigned long long* ps = part_sums + job * (S::kPitch * D);
    uint32_t* pc = part_counts + job * S::kClusters;
#pragma unroll
    for (int j = 0; j < D; ++j)
        for (uint32_t t = threadIdx.x; t < k_n; t += kThreads) ps[j * S::kPitch + t] = sum[j * S::kPitch + t];
    if (kCounted)
        for (uint32_t t = threadIdx.x; t < k_n; t += kThreads) pc[t] = cnt[t];
}

// Adds the ranges of every cluster (integers: any order gives the same bits; this one is fixed anyway), leaves the
// totals in the workspace and writes the means (or, mean = 0, the plain sums). An empty cluster keeps prev. A workgroup
// finishes 64 neighbouring clusters of one component, its waves take turns at the ranges (one thread per cluster and
// component waited 75 us for 256 ranges at K = 1024). COUNTED is known to the compiler: with a branch around each count the loads
// of a wave went out one by one (256 ranges of one slice 8.3 us instead of 5.6).
template <int D, int W, int RECORDS, bool COUNTED>
__global__ __launch_bounds__(64 * W) void sliced_finalize_kernel(const unsigned long long* __restrict__ part_sums,
                                                                   const uint32_t* __restrict__ part_counts, uint32_t ranges,
                                                                   const float* prev, float* out, uint32_t* counts_out, uint32_t K,
                                                                   uint32_t N, WsHeader* hdr, int mean, long long* __restrict__ sums_ws,
                                                                   uint32_t* __restrict__ counts_ws, uint32_t width)
{
    using S = Slice<D, RECORDS>;
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
            if (COUNTED) n += part_counts[job * S::kClusters + local];
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
    sums_ws[size_t(k) * D + j] = isum;
    const size_t o = size_t(k) * width + j;
    if (COUNTED && j == 0) {
        counts_ws[k] = n;
        if (counts_out != nullptr) counts_out[k] = n;
    }
    const double total = ldexp(double(isum), -e);
    out[o] = !mean ? float(total) : (n > 0 ? float(total / double(n)) : prev[o]);
}

// Whether the rows go along (the head of this file says what it gives): there has to be room for as many ranges, or for the 8 that
// one per XCD takes. 16-bit rows of 8 and 16 at aligned places: up to 2^24 numbers, and at 8 with slices of which an XCD does not hold whole ranges (entries
// of one range then come through two L2s). bf16, by entries / rows along, us: g = 16: 4096x6144, K = 4096 49 / 52, 4096x8192 55 / 62 to 75 / 82, 8192x14336
// 124 / 171 to 167 / 204 (up to 4096x4096, by entries with the last kernel of before: 46 / 43, 63 / 62); g = 8: 4096x11008, K = 4096 69 / 73, K = 20000 75 / 79,
// K = 35000 78 / 81, 8192x14336, K = 4096 129 / 172, K = 20000 172 / 180, K = 35000 181 / 178; with that last kernel K = 50000 212 / 198, K = 45000 194 / 188.
template <int D, int SRC>
bool records_pay(uint32_t N, uint32_t K, bool fresh)
{
    if (!fresh || update_one_slice(D, K)) return false;
    const Cut c = cut_of<D, 1>(N, K);
    if (D >= 8 && SRC != 0 && uint64_t(N) * D > 1u << 24 && !(D == 8 && c.slices > 20 && c.slices < 32)) return false;
    return c.ranges >= std::min(cut_of<D>(N, K).ranges, 8u);
}

// Rows that go along take slices as wide as entries do (RECORDS = 2) for many fp32 vectors of 6 to 8 narrow slices: where a chunk's numbers turn out to
// have no 16 bits, every line is fetched by as many workgroups as there are slices. us a call by entries / narrow / wide, numbers without 16 bits: K = 15000:
// 11.3 M 120 / 116 / 114, 14 M 145 / 150 / 140, 28 M 282 / 298 / 271; K = 12000: 20 M 194 / 202 / 195. 16-bit numbers pay for twice the partial sums: K = 15000:
// 11.3 M 119 / 105 / 109, 20 M 201 / 158 / 162, 28 M 282 / 217 / 220. Beside these K the others lose little or nothing: 20 M, K = 5000 207 / 196 / 219, K = 8192
// 182 / 187 / 186, K = 9000 211 / 208 / 214, K = 20000 227 / 217 / 205 (16-bit ones 227 / 166 / 175).
bool wide_records_pay(uint32_t N, uint32_t K) { return N > 3u << 22 && K > 5 * Slice<4, 1>::kClusters && K <= 8 * Slice<4, 1>::kClusters; }

template <int D, int SRC, bool LISTED, int RECORDS>
hipError_t launch_t(const Cut& c, const void* X, uint32_t N, const void* idx, const float* prev, uint32_t K, float* out,
                    uint32_t* counts_out, const Workspace& w, bool mean, bool fresh, const RowPlace& place, hipStream_t s)
{
    using S = Slice<D, RECORDS>;
    const uint32_t jobs = c.slices * c.ranges;
    unsigned long long* part_sums = reinterpret_cast<unsigned long long*>(w.records);
    uint32_t* part_counts = SRC == 0 ? reinterpret_cast<uint32_t*>(w.records + size_t(jobs) * S::kSumBytes) : nullptr;
    ScanPart* parts = reinterpret_cast<ScanPart*>(w.records + c.sum_bytes);
    uint32_t* entries = reinterpret_cast<uint32_t*>(w.records + c.sum_bytes + c.part_bytes);
    uint32_t* starts = reinterpret_cast<uint32_t*>(w.records + c.sum_bytes + c.part_bytes + c.entry_bytes);
    // per call: the attribute belongs to the current device
    if (const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sliced_accumulate_kernel<D, SRC, LISTED, RECORDS>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(S::kLdsBytes)); e != hipSuccess)
        return e;
    if constexpr (RECORDS) {
        const dim3 threads(kChunkThreadsOf<D, 1>);
        char* records = reinterpret_cast<char*>(entries);
        if constexpr (SRC != 0) {
            if (place.per_row != 0)
                hipLaunchKernelGGL((record_chunk_kernel<D, SRC, false, RECORDS>), dim3(c.chunks), threads, 0, s, X, idx, N, K, c.slices, place, parts, records, starts);
            else
                hipLaunchKernelGGL((record_chunk_kernel<D, SRC, true, RECORDS>), dim3(c.chunks), threads, 0, s, X, idx, N, K, c.slices, place, parts, records, starts);
        } else {
            hipLaunchKernelGGL((record_chunk_kernel<D, SRC, true, RECORDS>), dim3(c.chunks), threads, 0, s, X, idx, N, K, c.slices, place, parts, records, starts);
        }
    } else if (fresh)
        hipLaunchKernelGGL((slice_chunk_kernel<D, SRC, true, LISTED>), dim3(c.chunks), dim3(kChunkThreads), 0, s, X, idx, N, K, c.slices, w.hdr,
                           parts, entries, starts);
    else if constexpr (LISTED && SRC == 0)
        hipLaunchKernelGGL((slice_chunk_kernel<D, SRC, false, true>), dim3(c.chunks), dim3(kChunkThreads), 0, s, X, idx, N, K, c.slices, w.hdr,
                           parts, entries, starts);
    hipLaunchKernelGGL((sliced_accumulate_kernel<D, SRC, LISTED, RECORDS>), dim3(8 * ((jobs + 7) / 8)), dim3(kThreads), S::kLdsBytes, s, X, N, idx,
                       K, c.slices, c.chunks, c.ranges, c.sharers, c.entry_sharers, w.hdr, fresh ? parts : nullptr, entries, starts, part_sums, part_counts);
    const uint32_t width = place.per_row != 0 ? place.g : D;   // of a row of the result
    const dim3 done((K + 63) / 64 * width);
    if (c.ranges > 32)
        hipLaunchKernelGGL((sliced_finalize_kernel<D, 16, RECORDS, SRC == 0>), done, dim3(1024), 0, s, part_sums, part_counts, c.ranges, prev, out,
                           counts_out, K, N, w.hdr, mean ? 1 : 0, w.sums, w.counts, width);
    else
        hipLaunchKernelGGL((sliced_finalize_kernel<D, 4, RECORDS, SRC == 0>), done, dim3(256), 0, s, part_sums, part_counts, c.ranges, prev, out,
                           counts_out, K, N, w.hdr, mean ? 1 : 0, w.sums, w.counts, width);
    return hipGetLastError();
}

template <int D, int SRC>
hipError_t update_sliced_t(const void* X, uint32_t N, const void* idx, const float* prev, uint32_t K, float* out,
                           uint32_t* counts_out, const Workspace& w, bool mean, bool fresh, hipStream_t s, const RowPlace& place = RowPlace{})
{
    const Cut c = cut_of<D>(N, K);
    if constexpr (SRC != 0 || D == 4)
        if (place.per_row != 0 || records_pay<D, SRC>(N, K, fresh)) {
            if constexpr (SRC == 0)
                if (wide_records_pay(N, K))
                    return launch_t<D, SRC, true, 2>(cut_of<D, 2>(N, K), X, N, idx, prev, K, out, counts_out, w, mean, fresh, place, s);
            return launch_t<D, SRC, true, 1>(cut_of<D, 1>(N, K), X, N, idx, prev, K, out, counts_out, w, mean, fresh, place, s);
        }
    if (c.listed) return launch_t<D, SRC, true, 0>(c, X, N, idx, prev, K, out, counts_out, w, mean, fresh, place, s);
    return launch_t<D, SRC, false, 0>(c, X, N, idx, prev, K, out, counts_out, w, mean, fresh, place, s);
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

// The sums (not the means) of the sub-vectors of a layer's 16-bit gradient (dtype 1 = fp16, 2 = bf16) by their 16-bit codes, read in
// place. Leaves the header as a reset and a scan of the rows would. Same fixed-point sums as launch_update on the converted rows:
// same bits. Rows at aligned places are loaded as they are; others (g other than 4, 8, 16, a padded last one, a gradient that does not
// begin at 16 bytes) number by number: 92 of 143 us at 4096 x 11008, g = 6.
template <int D>
hipError_t sum_rows16_t(const void* grad, int dtype, uint32_t N, uint32_t out_features, uint32_t g, const uint16_t* codes, uint32_t K, float* out,
                        const Workspace& w, hipStream_t s)
{
    const uint32_t per_row = (out_features + g - 1) / g;
    const bool whole = g == D && out_features % g == 0 && reinterpret_cast<uintptr_t>(grad) % 16 == 0;
    const RowPlace place = whole ? RowPlace{0, 0, 0} : RowPlace{per_row, g, per_row * g - out_features};
    return dtype == 2 ? update_sliced_t<D, 2>(grad, N, codes, nullptr, K, out, nullptr, w, false, true, s, place)
                      : update_sliced_t<D, 1>(grad, N, codes, nullptr, K, out, nullptr, w, false, true, s, place);
}

bool sum_rows16_applies(uint32_t N, uint32_t d, uint32_t K, const Workspace& w)
{
    if (!update_sliced_applies(N, d, K, w)) return false;
    return (d == 4 ? cut_of<4, 1>(N, K).ranges : (d == 8 ? cut_of<8, 1>(N, K).ranges : cut_of<16, 1>(N, K).ranges)) > 0;
}

hipError_t launch_sum_rows16(const void* grad, int dtype, uint32_t N, uint32_t out_features, uint32_t g, const uint16_t* codes, uint32_t K,
                             float* out, const Workspace& w, hipStream_t s)
{
    if (!sum_rows16_applies(N, w.d, K, w) || (dtype != 1 && dtype != 2)) return hipErrorInvalidValue;
    switch (w.d) {
        case 4: return sum_rows16_t<4>(grad, dtype, N, out_features, g, codes, K, out, w, s);
        case 8: return sum_rows16_t<8>(grad, dtype, N, out_features, g, codes, K, out, w, s);
        case 16: return sum_rows16_t<16>(grad, dtype, N, out_features, g, codes, K, out, w, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cc
