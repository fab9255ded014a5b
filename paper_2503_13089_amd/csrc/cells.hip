// E-step of a fit by cells (Section 3.1: the codes are the argmin over ALL centroids; a centroid can be skipped for a
// vector only if it provably cannot be that argmin), for sub-vectors of up to 8 numbers and K <= 65536.
//
// After the first iteration, or from a bootstrap's codes on (cells_from_first in api.hip), the vectors are grouped by the code they
// have: the group of centroid c is its cell. For a
// vector x of the cell with previous code h, u = ||x - c_h|| bounds the distance of its nearest centroid c', so
//     ||c - c'|| <= ||x - c|| + ||x - c'|| <= ||x - c|| + u =: t(x).
// Once per E-step every centroid gets the list of the centroids within a radius R of it; the vectors of its cell with
// t(x) <= R ("near") are decided on that list alone. It is 10^2 .. 10^3 times shorter than the codebook where the
// (norm, cosine) windows of sort.hip leave 3 % (d = 4) or 66 % (d = 8) of it: a ball in d dimensions against a shell.
// The other vectors ("far", 0.7 to 4 %) are collected in their norm order and go through a windowed matrix-core E-step, the
// 32 to 256 neighbours of a workgroup to a window. A centroid left out is farther than the previous code by a margin that no fp32 comparison can bridge, so the
// codes are the same bits as those of every other route, whatever the radius, however old the grouping.
// Measured, kernels of an E-step, means over a fit: N = 11 M, d = 4, K = 65536: lists 0.07 ms, near vectors 0.14, far ones 0.02 to collect and
// 0.03 to score, refinement 0.02, the centroids' order 0.03 (1.2 ms by windows). N = 29 M, d = 8: 0.47, 2.8, 0.12, 1.5, 0.06, 0.03
// (53 ms). At 2.8 M, d = 8: 0.25, 0.30, 0.02, 0.05, 0.02, 0.03.
//
// The grouping is only renewed now and then: a vector that has moved to a neighbouring cell meanwhile still has a t(x)
// against the cell it is stored with, just a larger one. The radius follows from what the last E-step saw: about
// kTarget centroids per list, and no more than the largest t(x) of the cell.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "f16_scores.h"
#include "ordering.h"
#include "score_sets.h"

namespace cc {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// A cell's list: the centroids within r1 of its centroid, then (d = 8) those between r1 and r2. Room in all for 4096 entries
// where 1500 are aimed at: the vectors of a longer one are far. 29 M vectors, K = 65536, 10 iterations: room for 6144
// 152.7 ms, 4096 153.4, 2560 157.5; 2.8 M vectors 28.4, 28.3 and 28.3 ms with 805, 537 and 335 MB of lists. How many are aimed at, d = 4: 36 / 44 / 54 / 60 / 74 entries, 11 M,
// K = 65536, 20 iterations 13.27 / 12.30 / 11.93 / 11.92 / 11.92 ms, 4.2 M, K = 4096 4.66 / 4.55 / 4.54 / 4.54 / 4.58; 2 M, K = 40000, 10 2.85 (44) / 2.80 (60). d = 8: 400 +
// 1100 / 400 + 800 / 330 + 870 / 500 + 1000, 29 M, K = 65536 77.0 / 78.8 / 78.9 / 77.4, 2.8 M of 6, K = 65500 17.38 / 17.16 / 17.29 / 17.22.
template <int D>
struct Lists {
    static constexpr uint32_t kCap1 = D == 4 ? 128 : 1024;            // room for entries within r1 ...
    static constexpr uint32_t kCap2 = D == 4 ? 0 : 3072;              // ... and between r1 and r2
    static constexpr uint32_t kCap = kCap1 + kCap2;
    static constexpr float kTarget1 = D == 4 ? 60.0f : 400.0f;        // entries within r1 / r2 that a list should have
    static constexpr float kTarget2 = D == 4 ? 60.0f : 1500.0f;
};

}  // namespace

uint32_t cell_list_cap(uint32_t d) { return d == 4 ? Lists<4>::kCap : Lists<8>::kCap; }

namespace {

// Lists and near vectors need numbers that -2 x in fp16 can carry (rounded: bounds cover that): fp16 inputs are, others if
// they are below 2^14.
__device__ __forceinline__ bool lists_exist(const WsHeader* hdr)
{
    return hdr->x_not_f16 == 0 || max(hdr->cmax_bits, hdr->absmax_bits) < 0x46800000u;
}

// What bounds are kept as, towards more and towards less: the upper half of the fp32 number.
__device__ __forceinline__ uint16_t upper_half(float v) { return uint16_t((__float_as_uint(v) + 0xffffu) >> 16); }   // v >= 0
__device__ __forceinline__ uint16_t lower_half(float v) { return uint16_t(__float_as_uint(__builtin_fmaxf(v, 0.0f)) >> 16); }
__device__ __forceinline__ float from_half(uint32_t v) { return __uint_as_float(v << 16); }

// ---- grouping ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void cell_keys_kernel(const uint32_t* __restrict__ idx, uint32_t N, uint16_t* __restrict__ keys,
                                                             uint32_t* __restrict__ ids)
{
    const uint32_t p = blockIdx.x * kThreads + threadIdx.x;
    if (p >= N) return;
    keys[p] = uint16_t(idx[p]);
    ids[p] = p;
}

// New position p holds what stood at order[p]. order is turned into the norm rank of every position (the position in
// the norm order the fit began with: rank_old == NULL means that the old order is that one). position, the inverse, may be NULL: where the far vectors stand the near
// kernels write in every E-step, and all of it only a later call asks for. 4-byte writes in random order were half of this kernel's time:
// 29 M vectors 1070, 850 and 720 us / 560, 480 and 275 without, 11 M 355 / 200.
__global__ __launch_bounds__(kThreads) void cell_apply_kernel(const uint16_t* __restrict__ sorted_keys, uint32_t N, uint32_t* order,
                                                              const uint32_t* __restrict__ rank_old,
                                                              const uint32_t* __restrict__ perm_old, uint32_t* __restrict__ perm_new,
                                                              uint32_t* __restrict__ position, uint32_t* __restrict__ idx)
{
    const uint32_t p = blockIdx.x * kThreads + threadIdx.x;
    if (p >= N) return;
    const uint32_t q = order[p];
    const uint32_t r = rank_old != nullptr ? rank_old[q] : q;
    order[p] = r;
    if (position != nullptr) position[r] = p;
    perm_new[p] = perm_old[q];
    idx[p] = sorted_keys[p];
}

// First vector of every cell (codes are sorted: a binary search each).
__global__ __launch_bounds__(kThreads) void cell_starts_kernel(const uint16_t* __restrict__ sorted_keys, uint32_t N, uint32_t K,
                                                               CellHead* __restrict__ heads)
{
    const uint32_t t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= K) return;
    uint32_t bound[2];
#pragma unroll
    for (uint32_t u = 0; u < 2; ++u) {
        uint32_t a = 0, b = N;
        while (a < b) {
            const uint32_t m = a + (b - a) / 2;
            if (uint32_t(sorted_keys[m]) >= t + u) b = m; else a = m + 1;
        }
        bound[u] = a;
    }
    heads[t].start = bound[0];
    heads[t].members = bound[1] - bound[0];
}

// ---- radius -----------------------------------------------------------------------------------------------------
// Mean and largest t(x) of a cell's first n <= 256 vectors, by one wave.
template <int D>
__device__ __forceinline__ void cell_bounds(const float* X, const uint32_t* idx, const float* C, uint32_t K, uint32_t c, uint32_t s0, uint32_t n,
                                            float& mean, float& most)
{
    float row[D], sum = 0.0f;
    load_row<D>(C + size_t(c) * D, row);
    most = 0.0f;
    for (uint32_t i = threadIdx.x & 63; i < n; i += 64) {
        float x[D], ch[D];
        load_row<D>(X + size_t(s0 + i) * D, x);
        load_row<D>(C + size_t(min(idx[s0 + i], K - 1)) * D, ch);
        const float t = __builtin_sqrtf(direct_sqdist<D>(x, row)) + __builtin_sqrtf(direct_sqdist<D>(x, ch));
        sum += t;
        most = __builtin_fmaxf(most, t);
    }
    for (int off = 32; off > 0; off >>= 1) {
        sum += __shfl_xor(sum, off, 64);
        most = __builtin_fmaxf(most, __shfl_xor(most, off, 64));
    }
    mean = n > 0 ? sum / float(n) : 0.0f;
}

// First radii of a cell: multiples of the mean t(x) of (up to 256 of) its vectors. One wave per cell.
template <int D>
__global__ __launch_bounds__(kThreads) void cell_first_radius_kernel(const float* __restrict__ X, const uint32_t* __restrict__ idx,
                                                                     CellHead* __restrict__ heads, const float* __restrict__ C,
                                                                     uint32_t K, float factor1, float factor2)
{
    const uint32_t c = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (c >= K) return;
    float mean, most;
    cell_bounds<D>(X, idx, C, K, c, heads[c].start, min(heads[c].members, 256u), mean, most);
    if ((threadIdx.x & 63) == 0) {
        heads[c].r1 = factor1 * mean;
        heads[c].r2 = factor2 * mean;
    }
}

// Work items of at most `item` vectors of one cell: cell c owns the slots [start / item + c, next cell's) of the item
// table, always enough for its ceil(members / item) items; the slots it does not need are marked empty.
// A cell that had one vector, or none, at the grouping before was left with a radius of about zero, and what it has been given
// since would be far for good: a cell with a short list and a radius below a tenth of its mean t(x) gets a first radius again,
// within what its vectors need, with counts and a largest t(x) that let the next E-step take it as it is. (Clumped data, half
// of the vectors in such cells: 0.3 to 0.5 instead of 2.9 tiles of 32 centroids scored per 512 vectors.)
template <int D>
__global__ __launch_bounds__(kThreads) void cell_items_kernel(CellHead* __restrict__ heads, uint32_t K, uint32_t slots, uint32_t item,
                                                              uint4* __restrict__ items, const float* __restrict__ X,
                                                              const uint32_t* __restrict__ idx, const float* __restrict__ C,
                                                              float factor1, float factor2, int first_time)
{
    using L = Lists<D>;
    const uint32_t c = blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (c >= K) return;
    const uint32_t s0 = heads[c].start, members = heads[c].members;
    const uint32_t first = s0 / item + c, end = c + 1 < K ? (s0 + members) / item + c + 1 : slots;
    const uint32_t used = first + (members + item - 1) / item;
    for (uint32_t s = first + (threadIdx.x & 63); s < end; s += 64) items[s] = make_uint4(s < used ? c : 0xffffffffu, s0, (s - first) * item, members);
    if (first_time || heads[c].n1 >= uint32_t(L::kTarget1 / 4)) return;
    float mean, most;
    cell_bounds<D>(X, idx, C, K, c, s0, min(members, 256u), mean, most);
    if ((threadIdx.x & 63) == 0 && heads[c].r1 < 0.1f * mean) {
        heads[c].r1 = __builtin_fminf(factor1 * mean, 1.05f * most);
        heads[c].r2 = __builtin_fminf(factor2 * mean, 1.05f * most);
        heads[c].n1 = uint32_t(L::kTarget1);
        heads[c].n2 = uint32_t(L::kTarget2) - uint32_t(L::kTarget1);
        heads[c].tmax = 0x7f800000u;
    }
}

static_assert(kStageTiles % kSetGroup == 0 && kStageTilesMax % kSetGroup == 0, "runs share no group, the packed codebook has room for whole ones");

// ---- centroids: order, operands, radii ------------------------------------------------------------------------------
// Three launches put the centroids into the order of sort.hip's (norm shell, cosine) key with everything the E-step needs
// of them: keys and histogram; prefix sums (which are the key -> first position table); rows, permutations and operands
// straight to their places. Unlike the stable radix sort this leaves the order among equal keys to scheduling, which
// decides nothing but which tile a centroid shares; eight launches of 4 us for a few microseconds of work became three.

// Keys and their histogram, the largest magnitude; and what has to happen once per E-step: the radii follow the lengths
// of the cell's last list (towards the targets, at most 18 % a step unless the centroids stayed) and never exceed what any vector
// of the cell needed;
// the bitmaps of changed codes and far vectors and the refine counter are cleared.
template <int D>
__global__ __launch_bounds__(kThreads) void cell_keys_of_centroids_kernel(const float* __restrict__ C, uint32_t K, uint32_t words,
                                                                          int radii, uint16_t* __restrict__ keys,
                                                                          uint32_t* __restrict__ hist, CellHead* __restrict__ heads,
                                                                          uint32_t* __restrict__ changed, uint32_t* __restrict__ far_bits, WsHeader* hdr,
                                                                          const float* __restrict__ csorted, const uint32_t* __restrict__ cinv,
                                                                          uint16_t* __restrict__ moves)
{
    using L = Lists<D>;
    const uint32_t t = blockIdx.x * kThreads + threadIdx.x;
    if (t == 0) hdr->refine_count = 0;
    if (t < words) {
        changed[t] = 0;
        far_bits[t] = 0;
    }
    uint32_t m = 0;
    if (t < K) {
        float c[D];
        load_row<D>(C + size_t(t) * D, c);
        float s = 0.0f, proj;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            s = __builtin_fmaf(c[j], c[j], s);
            m = max(m, __float_as_uint(c[j]) & 0x7fffffffu);
        }
        const uint32_t key = ordering_key<D>(c, __builtin_sqrtf(s), shell_base(hdr->absmax_bits, D), proj);
        keys[t] = uint16_t(key);
        atomicAdd(&hist[key], 1u);
        if (moves != nullptr) {   // how far it can have moved since the E-step before
            float before[D];
            load_row<D>(csorted + size_t(cinv[t]) * D, before);
            moves[t] = upper_half(__builtin_sqrtf(direct_sqdist<D>(c, before)) * 1.00001f + 3e-19f);
        }
        if (radii != kRadiiStay) {
            const CellHead h = heads[t];
            // vectors need longer lists in the first E-step, whose centroids are vectors themselves (29 M, K = 65536: 124 ms with
            // the targets as they are, 122.5 with 1.6 times as much, 123 with twice)
            const float longer = radii == kRadiiJump ? 1.6f : 1.0f, most = radii == kRadiiJump ? 2.0f : 1.18f;
            auto next = [&](float r, float target, uint32_t n) {
                float step = __builtin_sqrtf(__builtin_sqrtf(target / float(max(n, 1u))));
                if (D == 8) step = __builtin_sqrtf(step);
                const float to = r * fminf(fmaxf(step, radii == kRadiiJump ? 0.5f : 0.85f), most);
                return radii == kRadiiJump ? to : fminf(to, 1.05f * __uint_as_float(h.tmax));
            };
            const float r1 = next(h.r1, longer * L::kTarget1, h.n1);
            heads[t].r1 = r1;
            heads[t].r2 = fmaxf(r1, next(h.r2, longer * L::kTarget2, h.n1 + h.n2));
        }
        heads[t].tmax = 0;
        heads[t].mids = 0;
    }
    // one look at the running maximum per workgroup that has centroids: one per wave of the whole grid, all at one address, took 16 of 27 us
    __shared__ uint32_t wave_most[kWaves];
    for (int off = 32; off > 0; off >>= 1) m = max(m, uint32_t(__shfl_xor(int(m), off, 64)));
    if ((threadIdx.x & 63) == 0) wave_most[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x != 0 || t >= K) return;
    for (int v = 1; v < kWaves; ++v) m = max(m, wave_most[v]);
    if (m > __builtin_nontemporal_load(&hdr->cmax_bits)) atomicMax(&hdr->cmax_bits, m);
}

// Where a centroid stands among the operands of the lists. d = 8: tiles come in pairs, whose results for a lane are made one six-bit number each, the pair's in turn, by one
// instruction (score_bits); z, the place of its two bits in a word from the top, says which of the 2 x 8 results of that word it is.
struct ListRow {
    uint32_t tile, row;
};
__host__ __device__ constexpr ListRow paired_row(uint32_t at)
{
    const uint32_t word = (at >> 5) & 1u, h = (at >> 4) & 1u, p = 15u - (at & 15u), in = p / 3u;   // p: from the bottom
    const uint32_t turn = p % 3u == 2u ? in : (p % 3u == 1u ? 5u + in : 10u + in), reg = 8u * word + turn / 2u;
    return {(at >> 6) * 2u + (turn & 1u), reg % 4u + 8u * (reg / 4u) + 4u * h};
}
// Which bits of a word of three are sign and upper exponent bit of a number, 6 bits after the one before from bit 4 of the three on: the third's are the rest.
constexpr uint32_t kPairs0 = 0x30c30c30u, kPairs1 = 0x0c30c30cu, kPairs2 = ~(kPairs0 | kPairs1);
// Result i of tile u of a pair has the six bits from 12 i + 6 u on (of six words); paired_row has to send the centroid there that the word's place stands for.
constexpr bool pairs_stand_where_the_rows_say()
{
    for (uint32_t at = 0; at < 64; ++at) {
        const ListRow to = paired_row(at);
        const uint32_t i = to.row % 4 + 4 * (to.row / 8), bit = 12 * i + 6 * to.tile + 4, of_three = bit % 96 / 32, in_word = bit % 32;
        const uint32_t mask = of_three == 0 ? kPairs0 : (of_three == 1 ? kPairs1 : kPairs2);
        if (to.tile > 1 || to.row / 4 % 2 != (at >> 4 & 1) || bit / 96 != at >> 5 || ((mask >> in_word) & 3u) != 3u || 30 - in_word != 2 * (at & 15)) return false;
    }
    return (kPairs0 & kPairs1) == 0 && kPairs2 == 0xc30c30c3u;
}
static_assert(pairs_stand_where_the_rows_say(), "bits of the lists");

// Every centroid to its place: permutation and inverse, ordered row, the operand row of the E-step's packed codebook
// (assign_mfma_f16.hip) and the one of the lists: 8 product slots (the first fp16 part of each component) and
// 8 for norm and threshold: sigma ||c||^2 in three parts against the multipliers 2^8, 2^-3, 2^-14 of the other side, and
// those multipliers themselves. Positions past K get operands that never win and never enter a list. Inputs that are not fp16 numbers have
// their far vectors scored on fp32 operands (assign_mfma.hip), which take the packed codebook's place.
template <int D>
__global__ __launch_bounds__(kThreads) void cell_place_kernel(const float* __restrict__ C, uint32_t K, uint32_t padded,
                                                              const uint16_t* __restrict__ keys, uint32_t* __restrict__ cursor,
                                                              uint32_t* __restrict__ cperm, uint32_t* __restrict__ cinv,
                                                              float* __restrict__ csorted, char* __restrict__ packed,
                                                              char* __restrict__ operands, char* __restrict__ flat,
                                                              const WsHeader* __restrict__ hdr)
{
    using S = F16Shape<D>;
    static_assert(S::KM == 1, "one matrix instruction per tile");
    const uint32_t k = blockIdx.x * kThreads + threadIdx.x;
    if (k >= padded) return;
    const bool valid = k < K;
    float c[D];
#pragma unroll
    for (int j = 0; j < D; ++j) c[j] = 0.0f;
    uint32_t pos = k;
    if (valid) {
        load_row<D>(C + size_t(k) * D, c);
        pos = atomicAdd(&cursor[keys[k]], 1u);
        cperm[pos] = k;
        cinv[k] = pos;
#pragma unroll
        for (int q = 0; q < D / 4; ++q)
            reinterpret_cast<float4*>(csorted + size_t(pos) * D)[q] = make_float4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
    }
    double norm = 0.0;
#pragma unroll
    for (int j = 0; j < D; ++j) norm += double(c[j]) * double(c[j]);
    const bool f16 = hdr->x_not_f16 == 0;
    if (!f16) put_f32_operand<D>(reinterpret_cast<float*>(packed), pos, c, valid ? float(norm) : INFINITY);
    if (!lists_exist(hdr)) return;
    const float sigma = __builtin_ldexpf(1.0f, centroid_scale_log2(hdr->cmax_bits, D));
    _Float16 parts[D][3], g[3];
#pragma unroll
    for (int j = 0; j < D; ++j) split3(c[j] * sigma, parts[j]);
    const float scaled_norm = valid ? float(norm * double(sigma)) : INFINITY;
    if (valid) {
        split_norm(scaled_norm, g);
    } else {
        g[0] = _Float16(INFINITY);
        g[1] = g[2] = _Float16(0.0f);
    }
    if (f16) put_f16_operand<D>(packed, pos, parts, g, scaled_norm);
    if (flat != nullptr && valid) {  // d = 8: the operand pieces of one centroid side by side, for the near vectors
        f16x8* to = reinterpret_cast<f16x8*>(flat + size_t(k) * 64);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            f16x8 v;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = parts[j % D][p];
            to[p] = v;
        }
        const _Float16 o = _Float16(0.0f);
        to[3] = f16x8{g[0], g[1], g[2], o, o, o, o, o};
        if (k == 0) {   // row K never wins, and is finite so that a tag leaves it a number. Its score is 60000 * 2^8 = 1.54e7. The
                        // best of a near vector is below 5.9e6: its cell's centroid and its previous code are both on the list
                        // and their distances add up to R at most, so one of them is within R / 2; and where there is a list,
                        // sigma R^2 <= 1.5e7 + sigma ||c||^2 <= 1.5e7 + 2^23.
            f16x8* none = reinterpret_cast<f16x8*>(flat + size_t(K) * 64);
            none[0] = none[1] = none[2] = f16x8{o, o, o, o, o, o, o, o};
            none[3] = f16x8{_Float16(60000.0f), o, o, o, o, o, o, o};
        }
    }
    const uint32_t at = D == 4 ? pos : k;   // d = 8: lists take the whole codebook, and hold indices
    if (at >= list_tiles(D, K) * 32) return;   // tile by tile
    const ListRow row = D == 4 ? ListRow{at >> 5, 4 * ((at & 31u) >> 4) + (at & 3u) + 8 * ((at & 15u) >> 2)} : paired_row(at);
    const uint32_t m = row.row;
    char* op = operands + size_t(row.tile) * 1024;
    f16x8 lo, hi;
#pragma unroll
    for (int j = 0; j < 8; ++j) lo[j] = j < D ? parts[j % D][0] : _Float16(0.0f);
    const _Float16 z = _Float16(0.0f);
    hi = f16x8{valid ? g[0] : _Float16(60000.0f), g[1], g[2], _Float16(256.0f), _Float16(0.125f), _Float16(6.103515625e-05f), z, z};
    *reinterpret_cast<f16x8*>(op + m * 16) = lo;
    *reinterpret_cast<f16x8*>(op + (32 + m) * 16) = hi;
}

// ---- lists: one workgroup per 32 cells (neighbours in the norm order), its waves taking turns at the codebook ---------
// One matrix instruction gives sigma (||c'||^2 - 2 c.c' - (R^2 - ||c||^2 + slack)) for 32 x 32 (centroid, cell) pairs;
// an entry is kept where that is negative. Both sides' coordinates are fp16 (2^-11 relative each), which the slack covers: a
// list may hold a few centroids beyond R, never fewer than all within. The signs of a lane's 16 results are shifted into
// one word, at d = 8 with the upper bit of their exponents: a cell's side is scaled so that what lies within the inner radius scores -2
// or less. The cells' counters are in LDS. Where in a list an entry lands depends on scheduling; no result does.
// WINDOWED (d = 4): only the runs of the ordered codebook that the shells and cosines of sort.hip allow for the 32 cells;
// at d = 8 a ball that is 1 % of the codebook touches most of them.
// d = 8: sign and upper exponent bit of 32 results come out of one conversion to six-bit numbers (64 clocks; shifted into a word one by one they take 128) and
// two selections per word. Vector instructions (16 a tile with those of its hits; 35 before, with 64-bit addresses and operands copied out of the way of
// the next) take four fifths of the time, L2 most of the rest (a KB of operands per product, 2 bytes per entry written on their own). K = 65536: 4.3 G pairs at d = 8 in 0.22 ms
// (lists of 2.8 M vectors; 0.26 before), 0.06 at d = 4 (11 M). Entries gathered in LDS and written in runs, between barriers every 8 or 16 pairs of tiles:
// 0.28.
// Two products per tile (64 cells to a workgroup) halve the loads and lose: 0.32 -> 0.39.
constexpr float kListThrMax = 1.5e7f;     // what three fp16 parts against 2^8, 2^-3, 2^-14 can carry
// Waves of a workgroup. With 4 the whole launch is on the chip at once and ends on the few workgroups of the outer shells, whose lists are the longest;
// with 8 or 16 those start first and are shared by more.
template <int D> constexpr int kListWaves = D == 4 ? 8 : 16;
// Two bits of each of 2 x 16 results, sign and upper exponent bit (-2 or less after rounding to four of them: from -1.9375 on), as words of 16 pairs (paired_row).
// The last statement keeps the result out of the operands' registers: written there, it destroys what has not been read yet, and the compiler does not know.
__device__ __forceinline__ void score_bits(const f32x16& a, const f32x16& b, uint32_t (&word)[2])
{
    u32x6 v = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(a, b, 1.0f);
    asm volatile("" : "+v"(v) : "v"(a), "v"(b));
    uint32_t m0 = kPairs0, m1 = kPairs1;
    asm("" : "+s"(m0), "+s"(m1));   // two selections, which the compiler takes apart where it knows the masks, or what is asked of the word
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t rest = (v[3 * i + 1] & m1) | (v[3 * i + 2] & ~m1);
        word[i] = (v[3 * i] & m0) | (rest & ~m0);
        asm("" : "+v"(word[i]));
    }
}

template <int D, bool WINDOWED>
__global__ __launch_bounds__(64 * kListWaves<D>, 8) void cell_lists_kernel(const float* __restrict__ csorted, const uint32_t* __restrict__ cperm,
                                                              uint32_t K, const char* __restrict__ operands, uint32_t ntiles,
                                                              const uint32_t* __restrict__ key_starts, CellHead* __restrict__ heads,
                                                              uint32_t N, WsHeader* hdr, uint16_t* __restrict__ lists,
                                                              uint32_t* __restrict__ hist, uint32_t* __restrict__ queued_near)
{
    using L = Lists<D>;
    static_assert(WINDOWED == (D == 4), "d = 8: the whole codebook, by pairs of tiles");
    __shared__ uint32_t cnt1[32], cnt2[32], cell_ids[32], all_inner[32];
    __shared__ uint2 queues[kListWaves<D>][128];   // per wave: fewer than 64 entries left over + at most 64 of one tile
    for (uint32_t i = blockIdx.x * (64 * kListWaves<D>) + threadIdx.x; i < 65536; i += gridDim.x * (64 * kListWaves<D>)) {
        hist[i] = 0;  // for the next E-step
        if (D == 8) queued_near[i] = 0;
    }
    if (!lists_exist(hdr)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), h = lane >> 5, n = lane & 31;
    const uint32_t p0 = (gridDim.x - 1 - blockIdx.x) * 32;
    const uint32_t pos = min(p0 + n, K - 1), c = cperm[pos];
    if (threadIdx.x < 32) {
        cnt1[threadIdx.x] = 0;
        cnt2[threadIdx.x] = 0;
        cell_ids[threadIdx.x] = c;
    }
    float x[D];
    load_row<D>(csorted + size_t(pos) * D, x);
    const CellHead head = heads[c];
    float xn = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) xn = __builtin_fmaf(x[j], x[j], xn);
    const float norm = __builtin_sqrtf(xn);
    const float sigma = __builtin_ldexpf(1.0f, centroid_scale_log2(hdr->cmax_bits, D));
    // slack: 2^-9 ||c|| ||c'|| = 1.95e-3 for the rounded operands; everything else (accumulation, the split of norm and
    // threshold, fp16 subnormals) is far below the difference to 2.2e-3 and the constant term
    auto reach = [&](float R) { return sigma * (R * R * 1.0001f - xn + 2.2e-3f * norm * (norm + R)); };
    float r2 = L::kCap2 > 0 ? head.r2 : head.r1;
    if (reach(r2) + 0.05f > kListThrMax) r2 = head.r1;
    // The cell's side times f: what lies within r1 then scores -2 or less, and sign and upper exponent bit say both. f has 11 bits, so that
    // its products with the multipliers are exact (where 2^-3 f and 2^-14 f are subnormal numbers, what they lose is below 2^-18 of the norm),
    // and is at least 2 / gap after its rounding. What f < 1 does not scale is the error of a cell's operand among the
    // subnormal numbers, at most 2^-25 against every component of the other side.
    _Float16 f = _Float16(1.0f);
    bool apart = false;   // else everything within r2 counts as within r1
    if constexpr (L::kCap2 > 0) {
        const float gap = sigma * ((r2 * r2 - head.r1 * head.r1) * 1.0001f + 2.2e-3f * norm * (r2 - head.r1)), want = 2.004f / gap;
        apart = gap > 0.0f && want > 6.2e-5f && want < 255.0f && want * 2.0f * norm < 60000.0f &&
                want * __builtin_fabsf(reach(r2)) < 0.99f * kListThrMax;
        if (apart) f = _Float16(want);
    }
    const float scale = float(f), thr = L::kCap2 > 0 ? scale * (reach(r2) + 0.05f) + (3e-7f * sigma * __uint_as_float(hdr->cmax_bits) + 1e-3f) : reach(r2) + 0.05f;
    const bool carried = thr <= kListThrMax;  // else the cell goes without a list
    const bool live = p0 + n < K && head.members > 0 && head.r1 > 0.0f && carried;
    if (threadIdx.x < 32) all_inner[threadIdx.x] = apart ? 0u : 0xffffffffu;
    f16x8 b;
    {
        _Float16 tp[3];
        split_norm(live ? -thr : kListThrMax, tp);
        const _Float16 z = _Float16(0.0f);
        f16x8 lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) lo[j] = j < D ? _Float16(-2.0f * scale * x[j % D]) : z;
        const f16x8 hi = f16x8{_Float16(256.0f * scale), _Float16(0.125f * scale), _Float16(6.103515625e-05f * scale), tp[0], tp[1], tp[2], z, z};
        b = h ? hi : lo;
    }
    __syncthreads();
    f32x16 zero;
#pragma unroll
    for (int q = 0; q < 16; ++q) zero[q] = 0.0f;

    // runs of tiles to scan: with windows one per lane (shell), else a single run
    uint2 run = make_uint2(0, ntiles);
    uint32_t nruns = 1;
    if constexpr (WINDOWED) {
        const uint32_t base = shell_base(hdr->absmax_bits, D);
        float prj;
        (void)ordering_key<D>(x, norm, base, prj);
        float nlo = live ? norm - r2 : INFINITY, nhi = live ? norm + r2 : 0.0f;
        float plo = live ? prj - r2 : INFINITY, phi = live ? prj + r2 : -INFINITY;
        for (int off = 16; off > 0; off >>= 1) {
            nlo = __builtin_fminf(nlo, __shfl_xor(nlo, off, 64));
            nhi = __builtin_fmaxf(nhi, __shfl_xor(nhi, off, 64));
            plo = __builtin_fminf(plo, __shfl_xor(plo, off, 64));
            phi = __builtin_fmaxf(phi, __shfl_xor(phi, off, 64));
        }
        const float slack = nhi < 3.0e38f ? 1e-5f * nhi : 0.0f;
        nlo -= slack; nhi += slack; plo -= slack; phi += slack;
        const uint32_t smin = shell_of_key(nlo > 0.0f ? norm_key(nlo) : 0u, base);
        const uint32_t smax = shell_of_key(nhi < 3.0e38f ? norm_key(nhi) : 0xffffu, base);
        const bool wide = smax - smin + 1 > 64u;
        nruns = uint32_t(__builtin_amdgcn_readfirstlane(int(wide ? 1u : smax - smin + 1)));
        uint32_t klo = smin << 7, khi = (smax << 7) | 127u;
        if (!wide) shell_cosine_run(smin + min(uint32_t(lane), nruns - 1), base, plo, phi, klo, khi);
        run = make_uint2(0, 0);
        if (klo <= khi && nlo <= nhi) {
            const uint32_t first = key_starts[klo], end = key_starts[khi + 1];
            if (first < end) run = make_uint2(first / 32, (end + 31) / 32);
        }
    }
    // Lanes with a hit push (their rows' bits, tile and lane) onto a queue of their wave; 64 entries at a time are then
    // taken off it, one per lane. Worked off on the spot, a tile's few hits would keep the wave busy for six times as
    // many instructions as the rest of the tile.
    uint2* queue = queues[wave];
    uint32_t queued = 0;   // wave-uniform
    auto work_off = [&](uint32_t count) {   // the first `count` <= 64 entries
        if (uint32_t(lane) >= count) return;
        const uint2 q = queue[lane];
        const uint32_t cell = q.y & 31u, first_pos = (q.y >> 6) * 32 + (q.y & 32u ? 16u : 0u);
        if constexpr (D == 4) {
            uint32_t mask = q.x << 16, at = atomicAdd(&cnt1[cell], uint32_t(__popc(mask)));
            const uint32_t list = cell_ids[cell] * L::kCap, end = list + L::kCap1;
            at += list;
            while (mask != 0) {
                const uint32_t bit = uint32_t(__builtin_clz(mask));
                mask ^= 0x80000000u >> bit;
                if (at < end) lists[at] = uint16_t(first_pos + bit);
                ++at;
            }
        } else {
            const uint32_t all = q.x & 0xaaaaaaaau, inner = all & ((q.x << 1) | all_inner[cell]), outer = all ^ inner;
            const uint32_t n1 = __popc(inner), n2 = __popc(outer), at = cell_ids[cell] * L::kCap;
            const uint32_t at1 = at + (n1 ? atomicAdd(&cnt1[cell], n1) : 0u), at2 = at + L::kCap1 + (n2 ? atomicAdd(&cnt2[cell], n2) : 0u);
            auto put = [&](uint32_t mask, uint32_t at, uint32_t end) {   // in bytes of the whole table, 512 MB at most
                while (mask != 0) {
                    const uint32_t bit = uint32_t(__builtin_clz(mask));
                    mask ^= 0x80000000u >> bit;
                    if (at < end) *reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(lists) + at) = uint16_t(((first_pos << 16) | (bit << 15)) >> 16);
                    at += 2;
                }
            };
            put(inner, 2 * at1, 2 * (at + L::kCap1));
            put(outer, 2 * at2, 2 * (at + L::kCap));
        }
    };
    auto push = [&](uint32_t bits, uint32_t mask, uint32_t which) {   // 32 * which: the first of the rows
        const unsigned long long hits = __ballot(mask != 0);
        if (mask != 0)
            (queue + queued)[__builtin_amdgcn_mbcnt_hi(uint32_t(hits >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(hits), 0u))] = make_uint2(bits, (which << 6) | uint32_t(lane));
        queued += uint32_t(__popcll(hits));
        if (queued >= 64) {
            wave_order();
            work_off(64);
            queued -= 64;
            const uint2 rest = queue[64 + lane];
            wave_order();
            if (uint32_t(lane) < queued) queue[lane] = rest;
            wave_order();
        }
    };
    auto operand = [&](uint32_t t, f16x8* a, auto tiles) {   // neighbouring tiles
        typedef const __attribute__((address_space(1))) char* Global;
        Global tile = reinterpret_cast<Global>(reinterpret_cast<uintptr_t>(operands + size_t(t) * 1024));
        uint32_t lane_at = lane * 16;
        asm volatile("" : "+s"(tile), "+v"(lane_at));   // a scalar and 32 bits: else a 64-bit addition per request
#pragma unroll
        for (int u = 0; u < decltype(tiles)::value; ++u) a[u] = *reinterpret_cast<const __attribute__((address_space(1))) f16x8*>(tile + lane_at + 1024 * u);
    };
    using One = std::integral_constant<int, 1>;
    using Pair = std::integral_constant<int, 2>;
    if constexpr (D == 4) {
        uint32_t next = 0;
        for (uint32_t r = 0; r < nruns; ++r) {
            const uint32_t r0 = max(uint32_t(__builtin_amdgcn_readlane(int(run.x), int(r))), next);  // a tile on the border of
            const uint32_t t1 = uint32_t(__builtin_amdgcn_readlane(int(run.y), int(r)));             // two shells is visited once
            if (r0 >= t1) continue;
            next = t1;
            f16x8 a, an;
            operand(min(r0 + wave, t1 - 1), &a, One{});
            for (uint32_t t = r0 + wave; t < t1; t += kListWaves<D>) {   // one at a time: a run has a few
                operand(min(t + kListWaves<D>, t1 - 1), &an, One{});
                const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, zero, 0, 0, 0);
                float m = INFINITY;
#pragma unroll
                for (int q = 0; q < 8; ++q) m = __builtin_fminf(__builtin_fminf(m, acc[2 * q]), acc[2 * q + 1]);
                if (__any(m < 0.0f)) {
                    uint32_t bits = 0;   // row 0 uppermost
#pragma unroll
                    for (int q = 0; q < 16; ++q) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(acc[q]), 31);
                    push(bits, bits, t);
                }
                a = an;
            }
        }
    } else {
        const uint32_t pairs = ntiles / 2;
        f16x8 a[2];
        operand(2 * min(uint32_t(wave), pairs - 1), a, Pair{});
        for (uint32_t t = wave; t < pairs; t += kListWaves<D>) {
            f32x16 acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b, zero, 0, 0, 0), acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b, zero, 0, 0, 0);
            asm volatile("" : "+v"(acc0), "+v"(acc1));   // requested before the products, the next operands would need registers of their own
            operand(2 * min(t + kListWaves<D>, pairs - 1), a, Pair{});
            uint32_t word[2];
            score_bits(acc0, acc1, word);
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) push(word[u], word[u] & 0xaaaaaaaau, 2 * t + u);
        }
    }
    wave_order();
    work_off(queued);
    __syncthreads();
    if (wave == 0) {
        float scored = 0.0f;
        if (h == 0 && p0 + n < K) {
            heads[c].n1 = carried ? cnt1[n] : 0xffffffffu;
            heads[c].n2 = cnt2[n];
            if (r2 != head.r2) heads[c].r2 = r2;
            if (carried) scored = float(cnt1[n]) * float(head.members);
        }
        // statistics: pairs the near vectors look at, in units of (512 vectors x 32 centroids)
        for (int off = 32; off > 0; off >>= 1) scored += __shfl_xor(scored, off, 64);
        if (lane == 0) {
            const auto stages = static_cast<unsigned long long>(scored / 16384.0f + 0.5f);
            atomicAdd(&hdr->window_stages, stages);
            atomicAdd(&hdr->list_stages, stages);
            if (blockIdx.x == 0)
                atomicAdd(&hdr->window_total, static_cast<unsigned long long>((N + kWinTile - 1) / kWinTile) * ((K + 31) / 32));
        }
    }
}

// ---- what the near kernels share ---------------------------------------------------------------------------------
struct NearArgs {
    const float* X;
    const float* C;             // centroids by index
    const float* csorted;       // d = 4: centroids in the norm order ...
    const uint32_t* cperm;      // ... and their indices
    const char* flat;           // d = 8: operand pieces of the centroids, by index
    uint32_t K;
    CellHead* heads;
    const uint4* items;
    uint32_t slots;
    const uint16_t* lists;
    const uint32_t* rank;
    uint32_t* far_bits;         // by norm rank
    uint32_t* position;         // by norm rank: that of the far vectors
    uint32_t* queues;           // d = 8: positions of vectors to be scored, in their cell's places: those within r1 from its first on,
                                // those between r1 and r2 from its last backwards
    uint32_t* queued_near;      // [K] how many of the former (the latter: CellHead::mids)
    const uint32_t* moved;      // [K] most that a centroid of the list within r1 / of the whole list has moved: upper halves, low / high
    uint16_t* bound;            // by position: no centroid but the code's is nearer than that (lower_half); NULL: nobody asks
    bool bounded;               // the E-step before was one by cells, of this grouping
    uint32_t* idx;
    float* dmin;                // NULL: nobody reads the distances
    uint32_t* prev_out;         // NULL: changes are not tracked
    uint32_t* changed;
    WsHeader* hdr;
};

// Sets bit (p0 + lane) of a bitmap for every set bit of `m` (wave-uniform), where the 64 positions start anywhere.
__device__ __forceinline__ void or_bits(uint32_t* bits, uint32_t p0, unsigned long long m, int lane)
{
    if (m == 0) return;
    const uint32_t sh = p0 & 31u;
    const uint32_t w = lane == 0 ? uint32_t(m << sh) : (lane == 1 ? uint32_t(m >> (32 - sh)) : (sh ? uint32_t(m >> (64 - sh)) : 0u));
    if (lane < 3 && w != 0) atomicOr(bits + (p0 >> 5) + lane, w);
}

__device__ __forceinline__ void or_bit(uint32_t* bits, uint32_t p) { atomicOr(bits + (p >> 5), 1u << (p & 31u)); }

__device__ __forceinline__ void mark_far(const NearArgs& a, uint32_t p)
{
    const uint32_t r = a.rank[p];
    or_bit(a.far_bits, r);
    a.position[r] = p;
}

// A work item: `at`, the first of its vectors or of its places in a queue among those of cell c, which has `members` vectors from `start` on. One load says so, so that
// all that follows from it, the cell's head among it, is requested at once: a wave waits for memory twice before it scores, not four times.
struct NearItem {
    uint32_t c, start, at, members;
};
__device__ __forceinline__ bool near_item(const NearArgs& a, uint32_t slot, NearItem& it)
{
    if (slot >= a.slots) return false;
    const uint4 v = a.items[slot];
    it.c = uint32_t(__builtin_amdgcn_readfirstlane(int(v.x)));
    it.start = uint32_t(__builtin_amdgcn_readfirstlane(int(v.y)));
    it.at = uint32_t(__builtin_amdgcn_readfirstlane(int(v.z)));
    it.members = uint32_t(__builtin_amdgcn_readfirstlane(int(v.w)));
    return it.c < a.K;
}

// t(x), enlarged by more than the rounding of the two distances (the roots are within 1 ulp, those of subnormal numbers zero)
__device__ __forceinline__ float cell_bound(float to_centre, float to_hinted)
{
    return (to_centre + to_hinted * 1.001f) * 1.00001f + 3e-19f;
}
template <int D>
__device__ __forceinline__ float rough_distance(const float (&x)[D], const float (&c)[D])
{
    return __builtin_amdgcn_sqrtf(direct_sqdist<D>(x, c));
}

// ---- near vectors, d = 4: scores over the list, rows broadcast from LDS, one lane per vector (up to 4) ----------------
// What is scored is ||c' - c||^2 - 2 (x - c).(c' - c), c the cell's centroid: four multiply-adds a pair, and numbers no larger than the cell, so
// that fp32 tells all but a few candidates apart. Four entries of the list are a group; a group's minimum, with its number in the low 5 bits, goes into the running
// best and second best. The best group's four are then compared in direct form; a vector whose second best comes within the guard band is decided in direct form over
// the whole list, 64 entries at a time.
// Guard band: let a = ||x - c||. c is on its own list, so the nearest centroid c* has ||x - c*|| <= a, and whatever rivals it ||c' - c|| <= 2 a. The differences
// are rounded once (2^-24 of each), norm and products add up to 72 x 2^-24 a^2 in a score, direct-form distances are within 8 x 2^-24 a^2 of theirs: 160 x 2^-24 a^2
// for two candidates, of which 200 are taken; a tag takes 2^-18 of a score. Scores among the subnormal numbers are within 1e-37, always.
// Bound: vector instructions and, as much, LDS, which takes 8 clocks to give 64 lanes the same 16 bytes. Multiply-adds issue in 2 clocks, minima, compares and
// selects in 4 (measured with 8 waves per SIMD), so this is 13 clocks a pair where direct form over the list, a compare and two selects took 34; a set of 64
// vectors takes 268 instructions beside its pairs (bounds, the best four, what is written), nearly as many as for them. N = 11 M, K = 65536 (lists of 43 entries; 60 are aimed at now) 0.147 -> 0.129 ms, 4.2 M, K = 4096 0.061 -> 0.045. A workgroup is one wave,
// as in the kernels for d = 8: two in five items are empty or short, and in a workgroup of four the room of those waves waits for the longest. Three sets of 64 to an
// item leave six waves to a SIMD, four leave four: 0.153. Rows that are loaded again after the scan for the sake of two more waves, 0.153.
// Tried with the direct form: entries in the order of their distance and vectors in the order of t(x), each 64 looking only as far as their largest
// t(x): a third fewer instructions in all, 0.20 ms where 0.15 were taken.
constexpr uint32_t kScanGroup = 4;
constexpr uint32_t kScanTag = 31;
constexpr uint32_t kScanRoom = Lists<4>::kCap1 + kScanGroup;
static_assert(Lists<4>::kCap1 <= (kScanTag + 1) * kScanGroup, "the number of a group fits its tag");
template <int NV>
__device__ __forceinline__ void scan_list(const float4* to, const float* norms, uint32_t groups, const float (&y)[NV][4], float (&best)[NV], float (&second)[NV])
{
    for (uint32_t g = 0; g < groups; ++g) {
        const float4 n4 = *reinterpret_cast<const float4*>(norms + g * kScanGroup);
        const float n[kScanGroup] = {n4.x, n4.y, n4.z, n4.w};
        float4 r[kScanGroup];
#pragma unroll
        for (uint32_t u = 0; u < kScanGroup; ++u) r[u] = to[g * kScanGroup + u];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            float s[kScanGroup];
#pragma unroll
            for (uint32_t u = 0; u < kScanGroup; ++u)
                s[u] = __builtin_fmaf(y[v][3], r[u].w, __builtin_fmaf(y[v][2], r[u].z, __builtin_fmaf(y[v][1], r[u].y, __builtin_fmaf(y[v][0], r[u].x, n[u]))));
            const float m = __builtin_fminf(__builtin_fminf(__builtin_fminf(s[0], s[1]), s[2]), s[3]);
            take_score(best[v], second[v], __uint_as_float((__float_as_uint(m) & ~kScanTag) | g));
        }
    }
}

__global__ __launch_bounds__(64) void near_direct_kernel(NearArgs a)
{
    constexpr int D = 4;
    using L = Lists<D>;
    __shared__ float4 rows[kScanRoom], to[kScanRoom];   // of the list's entries: the centroid, -2 (c' - c) ...
    __shared__ __attribute__((aligned(16))) float norms[kScanRoom];   // ... ||c' - c||^2 ...
    __shared__ __attribute__((aligned(16))) uint32_t ids[kScanRoom];  // ... and the index
    const int lane = threadIdx.x;
    NearItem it;
    if (!near_item(a, blockIdx.x, it)) return;
    const uint32_t c = it.c, first = it.start + it.at, n = min(kCellItem, it.members - it.at);
    // of this item, by place within it
    const float4* X = reinterpret_cast<const float4*>(a.X) + first;
    uint32_t* idx = a.idx + first;
    float* dmin = a.dmin != nullptr ? a.dmin + first : nullptr;
    const uint16_t* list = a.lists + size_t(c) * L::kCap;
    const CellHead head = a.heads[c];
    float cc_row[D];
    load_row<D>(a.C + size_t(c) * D, cc_row);
    static_assert(L::kCap == 128, "two entries of a list per lane");
    const uint32_t listed[2] = {list[lane], list[64 + lane]};   // (past the list's end: whatever lies there)
    float tm = 0.0f;
    auto sets = [&](auto of) {   // of 64 vectors
        constexpr int NV = decltype(of)::value;
        float x[NV][D], y[NV][D], best[NV], second[NV], centre[NV], ch[NV][D];
        uint32_t hint[NV];
        bool near[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint32_t i = min(uint32_t(v * 64 + lane), n - 1);
            const float4 t4 = X[i];
            x[v][0] = t4.x; x[v][1] = t4.y; x[v][2] = t4.z; x[v][3] = t4.w;
            hint[v] = idx[i];
        }
        // lists are complete unless they ran out of room
        const bool usable = lists_exist(a.hdr) && head.n1 <= L::kCap1;
        const float R = usable ? head.r1 : -1.0f;
        const uint32_t len = usable ? head.n1 : 0u, groups = (len + kScanGroup - 1) / kScanGroup;
        float4 row[2];
        uint32_t id[2];
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            const float qnan = __uint_as_float(0x7fc00000u);   // past the list: never the nearest
            row[q] = make_float4(qnan, qnan, qnan, qnan);
            id[q] = 0;
            if (q * 64 + lane < len) {
                row[q] = reinterpret_cast<const float4*>(a.csorted)[listed[q]];
                id[q] = a.cperm[listed[q]];
            }
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) load_row<D>(a.C + size_t(min(hint[v], a.K - 1)) * D, ch[v]);
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            const uint32_t e = q * 64 + lane;
            if (e >= groups * kScanGroup) break;
            const bool on = e < len;
            const float r[D] = {row[q].x, row[q].y, row[q].z, row[q].w}, norm = direct_sqdist<D>(r, cc_row);
            const float4 step = make_float4(-2.0f * (r[0] - cc_row[0]), -2.0f * (r[1] - cc_row[1]), -2.0f * (r[2] - cc_row[2]), -2.0f * (r[3] - cc_row[3]));
            rows[e] = row[q];
            to[e] = on ? step : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            norms[e] = on ? norm : 1e38f;
            ids[e] = id[q];
        }
        wave_order();
#pragma unroll
        for (int v = 0; v < NV; ++v) {
#pragma unroll
            for (int j = 0; j < D; ++j) y[v][j] = x[v][j] - cc_row[j];
            centre[v] = direct_sqdist<D>(x[v], cc_row);
            const float t = cell_bound(__builtin_amdgcn_sqrtf(centre[v]), rough_distance<D>(x[v], ch[v]));
            near[v] = t <= R;
            if (uint32_t(v * 64 + lane) < n) tm = __builtin_fmaxf(tm, t);
            best[v] = second[v] = 3e38f;
        }
        scan_list<NV>(to, norms, groups, y, best, second);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint32_t o = v * 64 + lane, p = first + o;
            const bool live = o < n;
            uint32_t k = 0xffffffffu;
            float bd = INFINITY;
            if (groups != 0) {   // the best group in direct form: among equals the lowest index wins
                const uint32_t e0 = min(__float_as_uint(best[v]) & kScanTag, groups - 1) * kScanGroup;
                const uint4 i4 = *reinterpret_cast<const uint4*>(ids + e0);
                const uint32_t id[kScanGroup] = {i4.x, i4.y, i4.z, i4.w};
                float d[kScanGroup];
#pragma unroll
                for (uint32_t u = 0; u < kScanGroup; ++u) {
                    const float4 t = rows[e0 + u];
                    const float cr[D] = {t.x, t.y, t.z, t.w};
                    d[u] = direct_sqdist<D>(x[v], cr);
                }
                bd = __builtin_fminf(__builtin_fminf(__builtin_fminf(d[0], d[1]), d[2]), d[3]);
#pragma unroll
                for (uint32_t u = 0; u < kScanGroup; ++u) k = d[u] == bd ? min(k, id[u]) : k;
                const float band = 1.2e-5f * centre[v] + 3.814697265625e-06f * (__builtin_fabsf(best[v]) + __builtin_fabsf(second[v])) + 1e-37f;
                unsigned long long todo = __ballot(live && near[v] && !(second[v] - best[v] > band));
                while (todo != 0) {
                    const int src = __ffsll(static_cast<long long>(todo)) - 1;
                    todo &= todo - 1;
                    float z[D];
#pragma unroll
                    for (int j = 0; j < D; ++j) z[j] = __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(__float_as_uint(x[v][j])), src)));
                    unsigned long long key = ~0ull;
                    for (uint32_t e = lane; e < len; e += 64) {
                        const float4 t = rows[e];
                        const float cr[D] = {t.x, t.y, t.z, t.w};
                        const unsigned long long w = (static_cast<unsigned long long>(__float_as_uint(direct_sqdist<D>(z, cr))) << 32) | ids[e];
                        key = w < key ? w : key;
                    }
                    for (int off = 32; off > 0; off >>= 1) {
                        const unsigned long long w = __shfl_xor(key, off, 64);
                        key = w < key ? w : key;
                    }
                    if (lane == src) {
                        k = uint32_t(key & 0xffffffffull);
                        bd = __uint_as_float(uint32_t(key >> 32));
                    }
                }
            }
            if (live && near[v]) {
                idx[o] = k;
                if (dmin != nullptr) dmin[o] = bd;
            }
            if (live && !near[v]) mark_far(a, p);
            if (a.changed != nullptr) {
                const bool moved = live && (!near[v] || k != hint[v]);
                if (moved) a.prev_out[p] = hint[v];
                or_bits(a.changed, first + v * 64, __ballot(moved), lane);
            }
        }
    };
    static_assert(kCellItem <= 4 * 64, "at most four sets");
    switch ((n + 63) / 64) {
        case 1: sets(std::integral_constant<int, 1>{}); break;
        case 2: sets(std::integral_constant<int, 2>{}); break;
        case 3: sets(std::integral_constant<int, 3>{}); break;
        default:
            if constexpr (kCellItem > 192) sets(std::integral_constant<int, 4>{});
    }
    for (int off = 32; off > 0; off >>= 1) tm = __builtin_fmaxf(tm, __shfl_xor(tm, off, 64));
    if (lane == 0) atomicMax(&a.heads[c].tmax, __float_as_uint(tm));
}

// ---- near vectors, d = 8: matrix cores over the list -----------------------------------------------------------------
// A wave takes up to 64 vectors of one cell and works alone. The operands of the list's centroids (64 bytes each, one cache
// line) are laid out for v_mfma_f32_16x16x32_f16: 32 k slots hold the 24 products of d = 8 and sigma ||c||^2, so that scores
// need no accumulator to start from; the wave gathers them through LDS. Four tiles of 16 centroids are folded
// row by row: the minimum of the four scores of a row, with the row in the low 4 bits, goes into the running best and second best, 21 vector
// instructions per 1024 scores. The winner is then known up to 4 centroids: as many direct-form distances. (Two by two it took 35 instructions and two distances: 29 M
// vectors 13.6 + 13.5 ms a fit, now 13.2 + 12.6. Half of the requests to L2, which are what bounds it now, 0.3 per clock and compute unit, are operands of the lists, a
// quarter those rows.) What the tag costs in precision (2^-19 of a score) goes into the guard band, as does twice the accumulation bound (this instruction is
// within 4.5 x 2^-24 of the sum of its terms in tests/test_gpu_mfma_bound16.py; 16 is assumed); a vector whose second best
// comes within the band is decided in direct form over the list, 64 centroids at a time.
// Lists hold indices here, in the order of the codebook: nothing has to be looked up for the winner, and what a list that runs out of room in the first iteration keeps of
// its ball is a fair share of it, where positions in the norm order left the ball's far side out (far vectors of the first two E-steps 7.6 -> 5.0 ms).
// Vectors between r1 and r2 are queued by cell and scored over the whole list in a second launch (MID), 64 per wave.
// Inputs that are no fp16 numbers take two operands: fp16 part and rest, 22 bits or more; the band grows accordingly.
// Measured at N = 29 M, K = 65536 (list of 400, 1500 with the outer part): 1.9 ms per E-step that scores every vector, 0.9 to 1.9
// + 1.0 to 1.8 ms with 0.36 to sort out those that need not be and 0.07 for the moves of the lists; N = 2.8 M: 0.20 ms +
// 0.09 ms, where the windowed kernel takes 53 ms and 1.6 ms. What bounds it is the chain of dependent loads of a wave (cell,
// list, operands, scores, rows), so a wave works alone and keeps 64 vectors at four waves per SIMD: workgroups that shared
// the list through LDS, 128 vectors per wave, took 6.1 to 7.8 ms for the same.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kVT = 4;                    // tiles of 16 vectors per wave
constexpr uint32_t kSetVectors = 16 * kVT;
constexpr uint32_t kGroup = 64;           // list entries folded together: 4 tiles of 16
constexpr uint32_t kTag = 15;

struct Scores {
    float best[kVT], second[kVT];
    uint32_t grp[kVT];
};

__device__ __forceinline__ void clear_scores(Scores& s)
{
#pragma unroll
    for (int vt = 0; vt < kVT; ++vt) {
        s.best[vt] = INFINITY;
        s.second[vt] = INFINITY;
        s.grp[vt] = 0;
    }
}

// The lane's part of a vector's operand: k slots 8 g .. 8 g + 7 (g = 0 .. 2: the products with parts 0 .. 2 of the centroids'
// components; g = 3: the multipliers of the norm's parts)
__device__ __forceinline__ f16x8 near_operand(const float (&x)[8], int g)
{
    f16x8 b;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const _Float16 fixed = j == 0 ? _Float16(256.0f) : (j == 1 ? _Float16(0.125f) : (j == 2 ? _Float16(6.103515625e-05f) : _Float16(0.0f)));
        b[j] = g < 3 ? _Float16(-2.0f * x[j]) : fixed;
    }
    return b;
}

// LOW: the operands' lower parts (64 lanes apart) are added first.
template <int NVT, bool LOW>
__device__ __forceinline__ void score_group(const f16x8 (&a)[4], const f16x8 (&b)[kVT], const f16x8* low, uint32_t row0, uint32_t group, float minus_inf,
                                            Scores& s)
{
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) {
        f32x4 r[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            r[t] = zero;
            if constexpr (LOW) r[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t], low[vt * 64], zero, 0, 0, 0);
            r[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t], b[vt], r[t], 0, 0, 0);
        }
        const float before = s.best[vt];
        auto quad = [&](int i) {
            // median with -inf = minimum of two: fminf on fresh matrix results costs two more instructions to quiet them (that of three does not)
            const float m = __builtin_fminf(__builtin_fminf(__builtin_amdgcn_fmed3f(r[0][i], r[1][i], minus_inf), r[2][i]), r[3][i]);
            return __uint_as_float((__float_as_uint(m) & ~kTag) | (row0 + i));
        };
#pragma unroll
        for (int i = 0; i < 4; i += 2) {   // two at once: the second best of all is that of {best, u, v} or the second best so far
            const float u = quad(i), v = quad(i + 1), middle = __builtin_amdgcn_fmed3f(s.best[vt], u, v);
            asm("v_min_f32 %0, %1, %2" : "=v"(s.second[vt]) : "v"(s.second[vt]), "v"(middle));
            s.best[vt] = __builtin_fminf(__builtin_fminf(s.best[vt], u), v);
        }
        s.grp[vt] = s.best[vt] < before ? group : s.grp[vt];
    }
}

// Most that a centroid of a cell's list has moved since the E-step before: within r1, and on the whole list. One wave per cell, the moves of
// all centroids in LDS.
constexpr int kMovedThreads = 1024;
__global__ __launch_bounds__(kMovedThreads) void cell_moved_kernel(const uint16_t* __restrict__ moves, uint32_t K, const CellHead* __restrict__ heads,
                                                                   const uint16_t* __restrict__ lists, uint32_t* __restrict__ moved,
                                                                   const WsHeader* __restrict__ hdr)
{
    using L = Lists<8>;
    extern __shared__ __attribute__((aligned(16))) uint16_t by_index[];
    if (!lists_exist(hdr)) return;
    for (uint32_t i = threadIdx.x; i < (K + 7) / 8; i += kMovedThreads)   // (the buffer is a whole number of 256 bytes)
        reinterpret_cast<uint4*>(by_index)[i] = reinterpret_cast<const uint4*>(moves)[i];
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, waves = gridDim.x * (kMovedThreads / 64);
    for (uint32_t c = blockIdx.x * (kMovedThreads / 64) + (threadIdx.x >> 6); c < K; c += waves) {
        const uint32_t all1 = heads[c].n1, n1 = all1 != 0xffffffffu ? min(all1, L::kCap1) : 0u, n2 = min(heads[c].n2, L::kCap2);   // (a cell without a list: ~0)
        const uint16_t* list = lists + size_t(c) * L::kCap;
        auto most = [&](const uint16_t* from, uint32_t n) {
            uint32_t m = 0;
            for (uint32_t e0 = lane * 8; e0 < n; e0 += 512) {
                const uint4 v = *reinterpret_cast<const uint4*>(from + e0);
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (uint32_t q = 0; q < 8; ++q) {
                    const uint32_t id = (w[q / 2] >> (16 * (q & 1))) & 0xffffu;
                    if (e0 + q < n) m = max(m, uint32_t(by_index[id]));
                }
            }
            for (int off = 32; off > 0; off >>= 1) m = max(m, uint32_t(__shfl_xor(int(m), off, 64)));
            return m;
        };
        const uint32_t m1 = most(list, n1), m2 = most(list + L::kCap1, n2);
        if (lane == 0) moved[c] = m1 | (max(m1, m2) << 16);
    }
}

// Codes that cannot change. An E-step leaves for every vector x it decided on its cell's list, with nearest centroid k, a bound on the
// distance of all others: what else is on the list is no nearer than the second best, what is not on it lies beyond R from the cell's
// centroid c, hence beyond R - ||x - c|| from x. Until the next E-step the centroids move; of those that can be nearest then (the cell's new
// list) none has come nearer by more than the largest move among them. Where the bound less that move is above the new ||x - c_k||, k stays,
// its distance is known, and the new bound is the smaller of what is left of the old one and R - ||x - c||.
// Every bound gives way by more than its rounding (1e-5 of the distances behind it, 3e-19 for squares among the subnormal numbers), so the
// others' distances are larger in fp32 as well: no tie, the same code.
__device__ __forceinline__ float bound_of(float others, float R, float to_centre)
{
    return __builtin_fminf(others, R * 0.99999f - to_centre * 1.00001f) - 3e-19f;
}

// The vectors of an item, one lane each: which are near (returned), to the mid queue, to the far ones, or done.
__device__ __forceinline__ bool sort_out(const NearArgs& a, uint32_t c, const CellHead& head, uint32_t first, uint32_t n, int lane,
                                         const float (&x)[8], uint32_t hint)
{
    constexpr int D = 8;
    using L = Lists<D>;
    const bool on = uint32_t(lane) < n;
    const uint32_t p = first + min(uint32_t(lane), n - 1);
    float row[D], ch[D];
    const float was = a.bounded ? from_half(a.bound[p]) : 0.0f;
    const uint32_t moved = a.bounded ? a.moved[c] : 0u;
    load_row<D>(a.C + size_t(c) * D, row);
    load_row<D>(a.C + size_t(min(hint, a.K - 1)) * D, ch);
    // lists are complete unless they ran out of room
    const bool usable = lists_exist(a.hdr) && head.n1 <= L::kCap1 && head.n1 > 0;
    const float r1 = usable ? head.r1 : -1.0f, r2 = usable && head.n2 <= L::kCap2 ? fmaxf(head.r1, head.r2) : r1;
    const float sq = direct_sqdist<D>(x, ch), to_hinted = __builtin_amdgcn_sqrtf(sq), to_centre = rough_distance<D>(x, row);
    const float t = cell_bound(to_centre, to_hinted);
    bool near = on && t <= r1, mid = on && !near && t <= r2;
    const bool far = on && !near && !mid;
    if (a.bounded) {
        const float others = was - from_half(near ? moved & 0xffffu : moved >> 16) - 2e-7f * was;
        if ((near || mid) && to_hinted * 1.00002f + 6e-19f < others) {
            if (a.dmin != nullptr) a.dmin[p] = sq;
            a.bound[p] = lower_half(bound_of(others, near ? r1 : r2, to_centre));
            near = mid = false;
        }
    }
    float tm = on ? t : 0.0f;
    for (int off = 32; off > 0; off >>= 1) tm = __builtin_fmaxf(tm, __shfl_xor(tm, off, 64));
    if (lane == 0) atomicMax(&a.heads[c].tmax, __float_as_uint(tm));
    const unsigned long long mids = __ballot(mid);
    if (mids != 0) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&a.heads[c].mids, uint32_t(__popcll(mids)));
        at = uint32_t(__builtin_amdgcn_readfirstlane(int(at)));
        if (mid) a.queues[head.start + head.members - 1 - __builtin_amdgcn_mbcnt_hi(uint32_t(mids >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mids), at))] = p;
    }
    if (far) {
        mark_far(a, p);
        if (a.bound != nullptr) a.bound[p] = 0;
    }
    if (a.changed != nullptr) {
        if (far) a.prev_out[p] = hint;
        or_bits(a.changed, first, __ballot(far), lane);
    }
    return near;
}

// Near vectors that have to be scored, to their cell's queue: 64 of them then share a gather of the list.
__global__ __launch_bounds__(kThreads) void near_sort_out_kernel(NearArgs a)
{
    constexpr int D = 8;
    const int lane = threadIdx.x & 63;
    NearItem it;
    if (!near_item(a, blockIdx.x * kWaves + (threadIdx.x >> 6), it)) return;
    const uint32_t c = it.c, first = it.start + it.at, n = min(kSetVectors, it.members - it.at);
    const CellHead head = a.heads[c];
    const uint32_t p = first + min(uint32_t(lane), n - 1), hint = a.idx[p];
    float x[D];
    load_row<D>(a.X + size_t(p) * D, x);
    const bool near = sort_out(a, c, head, first, n, lane, x, hint);
    const unsigned long long some = __ballot(near);
    if (some == 0) return;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&a.queued_near[c], uint32_t(__popcll(some)));
    at = uint32_t(__builtin_amdgcn_readfirstlane(int(at)));
    if (near) a.queues[head.start + __builtin_amdgcn_mbcnt_hi(uint32_t(some >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(some), at))] = p;
}

enum NearMode : int { kNear, kQueued, kMid, kHint };   // kNear: sorts its vectors out itself; kQueued: the near ones of near_sort_out_kernel; kHint: the best of the list within r1 (or what of it there is room for) for every vector of
                                              // the cell, no matter whether that is its nearest centroid
template <int MODE>
__global__ __launch_bounds__(64, 4) void near_mfma_kernel(NearArgs a)
{
    constexpr bool MID = MODE == kMid, QUEUED = MID || MODE == kQueued;
    constexpr int D = 8;
    using L = Lists<D>;
    const int lane = threadIdx.x, g = lane >> 4, n16 = lane & 15;
    NearItem it;
    if (!near_item(a, blockIdx.x, it)) return;
    const uint32_t c = it.c;
    const CellHead head = a.heads[c];
    const uint32_t first = MID ? it.start + it.members - 1 - it.at : it.start + it.at;   // of the vectors, or of the places in the queue
    const uint32_t have = MID ? head.mids : (QUEUED ? a.queued_near[c] : it.members);
    if (it.at >= have) return;
    const uint32_t n = min(kSetVectors, have - it.at);
    // lists are complete unless they ran out of room
    const bool usable = lists_exist(a.hdr) && head.n1 <= L::kCap1 && head.n1 > 0;
    const bool whole = usable && head.n2 <= L::kCap2;
    const float r1 = usable ? head.r1 : -1.0f, r2 = whole ? fmaxf(head.r1, head.r2) : r1;
    const uint32_t len1 = MODE == kHint ? (lists_exist(a.hdr) && head.n1 != 0xffffffffu ? min(head.n1, L::kCap1) : 0u) : (usable ? head.n1 : 0u);
    const uint32_t len = MID && whole ? head.n1 + head.n2 : len1;
    if (MODE == kHint && len == 0) return;
    const uint16_t* list = a.lists + size_t(c) * L::kCap;
    auto entry = [&](uint32_t e) { return uint32_t(list[!MID || e < len1 ? e : L::kCap1 + (e - len1)]); };
    const uint32_t cmax_bits = a.hdr->cmax_bits;
    const float sigma = __builtin_ldexpf(1.0f, centroid_scale_log2(cmax_bits, D));
    const float sigma_cmax = sigma * __uint_as_float(cmax_bits);
    float minus_inf;   // out of the compiler's sight, which would turn a median with it back into fminf
    asm("s_mov_b32 %0, 0xff800000" : "=s"(minus_inf));
    const uint32_t row0 = 4 * g;
    const bool f16 = a.hdr->x_not_f16 == 0;
    __shared__ f16x8 low[kVT * 64];   // other inputs: what a vector's operand has below its fp16 part
    __shared__ f16x8 turn[4 * 64];   // the operands of a group of list entries
    f16x8 b[kVT];
    Scores s;
    clear_scores(s);

    // ---- the vectors: operands, bounds and previous codes (one vector per lane)
    bool on = uint32_t(lane) < n;
    auto position = [&](uint32_t v) { return QUEUED ? a.queues[MID ? first - v : first + v] : first + v; };
    const uint32_t p = position(min(uint32_t(lane), n - 1));
    float x[D];
    load_row<D>(a.X + size_t(p) * D, x);
    const uint32_t hint = a.idx[p];
    // The four lanes with a piece of a vector's operand take its row from LDS, where rows are 48 bytes apart: eight lanes meet no bank twice. From memory these
    // rows were as many L1 accesses as the gather of 450 list entries (29 M vectors: 89.9 -> 89.1 ms a fit).
    float4* const xs = reinterpret_cast<float4*>(turn);
    xs[lane * 3] = make_float4(x[0], x[1], x[2], x[3]);
    xs[lane * 3 + 1] = make_float4(x[4], x[5], x[6], x[7]);
    wave_order();
#pragma unroll
    for (int vt = 0; vt < kVT; ++vt) {
        const float4 lo4 = xs[(vt * 16 + n16) * 3], hi4 = xs[(vt * 16 + n16) * 3 + 1];
        float xo[D] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
        b[vt] = near_operand(xo, g);
        if (!f16) {
#pragma unroll
            for (int j = 0; j < D; ++j) xo[j] -= float(_Float16(xo[j]));
            f16x8 lo = near_operand(xo, g);
#pragma unroll
            for (int j = 0; j < 8; ++j) lo[j] = g < 3 ? lo[j] : _Float16(0.0f);
            low[vt * 64 + lane] = lo;
        }
    }
    if constexpr (MODE == kNear) {
        on = sort_out(a, c, head, first, n, lane, x, hint);
        if (!__any(on)) return;
    }
    // ---- scores: 64 list entries at a time, the operands of a group gathered while the one before it is scored, its list
    // entries one group earlier; past the end, the operand that never wins
    {
        const uint32_t groups = (len + kGroup - 1) / kGroup, tiles = (n + 15) / 16;
        // Four neighbouring lanes to an operand of 64 bytes, which L1 serves at once, and through LDS to the lanes where the product wants the pieces, those of
        // row r rotated so that eight lanes meet no bank twice. L1 was the bound while every lane loaded its piece of a row of its own: 56
        // accesses a load, one each clock of the kernel. 29 M vectors, K = 65536: 1.40 and 1.43 ms (near and between r1 and r2) -> 1.27 and
        // 1.27, 2.8 M 0.221 and 0.131 -> 0.204 and 0.112; of that, a half for one load of list entries per group in place of four.
        const uint32_t row = lane >> 2, from = (lane ^ (row + (row >> 2))) & 3u, to_row = 4 * n16 + ((g ^ (n16 + (n16 >> 2))) & 3);
        uint32_t begins = 0;   // where the operand of entry `lane` of a group does: a scalar and 32 bits of address per request, 64-bit additions otherwise
        f16x8 av[4];
        auto entries = [&](uint32_t gr) {
            const uint32_t e = gr * kGroup + lane, at = entry(min(e, max(len, 1u) - 1u));
            begins = (e < len ? at : a.K) * 64;
        };
        auto gather = [&]() {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t at = uint32_t(__shfl(int(begins), 16 * t + int(row), 64)) | from * 16;
                asm volatile("" : "+v"(at));
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a.flat + at), (__attribute__((address_space(3))) void*)(turn + t * 64), 16, 0, 0);
            }
        };
        // A loop for each number of tiles: one that chose in every group kept scores in other registers for each choice, 25 copies beside 80 instructions.
        // Lists of 2.8 M vectors 188 / 179 us (three tiles of four where cells hold 43 vectors), bf16 layer of 4096^2 at g = 6 16.48 / 16.30 ms, 8192 x 28672 77.7 / 77.0.
        // (QUEUED: the loop of three tiles leaves a pair of registers in scratch memory while it runs, once per wave.)
        auto score = [&](auto tiles, auto low_too) {
            entries(0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the rows have been read
            gather();
            entries(1);
            for (uint32_t gr = 0; gr < groups; ++gr) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the operands have landed
#pragma unroll
                for (int t = 0; t < 4; ++t) av[t] = turn[t * 64 + to_row];
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // ... and are read before the next ones land there
                gather();
                entries(gr + 2);
                score_group<decltype(tiles)::value, decltype(low_too)::value>(av, b, low + lane, row0, gr, minus_inf, s);
            }
        };
        if (!f16) score(std::integral_constant<int, 4>{}, std::true_type{});
        else if (tiles == 1) score(std::integral_constant<int, 1>{}, std::false_type{});
        else if (tiles == 2) score(std::integral_constant<int, 2>{}, std::false_type{});
        else if (tiles == 3) score(std::integral_constant<int, 3>{}, std::false_type{});
        else score(std::integral_constant<int, 4>{}, std::false_type{});
    }
    // ---- best, second best and group over the four lanes that share a vector; lane (n16, g) takes vector n16 of tile g
    float best = 0.0f, second = 0.0f;
    uint32_t grp = 0;
#pragma unroll
    for (int t = 0; t < kVT; ++t) {
        float tb = s.best[t], ts = s.second[t];
        uint32_t tg = s.grp[t];
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float ob = __shfl_xor(tb, off, 64), os = __shfl_xor(ts, off, 64);
            const uint32_t og = uint32_t(__shfl_xor(int(tg), off, 64));
            ts = __builtin_fminf(__builtin_fminf(ts, os), __builtin_fmaxf(tb, ob));
            tg = ob < tb ? og : tg;   // scores of different lanes differ in their row number
            tb = __builtin_fminf(tb, ob);
        }
        best = g == t ? tb : best;
        second = g == t ? ts : second;
        grp = g == t ? tg : grp;
    }
    // ---- the decision
    const uint32_t e0 = grp * kGroup + (__float_as_uint(best) & kTag);
    uint32_t at[4];
    float of[4];
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
        const uint32_t e = e0 + 16 * t;
        at[t] = entry(min(e, len - 1));
        float row[D];
        load_row<D>(a.C + size_t(at[t]) * D, row);
        of[t] = direct_sqdist<D>(x, row);
        if (e >= len) of[t] = INFINITY;
    }
    float d = __builtin_fminf(__builtin_fminf(__builtin_fminf(of[0], of[1]), of[2]), of[3]);
    float rival = INFINITY;   // the second of them
    uint32_t k = a.K - 1;
    bool seen = false;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const bool is = of[t] == d;
        if (!is || seen) rival = __builtin_fminf(rival, of[t]);
        k = is ? (seen ? min(k, at[t]) : at[t]) : k;
        seen |= is;
    }
    if constexpr (MODE == kHint) {
        if (on) a.idx[p] = k;
        return;
    }
    float xn = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) xn = __builtin_fmaf(x[j], x[j], xn);
    float slack = 1.9073486328125e-06f * (__builtin_fabsf(best) + __builtin_fabsf(second));   // the tags: 2^-19
    if (!f16) slack += 16.0f * sigma_cmax * (2.384185791015625e-07f * __builtin_sqrtf(xn) + 1.6e-07f);   // what x has beyond 22 bits
    const float delta = f16_guard_band<D, 3, true, 16>(x, d, sigma, sigma_cmax) + slack;
    const bool clear = (second - best) > delta;
    unsigned long long todo = __ballot(on && !clear);
    while (todo != 0) {  // direct form over the whole list, one vector at a time
        const int src = __ffsll(static_cast<long long>(todo)) - 1;
        todo &= todo - 1;
        float y[D];
#pragma unroll
        for (int j = 0; j < D; ++j) y[j] = __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(__float_as_uint(x[j])), src)));
        unsigned long long key = ~0ull;
#pragma unroll 4
        for (uint32_t le = lane; le < len; le += 64) {
            const uint32_t id = entry(le);
            float c2[D];
            load_row<D>(a.C + size_t(id) * D, c2);
            const unsigned long long v = (static_cast<unsigned long long>(__float_as_uint(direct_sqdist<D>(y, c2))) << 32) | id;
            key = v < key ? v : key;
        }
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long v = __shfl_xor(key, off, 64);
            key = v < key ? v : key;
        }
        if (lane == src) {
            k = uint32_t(key & 0xffffffffull);
            d = __uint_as_float(uint32_t(key >> 32));
        }
    }
    if (on) {
        a.idx[p] = k;
        if (a.dmin != nullptr) a.dmin[p] = d;
    }
    if (on && a.bound != nullptr) {
        // others: the next of the winner's four, and whatever scored no better than the second best four. The band is the one of a
        // centroid twice as far as the winner, which is as much as is made of the scores of those beyond.
        float row[D];
        load_row<D>(a.C + size_t(c) * D, row);
        const float scored = (second - f16_guard_band<D, 3, true, 16>(x, 4.0f * d, sigma, sigma_cmax) - slack) / sigma + xn * 0.999999f;
        const float sq = __builtin_fminf(__builtin_fminf(scored, 4.0f * d), rival);
        const float others = clear ? __builtin_sqrtf(__builtin_fmaxf(0.0f, sq)) * 0.99999f : 0.0f;
        a.bound[p] = lower_half(bound_of(others, MID ? r2 : r1, rough_distance<D>(x, row)));
    }
    if (a.changed != nullptr) {
        const bool moved = on && k != hint;
        if (moved) a.prev_out[p] = hint;
        if constexpr (QUEUED) {
            if (moved) or_bit(a.changed, p);
        } else {
            or_bits(a.changed, first, __ballot(moved), lane);
        }
    }
}

// ---- far vectors ------------------------------------------------------------------------------------------------------
// Far vectors among every 8192 norm ranks, and among the pieces of 2048 of them before each.
constexpr uint32_t kFarPiece = 64;                     // words of the bitmap
constexpr uint32_t kFarPieces = kThreads / kFarPiece;  // to a run of 8192 ranks
__global__ __launch_bounds__(kThreads) void far_count_kernel(const uint32_t* __restrict__ far_bits, uint32_t words, uint32_t* __restrict__ runs,
                                                             uint32_t* __restrict__ before)
{
    __shared__ uint32_t piece[kFarPieces];
    const uint32_t at_word = blockIdx.x * kThreads + threadIdx.x;
    uint32_t cnt = at_word < words ? uint32_t(__popc(far_bits[at_word])) : 0u;
    for (int off = kFarPiece / 2; off > 0; off >>= 1) cnt += uint32_t(__shfl_xor(int(cnt), off, 64));
    if (threadIdx.x % kFarPiece == 0) piece[threadIdx.x / kFarPiece] = cnt;
    __syncthreads();
    if (threadIdx.x > kFarPieces) return;
    uint32_t sum = 0;
    for (uint32_t i = 0; i < threadIdx.x; ++i) sum += piece[i];
    if (threadIdx.x < kFarPieces) before[blockIdx.x * kFarPieces + threadIdx.x] = sum;
    else runs[blockIdx.x] = sum;
}

// The flagged ranks, in order, to a dense list with their rows and previous codes, a piece per workgroup: far vectors are outliers
// and lie close together in the norm order (a workgroup per 8192 ranks: 17 to 24 us where 40 to 90 thousand of 4 M are far).
// Neighbours in the list are neighbours in norm, so those of a window need little more than each of them: the 4096 x 11008 fit
// spent 1.8 ms on its far vectors with them, 4.4 when runs of 8192 ranks lay in the order of their workgroups' arrival.
template <int D>
__global__ __launch_bounds__(kThreads) void far_compact_kernel(const uint32_t* __restrict__ far_bits, uint32_t words,
                                                               const uint32_t* __restrict__ runs, const uint32_t* __restrict__ before,
                                                               const uint32_t* __restrict__ position, const float* __restrict__ X,
                                                               const uint32_t* __restrict__ idx, WsHeader* hdr,
                                                               uint32_t* __restrict__ far_pos, float* __restrict__ far_x,
                                                               uint32_t* __restrict__ far_idx)
{
    __shared__ uint16_t offsets[kFarPiece * 32];
    __shared__ uint32_t total, wave_before[kWaves];
    const uint32_t run = blockIdx.x / kFarPieces;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t b = 0;
    for (uint32_t r = threadIdx.x; r < run; r += kThreads) b += runs[r];
    for (int off = 32; off > 0; off >>= 1) b += uint32_t(__shfl_xor(int(b), off, 64));
    if (lane == 0) wave_before[wave] = b;
    if (wave == 0) {
        const uint32_t at_word = blockIdx.x * kFarPiece + lane;
        const uint32_t word = uint32_t(lane) < kFarPiece && at_word < words ? far_bits[at_word] : 0u, cnt = __popc(word);
        uint32_t incl = cnt;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = uint32_t(__shfl_up(int(incl), off, 64));
            if (lane >= off) incl += t;
        }
        if (lane == 63) total = incl;
        uint32_t at = incl - cnt;
        for (uint32_t bits = word; bits != 0; bits &= bits - 1) offsets[at++] = uint16_t(lane * 32 + (__ffs(int(bits)) - 1));
    }
    __syncthreads();
    uint32_t to = before[blockIdx.x];
    for (int w = 0; w < kWaves; ++w) to += wave_before[w];
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) hdr->far_count = to + total;
    for (uint32_t e = threadIdx.x; e < total; e += kThreads) {
        const uint32_t p = position[blockIdx.x * (kFarPiece * 32) + offsets[e]];
        far_pos[to + e] = p;
        far_idx[to + e] = idx[p];
#pragma unroll
        for (int q = 0; q < D / 4; ++q)
            reinterpret_cast<float4*>(far_x + size_t(to + e) * D)[q] = reinterpret_cast<const float4*>(X + size_t(p) * D)[q];
    }
}

// Windows of the far vectors, a wave to each: the hull of what their distances to the previous codes leave of norms and projections, as in sort.hip, one
// lane to a shell. Runs that share a tracking group of the kernel that scores them become one, so that none is visited twice.
template <int D>
__global__ __launch_bounds__(kThreads) void far_window_kernel(const float* __restrict__ X, const uint32_t* __restrict__ hint, const float* __restrict__ C,
                                                              uint32_t N, uint32_t K, const uint32_t* __restrict__ key_starts, WsHeader* hdr,
                                                              uint2* __restrict__ windows)
{
    __shared__ uint32_t held[kWaves];
    const uint32_t far = hdr->far_count, tile = far_window_tile(hdr, D, N), base = shell_base(hdr->absmax_bits, D);
    const uint32_t whole = hdr->x_not_f16 != 0 ? kStageTiles : uint32_t(kSetGroup), lane = threadIdx.x & 63;
    uint32_t scored = 0;   // tiles, times vectors
    for (uint32_t w = blockIdx.x * kWaves + (threadIdx.x >> 6); w < (far + tile - 1) / tile; w += gridDim.x * kWaves) {
        float nlo = INFINITY, nhi = 0.0f, plo = INFINITY, phi = -INFINITY;
        for (uint32_t v = lane; v < tile; v += 64) {
            const uint32_t i = min(w * tile + v, far - 1);
            float x[D], c[D], s = 0.0f, prj;
            load_row<D>(X + size_t(i) * D, x);
            load_row<D>(C + size_t(min(hint[i], K - 1)) * D, c);
#pragma unroll
            for (int j = 0; j < D; ++j) s = __builtin_fmaf(x[j], x[j], s);
            const float nrm = __builtin_sqrtf(s), u = __builtin_sqrtf(direct_sqdist<D>(x, c)) * 1.001f + 1e-30f;
            (void)ordering_key<D>(x, nrm, base, prj);
            nlo = __builtin_fminf(nlo, nrm - u);
            nhi = __builtin_fmaxf(nhi, nrm + u);
            plo = __builtin_fminf(plo, prj - u);
            phi = __builtin_fmaxf(phi, prj + u);
        }
        for (int off = 32; off > 0; off >>= 1) {
            nlo = __builtin_fminf(nlo, __shfl_xor(nlo, off, 64));
            nhi = __builtin_fmaxf(nhi, __shfl_xor(nhi, off, 64));
            plo = __builtin_fminf(plo, __shfl_xor(plo, off, 64));
            phi = __builtin_fmaxf(phi, __shfl_xor(phi, off, 64));
        }
        const float slack = nhi < 3.0e38f ? 1e-5f * nhi : 0.0f;   // as in sort.hip
        nlo -= slack; nhi += slack; plo -= slack; phi += slack;
        const uint32_t smin = shell_of_key(nlo > 0.0f ? norm_key(nlo) : 0u, base), smax = shell_of_key(nhi < 3.0e38f ? norm_key(nhi) : 0xffffu, base);
        const bool wide = smax - smin + 1 > uint32_t(kFarWinSlots);
        uint32_t klo = smin << 7, khi = (smax << 7) | 127u, x = 0, y = 0;   // the run of this lane's shell, in tiles
        if (!wide) shell_cosine_run(smin + lane, base, plo, phi, klo, khi);
        if (lane <= (wide ? 0u : smax - smin) && klo <= khi) {
            const uint32_t first = key_starts[klo], end = key_starts[khi + 1];   // keys are ascending
            if (first < end) { x = first / 32; y = (end + 31) / 32; }
        }
        if (!__any(x < y)) {   // cannot happen: a hinted centroid lies inside its own runs
            x = 0;
            y = lane == 0 ? (K + 31) / 32 : 0u;
        }
        uint32_t reach = y;   // the furthest end of the runs up to this one
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = uint32_t(__shfl_up(int(reach), off, 64));
            if (lane >= uint32_t(off)) reach = max(reach, o);
        }
        const uint32_t before = uint32_t(__shfl_up(int(reach), 1, 64));
        const unsigned long long starts = __ballot(x < y && (lane == 0 || before == 0 || x / whole > (before - 1) / whole));
        const uint32_t n = uint32_t(__popcll(starts)), nth = uint32_t(__popcll(starts & ((2ull << lane) - 1)));   // runs up to this lane's
        uint2* out = windows + size_t(w) * kFarWinStride;
        const bool last = lane == 63 || ((starts >> (lane + 1)) & 1) != 0;   // of its run
        if ((starts >> lane) & 1) out[nth].x = x;
        if (last && nth > 0) out[nth].y = reach;
        uint32_t total = ((starts >> lane) & 1 ? 0u - x : 0u) + (last && nth > 0 ? reach : 0u);
        for (int off = 32; off > 0; off >>= 1) total += uint32_t(__shfl_xor(int(total), off, 64));
        if (lane == 0) out[0] = make_uint2(n, total);
        scored += total * min(tile, far - w * tile);
    }
    // statistics, in units of (512 vectors x 32 centroids)
    if (lane == 0) held[threadIdx.x >> 6] = scored;
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned long long all = 0;
    for (int v = 0; v < kWaves; ++v) all += held[v];
    if (all != 0) atomicAdd(&hdr->window_stages, (all + kWinTile / 2) / kWinTile);
}

// The far vectors' windowed E-step: a workgroup takes 32 VT vectors (a part of a window tile), its waves take turns at the
// window's tiles and load operands straight from the packed codebook. The kernel of assign_mfma_f16.hip gives 512
// vectors to 4 waves and shares every tile through LDS: better with many vectors, but the far ones are outliers, few, with
// windows that span much of the codebook, and left most of the chip without work.
// Bound: instructions. By the counters (d = 8, 29 M) 82 clocks per 1024 pairs at 1.9 GHz: 32 of the matrix cores, 11.2 vector instructions,
// 8 of which take the minimum of 16 scores; 4 or 16 waves, 128 or 256 vectors and the order of instructions changed that by 10 %. Operands
// are loaded a group ahead across the ends of runs, and the norms of d = 8
// pass through LDS, loaded by one lane each: 64 lanes that fetch 64 bytes each when their product needs them waited for L2 at every tile
// (96 cycles). Kernel time of a fit: 29 M vectors of 8 (1.0 to 2 M of them far, 10 iterations) 38.0 -> 27.3 ms, 11 M of 4 1.74 -> 1.28,
// 2.8 M of 6 (4 to 11 thousand far) 1.78 -> 1.02.
template <int D>
struct FarShape {
    static constexpr int kWaves = 8, kMostVT = D == 4 ? 4 : 8;
    static constexpr int kLds = kWaves * kMostVT * 64;
};

template <int D>
__global__ __launch_bounds__(64 * FarShape<D>::kWaves) void far_kernel(const float* __restrict__ X, const float* __restrict__ rows,
                                                                       const uint32_t* __restrict__ cperm, uint32_t all, uint32_t K,
                                                                       const char* __restrict__ packed, const uint2* __restrict__ windows,
                                                                       const uint32_t* __restrict__ far_pos, uint32_t* __restrict__ idx,
                                                                       float* __restrict__ dmin, WsHeader* hdr, uint32_t* __restrict__ refine_list)
{
    using F = FarShape<D>;
    __shared__ float x_best[F::kLds], x_second[F::kLds];
    __shared__ uint32_t x_grp[F::kLds];
    __shared__ __attribute__((aligned(16))) float norms[F::kWaves * 32 * kSetGroup];
    const uint32_t N = hdr->far_count;
    if (hdr->x_not_f16 != 0) return;
    const uint32_t tile = far_window_tile(hdr, D, all);
    auto sets = [&](auto vt) {
        score_sets<D, decltype(vt)::value, F::kWaves, true>(
            X, rows, cperm, N, K, packed, 0u, windows, tile, uint32_t(kFarWinStride), hdr->cmax_bits, x_best, x_second, x_grp, norms,
            [&](uint32_t i, bool mine, const float (&)[D], uint32_t k, float distance, bool safe) {
                if (!mine) return;
                const uint32_t p = far_pos[i];
                idx[p] = k;
                dmin[p] = distance;
                if (!safe) refine_list[atomicAdd(&hdr->refine_count, 1u)] = i;
            });
    };
    if (N <= kFarFew1) sets(std::integral_constant<int, 1>{});
    else if (N <= kFarFew2) sets(std::integral_constant<int, 2>{});
    else if (F::kMostVT == 4 || N <= kFarFew4) sets(std::integral_constant<int, 4>{});
    else sets(std::integral_constant<int, F::kMostVT>{});
}

// Whether the codes that cannot change are left out (d = 8): where that leaves fewer sets of 64 to a cell, which share a gather of its list
// (where a cell has one set at most, the gather stays). Fits, ms, without / with: N = 29 M, K = 65536 (447 vectors per centroid) 109.8 / 104.8;
// 4.2 M, K = 4096 (1024), 20 iterations 15.7 / 14.4, K = 16384 (256) 13.9 / 13.65, K = 32768 (128), 20 iterations 32.6 / 32.2; 4.9 M of 5,
// K = 35000 (140) 18.8 / 19.1; 2.8 M of 6, K = 65500 (43) 24.8 / 25.8. At d = 4 it cost more than it saved (near_direct_kernel of the
// 11 M fit: 40 % fewer vector instructions, 3.0 -> 3.4 ms, for the bounds and the second pass over what is left).
bool cells_bounded(uint64_t N, uint32_t d, uint32_t K) { return d == 8 && N >= 192ull * K; }

uint32_t item_of(uint32_t d) { return d == 4 ? kCellItem : kSetVectors; }

template <int D>
hipError_t cells_order_t(const float* X, const float* C, uint32_t N, uint32_t K, Workspace& w, bool first, bool last, float factor, hipStream_t s)
{
    const dim3 per_vector((N + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(cell_keys_kernel, per_vector, dim3(kThreads), 0, s, w.idx_sorted, N, w.vkeys, w.cell_order);
    if (hipError_t e = launch_sort_u16(w.vkeys, w.cell_order, w.vkeys_tmp, w.vperm_tmp, N, w.sort_hist, s); e != hipSuccess) return e;
    if (first) std::swap(w.idx_sorted, w.idx_prev);
    hipLaunchKernelGGL(cell_apply_kernel, per_vector, dim3(kThreads), 0, s, w.vkeys, N, w.cell_order, first ? nullptr : w.cell_rank,
                       w.vperm, w.vperm_tmp, last ? w.cell_position : nullptr, w.idx_sorted);
    std::swap(w.vperm, w.vperm_tmp);
    std::swap(w.cell_rank, w.cell_order);
    if (hipError_t e = launch_gather_rows(X, w.vperm, N, D, w.xsorted, s); e != hipSuccess) return e;
    hipLaunchKernelGGL(cell_starts_kernel, dim3((K + kThreads - 1) / kThreads), dim3(kThreads), 0, s, w.vkeys, N, K, w.cell_heads);
    const uint32_t item = item_of(D), slots = N / item + K;
    const float wider = D == 4 ? 1.0f : 1.28f;   // (kTarget2 / kTarget1)^(1/8)
    hipLaunchKernelGGL(cell_items_kernel<D>, dim3((K + kWaves - 1) / kWaves), dim3(kThreads), 0, s, w.cell_heads, K, slots, item, cell_items(w),
                       w.xsorted, w.idx_sorted, C, factor, factor * wider, first ? 1 : 0);
    if (first) {
        hipLaunchKernelGGL(cell_first_radius_kernel<D>, dim3((K + kWaves - 1) / kWaves), dim3(kThreads), 0, s, w.xsorted, w.idx_sorted,
                           w.cell_heads, C, K, factor, factor * wider);
        if (hipError_t e = launch_fill_u32(w.cell_hist, 65536, 0u, s); e != hipSuccess) return e;
    }
    return hipGetLastError();
}

template <int D>
hipError_t cells_centroids_t(const float* C, uint32_t N, uint32_t K, const Workspace& w, Radii radii, bool bounded, hipStream_t s)
{
    // buffers of the centroids' order by norm alone, which no E-step by cells asks for
    uint16_t* moves = cells_bounded(N, D, K) && bounded ? w.ckeys_tmp : nullptr;
    const uint32_t words = (N + 31) / 32, tiles = (K + 31) / 32, padded = w.packed_tiles * 32;
    hipLaunchKernelGGL(cell_keys_of_centroids_kernel<D>, dim3((std::max(K, words) + kThreads - 1) / kThreads), dim3(kThreads), 0, s, C, K,
                       words, int(radii), w.ckeys, w.cell_hist, w.cell_heads, w.changed, w.far_bits, w.hdr, w.csorted, w.cinv, moves);
    if (hipError_t e = launch_key_starts(w.cell_hist, w.key_starts, w.cell_cursor, K, s); e != hipSuccess) return e;
    hipLaunchKernelGGL(cell_place_kernel<D>, dim3((padded + kThreads - 1) / kThreads), dim3(kThreads), 0, s, C, K, padded, w.ckeys,
                       w.cell_cursor, w.cperm, w.cinv, w.csorted, reinterpret_cast<char*>(w.packed), w.cell_operands, D == 8 ? w.cell_flat : nullptr, w.hdr);
    hipLaunchKernelGGL((cell_lists_kernel<D, D == 4>), dim3(tiles), dim3(64 * kListWaves<D>), 0, s, w.csorted, w.cperm, K, w.cell_operands, list_tiles(D, K),
                       w.key_starts, w.cell_heads, N, w.hdr, w.cell_lists, w.cell_hist, w.cell_cursor);
    if (moves != nullptr) {
        const uint32_t lds = (K + 7) / 8 * 16;
        if (hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&cell_moved_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 65536 * 2);
            e != hipSuccess) return e;
        hipLaunchKernelGGL(cell_moved_kernel, dim3(std::min((K + 15) / 16, 256u)), dim3(kMovedThreads), lds, s, moves, K, w.cell_heads, w.cell_lists,
                           w.cperm_tmp, w.hdr);
    }
    return hipGetLastError();
}

NearArgs near_args(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, bool track, bool bounded)
{
    return NearArgs{w.xsorted, C, w.csorted, w.cperm, w.cell_flat, K, w.cell_heads, cell_items(w), N / item_of(d) + K,
                    w.cell_lists, w.cell_rank, w.far_bits, w.cell_position, far_view(w, N, d).pos,
                    w.cell_cursor, w.cperm_tmp, cells_bounded(N, d, K) ? reinterpret_cast<uint16_t*>(w.cell_order) /* idle between groupings */ : nullptr,
                    cells_bounded(N, d, K) && bounded, w.idx_sorted, track ? nullptr : w.dmin /* track: an iteration's */,
                    track ? w.idx_prev : nullptr, track ? w.changed : nullptr, w.hdr};
}

template <int D>
void cells_near_t(const float* C, uint32_t N, uint32_t K, const Workspace& w, bool track, bool bounded, hipStream_t s)
{
    const NearArgs a = near_args(C, N, D, K, w, track, bounded);
    const dim3 grid(a.slots), wave(64);
    if constexpr (D == 4) {
        hipLaunchKernelGGL(near_direct_kernel, grid, wave, 0, s, a);
    } else {
        if (cells_bounded(N, D, K)) {
            hipLaunchKernelGGL(near_sort_out_kernel, dim3((a.slots + kWaves - 1) / kWaves), dim3(kThreads), 0, s, a);
            hipLaunchKernelGGL(near_mfma_kernel<kQueued>, grid, wave, 0, s, a);
        } else {
            hipLaunchKernelGGL(near_mfma_kernel<kNear>, grid, wave, 0, s, a);
        }
        hipLaunchKernelGGL(near_mfma_kernel<kMid>, grid, wave, 0, s, a);
    }
}

template <int D>
void cells_compact_t(const float* C, uint32_t N, uint32_t K, const Workspace& w, hipStream_t s)
{
    const uint32_t words = (N + 31) / 32;
    const FarView f = far_view(w, N, D);
    const uint32_t blocks = (words + kThreads - 1) / kThreads;
    uint32_t *runs = w.sort_hist, *before = runs + blocks;   // no sort runs during an E-step
    hipLaunchKernelGGL(far_count_kernel, dim3(blocks), dim3(kThreads), 0, s, w.far_bits, words, runs, before);
    hipLaunchKernelGGL(far_compact_kernel<D>, dim3(blocks * kFarPieces), dim3(kThreads), 0, s, w.far_bits, words, runs, before, w.cell_position,
                       w.xsorted, w.idx_sorted, w.hdr, f.pos, f.x, f.idx);
    hipLaunchKernelGGL(far_window_kernel<D>, dim3(1024), dim3(kThreads), 0, s, f.x, f.idx, C, N, K, w.key_starts, w.hdr, far_windows(w));
}

template <int D>
void cells_far_t(uint32_t N, uint32_t K, const Workspace& w, hipStream_t s)
{
    const FarView f = far_view(w, N, D);
    const uint32_t sets = (N + 31) / 32;
    hipLaunchKernelGGL(far_kernel<D>, dim3(std::min(sets, 4096u)), dim3(64 * FarShape<D>::kWaves), 0, s, f.x, w.csorted, w.cperm, N, K,
                       reinterpret_cast<const char*>(w.packed), far_windows(w), f.pos, w.idx_sorted, w.dmin, w.hdr, f.refine);
}

}  // namespace

hipError_t launch_cells_order(const float* X, const float* C, uint32_t N, uint32_t d, uint32_t d_caller, uint32_t K, Workspace& w,
                              bool first, bool last, hipStream_t s)
{
    // first radius over mean t: n(R) grows like R^d from about 10 (d = 4) or 150 (d = 8) centroids at the mean
    const float factor = d_caller <= 4 ? 1.45f : (d_caller <= 6 ? 1.25f : 1.13f);
    switch (d) {
        case 4: return cells_order_t<4>(X, C, N, K, w, first, last, factor, s);
        case 8: return cells_order_t<8>(X, C, N, K, w, first, last, factor, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_cells_centroids(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, Radii radii, bool bounded, hipStream_t s)
{
    switch (d) {
        case 4: return cells_centroids_t<4>(C, N, K, w, radii, bounded, s);
        case 8: return cells_centroids_t<8>(C, N, K, w, radii, bounded, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_cells_near(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, bool track, bool bounded, hipStream_t s)
{
    switch (d) {
        case 4: cells_near_t<4>(C, N, K, w, track, bounded, s); break;
        case 8: cells_near_t<8>(C, N, K, w, track, bounded, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_cells_hints(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s)
{
    if (d != 8) return hipErrorInvalidValue;
    const NearArgs a = near_args(C, N, d, K, w, false, false);
    hipLaunchKernelGGL(near_mfma_kernel<kHint>, dim3(a.slots), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_cells_compact(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: cells_compact_t<4>(C, N, K, w, s); break;
        case 8: cells_compact_t<8>(C, N, K, w, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_cells_far(uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s)
{
    switch (d) {
        case 4: cells_far_t<4>(N, K, w, s); break;
        case 8: cells_far_t<8>(N, K, w, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cc
