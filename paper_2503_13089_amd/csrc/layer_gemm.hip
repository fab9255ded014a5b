// Forward pass of the compressed linear layer at prefill-sized batches (the paper's layer listing: rebuild the
// weight from (codebook, codes), then y = x . W + bias), as two hand-written kernels:
//
//   1. layer_weight_frag_columns_kernel (small matrices: layer_weight_frag_kernel): the listing's gather, written straight into
//      the register layout of the matrix cores' B operand. One fragment = 32 output columns x 16 in-features = 64 lanes
//      x 8 consecutive k = 1 KB; fragments of one column block are contiguous along k. Padding in-features past the
//      end of the last fragment are zeros; columns past out_features are anything, nothing is stored of their sums.
//   2. gemm_frag_kernel: y[M][N] = x[M][K] . W on v_mfma_f32_32x32x16_{bf16,f16}. A workgroup of 8 waves owns a
//      256 x 256 tile of y, each wave 128 x 64 of it (4 x 2 accumulator tiles of 32 x 32, in registers for the whole
//      contraction), and steps through K in slices of 32. Only x goes through LDS (double-buffered, rows padded to 40
//      halves so that the 16-byte fragment reads of 16 lanes fall on 16 different bank quads). The fragments of W
//      come from memory as they are: one fully coalesced 1 KB load per fragment, requested two slices ahead. Every
//      memory instruction of the loop sits between two matrix instructions.
//      Products of two 16-bit values are exact in fp32; the sum is fp32 in a fixed order; bias (and, for the
//      quantised codebook, the scale) are applied to the finished sum and y is rounded once.
//      Workgroups are numbered so that one XCD (they are dealt to the 8 XCDs in turn) works on neighbouring column
//      panels with all row panels of x: its L2 then holds the fragments it is using, and x comes once per XCD.
//      Tiles that do not fill a round of the chip's workgroup slots are cut along the contraction: fp32 partial
//      tiles go to the workspace and a second kernel adds them in a fixed order - the result never depends on
//      scheduling.
//
// Bound: the bf16 / fp16 matrix cores (2 M N K flop against 2.5 PFLOP/s). Measured at M = 2048, 4096 x 11008: the
// product takes 169 us = 1.09 PFLOP/s in the first calls of a run, 177 to 219 in later ones by the card's clock, 194 on the mean of 20
// (0.95). The loop that it grew from took 189 us, and with every memory instruction taken out (matrix instructions
// only) 130: under sustained matrix work the chip clocks near 1.7 GHz instead of 2.4, and the 344 tiles take
// 1.5 rounds on 256 compute units where 1.34 would do - that, not 2.5 PFLOP/s, is the ceiling of this tile schedule.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "half_types.h"

namespace cc {

namespace {

constexpr int kThreads = 256;               // rebuild and finishing kernels
constexpr int WN = 4;                       // waves along the columns of a tile (2 along its rows)
constexpr int kGemmThreads = 128 * WN;
constexpr int BM = 256, BN = 64 * WN, BK = 32;
constexpr int LDT = BK + 8;                 // halves per LDS row (20 words: the 16-byte reads of 16 lanes hit 16 bank quads)
constexpr int kStageHalves = BM * LDT;
constexpr int kOutPitch = 64 + 4;             // floats per LDS row of the epilogue: 32 rows of a wave's 64 columns
constexpr uint32_t kGemmLdsBytes = 2 * WN * 32 * kOutPitch * 4;   // 69,632 bytes; the slices of x take 40,960
static_assert(kGemmLdsBytes >= 2 * kStageHalves * 2, "room for two slices");
constexpr int kFragHalves = 512;            // one B operand: 32 columns x 16 in-features

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c)
{
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The columns of a block of 32 lie in the order of n % g first, then the even ones and the odd ones of those: what a column of
// the codebook fills is together, and so is what one store of the rebuild by columns writes (two code columns a lane; a cache
// line at g = 4, its two halves of 8 in-features side by side). place and column are each other's inverse.
__device__ __forceinline__ uint32_t block_place(uint32_t column, uint32_t g)
{
    const uint32_t i = column * (1024 / g + 1) >> 10, r = column - i * g;   // column / g, column % g: column < 32, g <= 16
    const uint32_t count = 32 / g + (r < 32 % g ? 1 : 0);                   // columns with this remainder
    return r * (32 / g) + min(r, 32 % g) + i / 2 + (i % 2) * ((count + 1) / 2);
}
__device__ __forceinline__ uint32_t block_column(uint32_t place, uint32_t g)
{
    const uint32_t per = 32 / g, more = 32 % g * (per + 1);   // the first 32 % g remainders have per + 1 columns
    const uint32_t r = place < more ? place / (per + 1) : (place - more) / per + 32 % g;
    const uint32_t i = place - r * per - min(r, 32 % g), even = (per + (r < 32 % g ? 2 : 1)) / 2;
    return r + (i < even ? 2 * i : 2 * (i - even) + 1) * g;
}
// 16-byte piece of a fragment with in-features 8 h .. + 7 of the column at a place
__device__ __forceinline__ uint32_t frag_piece(uint32_t place, uint32_t h) { return place / 4 * 8 + 4 * h + place % 4; }

// ---- 1. rebuild into B-operand fragments: column block nb = n / 32, in-feature block kb = k / 16, fragment
// (nb * KB + kb) with KB = ceil(in_features / 16) blocks per column block, 16-byte piece frag_piece(block_place(n % 32), (k % 16) / 8)
// Three steps per 64 x 64 tile: the tile's codes (64 rows of W, the code columns that touch the tile) go to LDS with
// reads along the rows of the code matrix; then a wave takes one code column and its 64 lanes the 64 rows, so that
// the elements they write into the transposed tile are neighbours in LDS (lanes along n would hit the same banks);
// then the tile leaves as 2 x 4 fragments, 64 lanes x 16 bytes each.
constexpr int kWtTile = 64;
constexpr int kWtMaxCols = kWtTile + 2;  // code columns touching a tile: at most 64 / g + 2 <= 66 for g >= 1
__global__ __launch_bounds__(kThreads) void layer_weight_frag_kernel(const uint16_t* __restrict__ codebook, uint32_t K, uint32_t g,
                                                                     const uint16_t* __restrict__ codes, uint32_t per_row,
                                                                     uint32_t in_features, uint32_t out_features,
                                                                     uint32_t NB, uint32_t KB, uint16_t* __restrict__ wf)
{
    constexpr int T = kWtTile, LT = T + 8;
    __shared__ __attribute__((aligned(16))) uint16_t tile[T * LT];  // [n][k]
    __shared__ uint16_t ctile[T * kWtMaxCols];                      // [k][code column]
    const uint32_t n_lo = blockIdx.x * T, k0 = blockIdx.y * T;
    const uint32_t cn_lo = n_lo / g;
    const uint32_t cn_hi = min((n_lo + T - 1) / g, per_row - 1);
    const uint32_t cpr = cn_hi - cn_lo + 1;  // code columns that touch this tile
    const uint32_t items = T * cpr;
    const bool edge = n_lo + T > out_features || k0 + T > in_features;
    if (edge)  // padding is stored too, as zeros
        for (uint32_t e = threadIdx.x; e < T * LT / 2; e += kThreads) reinterpret_cast<uint32_t*>(tile)[e] = 0u;
    for (uint32_t it = threadIdx.x; it < items; it += kThreads) {
        const uint32_t kr = it / cpr, c = it % cpr;
        const uint32_t k = min(k0 + kr, in_features - 1);
        ctile[kr * cpr + c] = codes[size_t(k) * per_row + cn_lo + c];
    }
    __syncthreads();
    const int n_end = int(min(uint32_t(T), out_features - n_lo));
    for (uint32_t it = threadIdx.x; it < items; it += kThreads) {
        const uint32_t c = it / T, kr = it % T;
        if (k0 + kr >= in_features) continue;
        const uint32_t code = min(uint32_t(ctile[kr * cpr + c]), K - 1);
        const uint16_t* row = codebook + size_t(code) * g;
        const int nbase = int((cn_lo + c) * g) - int(n_lo);
        if (g == 4) {
            const uint2 r = *reinterpret_cast<const uint2*>(row);
            const uint16_t e[4] = {uint16_t(r.x), uint16_t(r.x >> 16), uint16_t(r.y), uint16_t(r.y >> 16)};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = nbase + j;
                if (n >= 0 && n < n_end) tile[n * LT + kr] = e[j];
            }
        } else if (g == 8) {
            const uint4 r = *reinterpret_cast<const uint4*>(row);
            const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int n = nbase + j;
                if (n >= 0 && n < n_end) tile[n * LT + kr] = uint16_t(w[j >> 1] >> (16 * (j & 1)));
            }
        } else {
            for (uint32_t j = 0; j < g; ++j) {
                const int n = nbase + int(j);
                if (n >= 0 && n < n_end) tile[n * LT + kr] = row[j];
            }
        }
    }
    __syncthreads();
    // fragment q = 4 (column block within the tile) + (in-feature block within the tile): a wave writes one, 1 KB
    const uint32_t lane = threadIdx.x & 63, half = lane / 4 % 2, column = block_column(lane / 8 * 4 + lane % 4, g);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const uint32_t q = pass * 4 + threadIdx.x / 64;
        const uint32_t nb = n_lo / 32 + q / 4, kb = k0 / 16 + q % 4;
        if (nb < NB && kb < KB)
            *reinterpret_cast<uint4*>(wf + (size_t(nb) * KB + kb) * kFragHalves + lane * 8) =
                *reinterpret_cast<const uint4*>(&tile[((q / 4) * 32 + column) * LT + (q % 4) * 16 + 8 * half]);
    }
}

// The same by columns of the codebook. Row by row, every code is a codebook row from L2, one line each, 0.3 to 0.4 a clock and compute
// unit; here a workgroup (one per compute unit, 16 waves) keeps J columns of all rows in LDS, an entry of 2 J bytes per row, and writes
// the elements of the matrix that come from them. What a lane looks up - 8 codes below one another, 2 side by side - are pieces of 16
// bytes of the fragments, so nothing is transposed. g / J workgroups read the same codes, side by side on one XCD.
// Measured for 4096 x 11008 (45 M weights; a fill of the 90 MB takes 15 us), us, row by row and now: K = 65536, g = 4 65 / 33,
// g = 6 192 / 39, g = 8 46 / 36; 8192 x 28672, g = 4 361 / 176. Without the stores 24 us at g = 4, without the
// lookups 41, without the codes 27, without the columns 33: codes and stores share the way to L2.
// Tried and no faster: 3, 4 or 6 items' codes ahead; codes 16 columns apart (whole 128-byte stores at g = 8, twice the loads);
// items along the rows; stores past L2 (20 us slower at g = 6 and 8).
constexpr int kColumnThreads = 1024;
constexpr uint32_t kBand = 2;               // code column groups of 32: 128 bytes of a row of codes
constexpr uint32_t kColumnLds = 160 * 1024;
constexpr uint32_t kUnits = 256;            // compute units
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32_2 __attribute__((aligned(2)));

template <int J>
__global__ __launch_bounds__(kColumnThreads, 4) void layer_weight_frag_columns_kernel(
    const uint16_t* __restrict__ codebook, const uint8_t* __restrict__ laid, uint32_t stride, uint32_t K, uint32_t g, const uint16_t* __restrict__ codes, uint32_t per_row,
    uint32_t in_features, uint32_t out_features, uint32_t NB, uint32_t KB, uint16_t* __restrict__ wf, uint32_t sets, uint32_t jobs, uint32_t k_steps,
    uint32_t items, uint32_t per_job)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    constexpr uint32_t E = 2 * J, NC = 2, kWaves = kColumnThreads / 64;
    const uint32_t lane = threadIdx.x & 63, n16 = lane & 15, kg = lane >> 4;
    const uint32_t wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    const uint32_t job = blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8;   // the sets of the same codes on one XCD
    if (job >= jobs) return;
    const uint32_t set = job % sets, begin = job / sets * per_job, end = min(begin + per_job, items);
    // A job's items, 16 NC code columns by 32 in-features: kBand side by side, then down the matrix, then the next kBand. Every 16th
    // is this wave's.
    uint32_t code[2][8];
    struct Item {
        uint32_t k0, group;
    };
    auto item = [&](uint32_t t) {
        const uint32_t band = t / kBand / k_steps;
        return Item{(t / kBand - band * k_steps) * 32, band * kBand + t % kBand};
    };
    auto next = [&](Item i) {
        i.k0 += kWaves / kBand * 32;
        while (i.k0 >= 32 * k_steps) {
            i.k0 -= 32 * k_steps;
            i.group += kBand;
        }
        return i;
    };
    const uint32_t lane_row = 8 * kg * per_row, last_k0 = (k_steps - 1) * 32;
    const uint32_t lane_row_last = (min(last_k0 + 8 * kg, in_features - 8) - last_k0) * per_row;   // rows past the end: the last 8 again
    auto column = [&](const Item& i) { return min(i.group * (16 * NC) + n16 * NC, per_row - NC); };
    auto request = [&](const Item& i, uint32_t (&c)[8]) {
        const char* from = reinterpret_cast<const char*>(codes + size_t(i.k0) * per_row);
        const uint32_t at = 2 * ((i.k0 == last_k0 ? lane_row_last : lane_row) + column(i));
#pragma unroll
        for (uint32_t r = 0; r < 8; ++r) {
            const char* q = from + size_t(2 * r) * per_row + at;
            c[r] = *reinterpret_cast<const u32_2*>(q);
        }
    };
    const uint32_t first = begin + wave, steps = first < end ? (end - first + kWaves - 1) / kWaves : 0u;
    Item now = item(first), ahead = now;
    uint32_t asked = 0;
    auto request_next = [&](uint32_t (&c)[8]) {   // of the wave's last item again where there is none left
        if (asked > 0 && asked < steps) ahead = next(ahead);
        ++asked;
        request(ahead, c);
    };
    if (steps > 0) {
        request_next(code[0]);
        request_next(code[1]);
    }
    // ---- the columns into LDS, each workgroup from another place on
    if (laid != nullptr) {
        constexpr int U = 8;
        const uint8_t* src = laid + size_t(set) * stride;
        const uint32_t pieces = stride / 16, turn = (blockIdx.x / 8 * 331u + blockIdx.x) % pieces;
        for (uint32_t i0 = threadIdx.x; i0 < pieces; i0 += U * kColumnThreads) {
            u32x4 e[U];
            uint32_t at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                at[u] = min(i0 + u * kColumnThreads, pieces - 1) + turn;
                at[u] = at[u] >= pieces ? at[u] - pieces : at[u];
                e[u] = *reinterpret_cast<const u32x4*>(src + 16 * size_t(at[u]));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) *reinterpret_cast<u32x4*>(smem + 16 * at[u]) = e[u];
        }
    } else {
        constexpr int U = 8;
        const uint32_t turn = (blockIdx.x / 8 * 331u + blockIdx.x) * 64u % K;
        for (uint32_t i0 = threadIdx.x; i0 < K; i0 += U * kColumnThreads) {
            uint16_t e[U][J];
            uint32_t at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                at[u] = min(i0 + u * kColumnThreads, K - 1) + turn;
                at[u] = at[u] >= K ? at[u] - K : at[u];
#pragma unroll
                for (uint32_t j = 0; j < J; ++j) e[u][j] = codebook[size_t(at[u]) * g + min(set * J + j, g - 1)];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (uint32_t j = 0; j < J; ++j) reinterpret_cast<uint16_t*>(smem)[at[u] * J + j] = e[u][j];
        }
    }
    __syncthreads();
    const u16x2 last = {uint16_t(K - 1), uint16_t(K - 1)};
    auto step = [&](uint32_t (&c)[8], auto more) {
        const uint32_t k = now.k0 + 8 * kg, col = column(now);
        uint32_t w[NC][4 * J];
#pragma unroll
        for (uint32_t v = 0; v < NC; ++v)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const u16x2 both = __builtin_elementwise_min(__builtin_bit_cast(u16x2, c[r]), last);   // never outside the codebook
                const uint32_t from = uint32_t(both[v]) * E;
                if constexpr (J == 1) {
                    u16x2 pair = __builtin_bit_cast(u16x2, w[v][r / 2]);
                    pair[r % 2] = *reinterpret_cast<const uint16_t*>(smem + from);
                    w[v][r / 2] = __builtin_bit_cast(uint32_t, pair);
                } else if constexpr (J == 2) {
                    w[v][r] = *reinterpret_cast<const uint32_t*>(smem + from);
                } else {
                    const uint2 x = *reinterpret_cast<const uint2*>(smem + from);
                    w[v][2 * r] = x.x; w[v][2 * r + 1] = x.y;
                }
            }
        if constexpr (more) {
            request_next(c);
            __builtin_amdgcn_sched_barrier(0);   // not behind the stores
        }
        // stores without a branch, so that the wait for the next codes does not become one for everything: what is not part of
        // the matrix goes to an offset past the end, which the store leaves out
        const uint32_t nb = min(now.group * (16 * NC), per_row - NC) * g / 32;
        const size_t left = (size_t(NB) - nb) * KB * (kFragHalves * 2);
        const auto block = __builtin_amdgcn_make_buffer_rsrc(wf + size_t(nb) * KB * kFragHalves, 0, int(min(left, size_t(0x7fffffff))), 0x00020000);
#pragma unroll
        for (uint32_t v = 0; v < NC; ++v)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint32_t e = set * J + j, n = (col + v) * g + e;
                const bool part = (J == 1 || e < g) && n < out_features && k / 16 < KB;
                u32x4 b;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (J == 1) b[i] = w[v][i];
                    else b[i] = __builtin_amdgcn_perm(w[v][(2 * i + 1) * (J / 2) + j / 2], w[v][2 * i * (J / 2) + j / 2], j % 2 ? 0x07060302u : 0x05040100u);
                    b[i] = k < in_features ? b[i] : 0u;
                }
                const uint32_t at = (__umul24(n / 32 - nb, KB) + k / 16) * (kFragHalves * 2) + frag_piece(block_place(n % 32, g), kg & 1) * 16;
                __builtin_amdgcn_raw_buffer_store_b128(b, block, part ? at : 0x80000000u, 0, 0);
            }
        now = next(now);
    };
    if (steps == 0) return;
    uint32_t i = 0;
    for (; i + 2 < steps; i += 2) {
        step(code[0], std::true_type{});
        step(code[1], std::true_type{});
    }
    step(code[0], std::false_type{});
    if (i + 1 < steps) step(code[1], std::false_type{});
}

// The codebook as 16-bit numbers by sets of J columns, `stride` of them a set (J = g: as it was). Integers of a quantised codebook
// (8 bits: signed bytes; 4 bits: two's-complement nibbles, element e in byte e / 2, low nibble first) are exact in both formats: the
// rebuilt matrix and the product hold the integers themselves.
template <int DT>
__global__ __launch_bounds__(kThreads) void codebook_columns_kernel(const uint8_t* __restrict__ book, int bits, uint32_t n, uint32_t g, uint32_t J,
                                                                    uint32_t stride, uint16_t* __restrict__ out)
{
    const uint32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e >= n) return;
    uint16_t v;
    if (bits == 16) v = reinterpret_cast<const uint16_t*>(book)[e];
    else if (bits == 8) v = from_f32<DT>(float(int(static_cast<int8_t>(book[e]))));
    else v = from_f32<DT>(float(int(((uint32_t(book[e >> 1]) >> (4 * (e & 1))) & 0xFu) ^ 8u) - 8));
    const uint32_t k = e / g, j = e % g;
    out[size_t(j / J) * stride + k * J + j % J] = v;
}

// 8 neighbouring numbers
__device__ __forceinline__ void load_8(const float* from, float (&v)[8])
{
    const float4 lo = reinterpret_cast<const float4*>(from)[0], hi = reinterpret_cast<const float4*>(from)[1];
    v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
    v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
}
// and as columns n .. n + 7 of a row of y, which ends at column N and may begin at any
template <int DT>
__device__ __forceinline__ void store_8(uint16_t* row, uint32_t n, uint32_t N, const float (&v)[8])
{
    typedef u32x4 u32x4_2 __attribute__((aligned(2)));
    u32x4 piece;
#pragma unroll
    for (int e = 0; e < 4; ++e) piece[e] = uint32_t(from_f32<DT>(v[2 * e])) | uint32_t(from_f32<DT>(v[2 * e + 1])) << 16;
    if (n + 8 <= N) {
        *reinterpret_cast<u32x4_2*>(row + n) = piece;
    } else {
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (n + e < N) row[n + e] = uint16_t(piece[e / 2] >> (16 * (e % 2)));
    }
}

// ---- 2. the product
// Jobs: the tiles of y in whole rounds of the chip's workgroup slots take the full contraction and write y themselves
// (`whole` of them); the tiles of the last, partial round are each cut into f in-feature slices, so that the round
// is short and full instead of long and half empty, and leave fp32 partial tiles for gemm_finish_kernel. The cut
// depends on the shape alone.
template <int DT>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_frag_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ wf, uint32_t M, uint32_t N, uint32_t K, uint32_t NB, uint32_t KB,
    const float* __restrict__ scale, const uint16_t* __restrict__ bias, uint16_t* __restrict__ y, float* __restrict__ partial,
    uint32_t m_tiles, uint32_t whole, uint32_t f, uint32_t k_per_split, uint32_t jobs, uint32_t g)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, l32 = lane & 31;
    const int wm = wave & 1, wn = wave >> 1;

    // job of this workgroup: XCD q (= blockIdx % 8) takes the q-th contiguous share of the whole tiles and then the
    // q-th share of the slices of the cut tiles; within a share the row panels of x vary fastest, so neighbours
    // share a column panel of W
    const uint32_t xcd = blockIdx.x % 8, local = blockIdx.x / 8;
    const uint32_t whole_per = (whole + 7) / 8, cut_per = (jobs - whole + 7) / 8;
    uint32_t job;
    if (local < whole_per) {
        job = xcd * whole_per + local;
        if (job >= whole) return;
    } else {
        job = whole + xcd * cut_per + (local - whole_per);
        if (local - whole_per >= cut_per || job >= jobs) return;
    }
    const bool direct = job < whole;
    const uint32_t cut = direct ? 0u : (job - whole) / f;   // which tile of the partial round
    const uint32_t split = direct ? 0u : (job - whole) % f;
    const uint32_t tile = direct ? job : whole + cut;
    const uint32_t mt = tile % m_tiles, nt = tile / m_tiles;
    const uint32_t m0 = mt * BM, n0 = nt * BN;
    const uint32_t k_begin = uint32_t(__builtin_amdgcn_readfirstlane(int(direct ? 0u : split * k_per_split)));
    const uint32_t k_end = uint32_t(__builtin_amdgcn_readfirstlane(int(direct ? K : min(k_begin + k_per_split, K))));

    // x: global -> registers -> LDS in 16-byte pieces, BK / 8 per row and slice; thread t takes piece t % PR of rows
    // t / PR + RP i. Rows past the edge are clamped (their results are never stored); a piece past k_end goes to LDS as
    // zeros (K and k_per_split are multiples of 8).
    // W: this wave's two column blocks, fragments straight from memory; a block past the last one is clamped (its
    // columns are never stored), a fragment past the end of the contraction reads the last one (and is never used).
    //
    // The global loads of the main loop are written as instructions, with the waits on them placed by hand: the
    // compiler otherwise moves each request down to the slice that uses it, where its whole latency is exposed. The
    // memory counter retires loads in order, so a wait names how many younger requests may still be in flight. Every
    // slice issues the same six requests, past the end of the contraction too (clamped offsets, results unused),
    // which keeps those numbers the same for every slice.
    constexpr int PR = BK / 8, RP = kGemmThreads / PR, NA = BM / RP;
    static_assert(NA == 2, "the wait counts below assume two pieces of x per thread and slice");
    const uint32_t prow = threadIdx.x / PR, pk = (threadIdx.x % PR) * 8;
    // Where a request goes is a buffer (the tile's rows of x, its column blocks of W), an offset of the lane's that does not change and one of the
    // contraction's that is a scalar, clamped to the last piece: with addresses made per request the loop had 30 vector instructions beside its 16 matrix
    // instructions, which share the issue with them (2048 x 4096 x 11008, bf16, a call 233 / 226 us; 4096^3 155 / 148). What lies past a buffer's end (the pieces
    // beside the last one, in the last row) reads as zero. A buffer has at most 512 K bytes, 2^31 - 2^15 at the most in-features that the rebuild takes.
    const uint32_t rows = min(uint32_t(BM), M - m0), block0 = n0 / 32, blocks = min(uint32_t(BN / 32), NB - block0);
    auto buffer = [](const uint16_t* from, size_t bytes) {
        const uint64_t at = reinterpret_cast<uint64_t>(from);
        return u32x4{uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(at)))), uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(at >> 32) & 0xffffu))),
                     uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(min(bytes, size_t(0x7fffffff)))))), 0x00020000u};
    };
    const u32x4 a_buffer = buffer(x + size_t(m0) * K, size_t(rows) * K * 2), b_buffer = buffer(wf + size_t(block0) * KB * kFragHalves, size_t(blocks) * KB * kFragHalves * 2);
    uint32_t a_off[NA], b_off[2];   // bytes
#pragma unroll
    for (int i = 0; i < NA; ++i) a_off[i] = (min(prow + RP * i, rows - 1) * K + pk) * 2;
#pragma unroll
    for (int j = 0; j < 2; ++j) b_off[j] = (min(uint32_t(wn * 2 + j), blocks - 1) * KB * kFragHalves + frag_piece(l32, h) * 8) * 2;
    auto request = [](u32x4& r, uint32_t off, const u32x4& from, uint32_t at) {
        asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen" : "=v"(r) : "v"(off), "s"(from), "s"(at));
    };
    auto request_a = [&](u32x4& r, int i, uint32_t k0) { request(r, a_off[i], a_buffer, min(k0, K - 8) * 2); };
    auto request_b = [&](u32x4& r, int j, uint32_t k) { request(r, b_off[j], b_buffer, min(k / 16, KB - 1) * (kFragHalves * 2)); };
#define CC_GEMM_ARRIVED(younger, r) asm volatile("s_waitcnt vmcnt(" #younger ")" : "+v"((r)[0]), "+v"((r)[1]))
    auto stash = [&](u32x4 (&a)[NA], int buf, uint32_t k0) {
        uint16_t* As = lds + buf * kStageHalves;
        if (k0 < k_end && k0 + BK > k_end) {   // a last slice that the contraction does not fill: zeros (past the end nobody reads)
            const uint32_t keep = k0 + pk < k_end ? 0xffffffffu : 0u;
#pragma unroll
            for (int i = 0; i < NA; ++i) a[i] &= keep;
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4*>(&As[(prow + RP * i) * LDT + pk]) = a[i];
    };
    const uint16_t* a_lds = lds + (wm * 128 + l32) * LDT + 8 * h;
    auto read_frag = [&](u32x4& a, int i, int buf, int kk) {
        a = *reinterpret_cast<const u32x4*>(a_lds + buf * kStageHalves + 32 * i * LDT + 16 * kk);
    };

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // One slice of 32 in-features = two batches of 8 matrix instructions (16 in-features each) with the barrier
    // between them. Every memory instruction of the loop is issued between two matrix instructions, one at a time: a
    // wave that issues its requests in a burst waits at them until the memory pipeline has taken those of all eight
    // waves, and issues no matrix instruction meanwhile (measured: loop without matrix instructions 111 us, matrix
    // instructions alone 85 us, both with the requests in bursts 209 us - the sum). The x fragments of the second
    // batch are read from LDS during the first four instructions of the first batch, those of the next slice's first
    // batch during the first four of the second batch, after the barrier. Batch t takes its fragments of W from ring
    // slot t % 4. Slices come in pairs so that every slot and buffer index is a constant. Requests of slice s, in
    // order: during the second half of its first batch x of slice s + 2 (2), then W of the second batch of slice s + 1
    // (2); during the second half of its second batch W of the first batch of slice s + 2 (2). What it needs, and how
    // many younger requests are out by then: W of its first batch (asked for in slice s - 2: 6), x of slice s + 1 for
    // LDS (slice s - 1: 8, this slice's four included), W of its second batch (slice s - 1, after x: 6).
    // (The hand-over to LDS also runs after the last slice, where it moves zeros.)
    u32x4 a0[4], a1[4], bq[4][2], ar[2][NA];
#define CC_GEMM_STEP(stmt)                     \
    stmt;                                      \
    __builtin_amdgcn_sched_barrier(0)
#define CC_GEMM_SLICE(P, k0)                                                                   \
    do {                                                                                       \
        CC_GEMM_ARRIVED(6, bq[2 * (P)]);                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        CC_GEMM_STEP(acc[0][0] = mma<DT>(a0[0], bq[2 * (P)][0], acc[0][0]));                   \
        CC_GEMM_STEP(read_frag(a1[0], 0, P, 1));                                               \
        CC_GEMM_STEP(acc[0][1] = mma<DT>(a0[0], bq[2 * (P)][1], acc[0][1]));                   \
        CC_GEMM_STEP(read_frag(a1[1], 1, P, 1));                                               \
        CC_GEMM_STEP(acc[1][0] = mma<DT>(a0[1], bq[2 * (P)][0], acc[1][0]));                   \
        CC_GEMM_STEP(read_frag(a1[2], 2, P, 1));                                               \
        CC_GEMM_STEP(acc[1][1] = mma<DT>(a0[1], bq[2 * (P)][1], acc[1][1]));                   \
        CC_GEMM_STEP(read_frag(a1[3], 3, P, 1));                                               \
        CC_GEMM_STEP(acc[2][0] = mma<DT>(a0[2], bq[2 * (P)][0], acc[2][0]));                   \
        CC_GEMM_STEP(request_a(ar[P][0], 0, (k0) + 2 * BK));                             \
        CC_GEMM_STEP(acc[2][1] = mma<DT>(a0[2], bq[2 * (P)][1], acc[2][1]));                   \
        CC_GEMM_STEP(request_a(ar[P][1], 1, (k0) + 2 * BK));                             \
        CC_GEMM_STEP(acc[3][0] = mma<DT>(a0[3], bq[2 * (P)][0], acc[3][0]));                   \
        CC_GEMM_STEP(request_b(bq[(2 * (P) + 3) % 4][0], 0, (k0) + BK + 16));            \
        CC_GEMM_STEP(acc[3][1] = mma<DT>(a0[3], bq[2 * (P)][1], acc[3][1]));                   \
        CC_GEMM_STEP(request_b(bq[(2 * (P) + 3) % 4][1], 1, (k0) + BK + 16));            \
        CC_GEMM_ARRIVED(8, ar[1 - (P)]);                                                       \
        stash(ar[1 - (P)], 1 - (P), (k0) + BK);                                                \
        __syncthreads();                                                                       \
        CC_GEMM_ARRIVED(6, bq[2 * (P) + 1]);                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        CC_GEMM_STEP(acc[0][0] = mma<DT>(a1[0], bq[2 * (P) + 1][0], acc[0][0]));               \
        CC_GEMM_STEP(read_frag(a0[0], 0, 1 - (P), 0));                                         \
        CC_GEMM_STEP(acc[0][1] = mma<DT>(a1[0], bq[2 * (P) + 1][1], acc[0][1]));               \
        CC_GEMM_STEP(read_frag(a0[1], 1, 1 - (P), 0));                                         \
        CC_GEMM_STEP(acc[1][0] = mma<DT>(a1[1], bq[2 * (P) + 1][0], acc[1][0]));               \
        CC_GEMM_STEP(read_frag(a0[2], 2, 1 - (P), 0));                                         \
        CC_GEMM_STEP(acc[1][1] = mma<DT>(a1[1], bq[2 * (P) + 1][1], acc[1][1]));               \
        CC_GEMM_STEP(read_frag(a0[3], 3, 1 - (P), 0));                                         \
        CC_GEMM_STEP(acc[2][0] = mma<DT>(a1[2], bq[2 * (P) + 1][0], acc[2][0]));               \
        CC_GEMM_STEP(acc[2][1] = mma<DT>(a1[2], bq[2 * (P) + 1][1], acc[2][1]));               \
        CC_GEMM_STEP(acc[3][0] = mma<DT>(a1[3], bq[2 * (P) + 1][0], acc[3][0]));               \
        CC_GEMM_STEP(request_b(bq[2 * (P)][0], 0, (k0) + 2 * BK));                       \
        CC_GEMM_STEP(acc[3][1] = mma<DT>(a1[3], bq[2 * (P) + 1][1], acc[3][1]));               \
        CC_GEMM_STEP(request_b(bq[2 * (P)][1], 1, (k0) + 2 * BK));                       \
    } while (0)

    // before the first slice: the same requests in the same order, as far as they exist
    request_a(ar[0][0], 0, k_begin);
    request_a(ar[0][1], 1, k_begin);
    request_b(bq[0][0], 0, k_begin);
    request_b(bq[0][1], 1, k_begin);
    request_a(ar[1][0], 0, k_begin + BK);
    request_a(ar[1][1], 1, k_begin + BK);
    request_b(bq[1][0], 0, k_begin + 16);
    request_b(bq[1][1], 1, k_begin + 16);
    request_b(bq[2][0], 0, k_begin + BK);
    request_b(bq[2][1], 1, k_begin + BK);
    CC_GEMM_ARRIVED(8, ar[0]);
    stash(ar[0], 0, k_begin);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) read_frag(a0[i], i, 0, 0);
    for (uint32_t k0 = k_begin;;) {
        CC_GEMM_SLICE(0, k0);
        if ((k0 += BK) >= k_end) break;
        CC_GEMM_SLICE(1, k0);
        if ((k0 += BK) >= k_end) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // requests past the end still write registers: let them land
#undef CC_GEMM_SLICE
#undef CC_GEMM_STEP
#undef CC_GEMM_ARRIVED

    // ---- epilogue: accumulator register r of lane (l32, h) is row r % 4 + 8 (r / 4) + 4 h, column l32 of its tile. 32 rows of the wave at a time go through
    // LDS, and from there as 16-byte pieces: stored from the registers, 2 bytes a lane, the tile took 128 store instructions a wave where these are 16 (2048 x 4096 x 11008, a call 226 / 219 us; 4096^3 148 / 142).
    __syncthreads();   // the last slice has been read
    const float sc = (direct && scale != nullptr) ? *scale : 1.0f;
    float bv[8];   // of this lane's columns
    if (direct && bias != nullptr) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bv[e] = to_f32<DT>(bias[min(n0 + wn * 64 + 8 * (lane % 8) + e, N - 1)]);
    }
    const uint32_t l_column = block_column(l32, g);
    float* const out = reinterpret_cast<float*>(lds) + wave * (32 * kOutPitch);
    float* ptile = partial + (size_t(cut) * f + split) * (BM * BN);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the rows before have been read
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[((r & 3) + 8 * (r >> 2) + 4 * h) * kOutPitch + 32 * j + l_column] = acc[i][j][r];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // a wave's own: no barrier
        if (direct) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {   // 8 rows of 8 pieces of 8 columns
                const uint32_t row = 8 * t + lane / 8, nl = wn * 64 + 8 * (lane % 8), n = n0 + nl, m = m0 + wm * 128 + 32 * i + row;
                float v[8];
                load_8(out + row * kOutPitch + 8 * (lane % 8), v);
                if (m >= M || n >= N) continue;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (scale != nullptr) v[e] *= sc;
                    if (bias != nullptr) v[e] += bv[e];
                }
                store_8<DT>(y + size_t(m) * N, n, N, v);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) {   // 4 rows of 16 pieces of 4 columns; columns past the edge nobody reads
                const uint32_t row = 4 * t + lane / 16, ml = wm * 128 + 32 * i + row;
                if (m0 + ml < M) *reinterpret_cast<float4*>(ptile + ml * BN + wn * 64 + 4 * (lane % 16)) = *reinterpret_cast<const float4*>(out + row * kOutPitch + 4 * (lane % 16));
            }
        }
    }
}

// The tiles of the partial round: y = round(scale * (sum of the f slices, in order) + bias); scale may be NULL (= 1).
// Bound: memory. 8 elements a thread; with one it took 12.2 us for 88 tiles of 2 slices (46 MB), now 10.0 (a call 218.6 / 217.6).
template <int DT>
__global__ __launch_bounds__(kThreads) void gemm_finish_kernel(const float* __restrict__ partial, uint32_t M, uint32_t N,
                                                               uint32_t m_tiles, uint32_t whole, uint32_t f,
                                                               const float* __restrict__ scale,
                                                               const uint16_t* __restrict__ bias, uint16_t* __restrict__ y)
{
    const uint32_t cut = blockIdx.y, tile = whole + cut;
    const uint32_t m0 = (tile % m_tiles) * BM, n0 = (tile / m_tiles) * BN;
    const uint32_t e = (blockIdx.x * kThreads + threadIdx.x) * 8;  // 8 elements of a row of the tile
    const uint32_t m = m0 + e / BN, n = n0 + e % BN;
    if (m >= M || n >= N) return;
    const float* p = partial + size_t(cut) * f * (BM * BN) + e;
    float v[8];
    load_8(p, v);
    uint32_t s = 1;
    for (; s + 1 < f; s += 2) {   // two slices' loads under way
        float a[8], b[8];
        load_8(p + size_t(s) * (BM * BN), a);
        load_8(p + size_t(s + 1) * (BM * BN), b);
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = v[c] + a[c] + b[c];
    }
    if (s < f) {
        float a[8];
        load_8(p + size_t(s) * (BM * BN), a);
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] += a[c];
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (scale != nullptr) v[c] *= *scale;
        if (bias != nullptr) v[c] += to_f32<DT>(bias[min(n + c, N - 1)]);
    }
    store_8<DT>(y + size_t(m) * N, n, N, v);
}

// Workgroups the chip holds at once: 256 compute units, each with room (registers) for the 8 waves of one workgroup.
constexpr uint32_t kGemmSlots = 256;

struct GemmShape {
    uint32_t m_tiles, n_tiles, whole, cut_tiles, f, k_per_split, jobs;
};

GemmShape gemm_shape(uint64_t M, uint32_t K, uint32_t N)
{
    GemmShape s;
    s.m_tiles = uint32_t((M + BM - 1) / BM);
    s.n_tiles = (N + BN - 1) / BN;
    const uint32_t tiles = s.m_tiles * s.n_tiles;
    const uint32_t ksteps = (K + BK - 1) / BK;
    s.cut_tiles = tiles % kGemmSlots;
    s.whole = tiles - s.cut_tiles;
    uint32_t f = 1;
    if (s.cut_tiles > 0) f = std::max(1u, std::min({kGemmSlots / s.cut_tiles, std::max(1u, ksteps / 8), 16u}));
    s.k_per_split = (ksteps + f - 1) / f * BK;
    s.f = (K + s.k_per_split - 1) / s.k_per_split;  // slices that are not empty
    if (s.f == 1) {  // nothing to gain from a cut: every tile takes the whole contraction
        s.whole = tiles;
        s.cut_tiles = 0;
    }
    s.jobs = s.whole + s.cut_tiles * s.f;
    return s;
}

}  // namespace

// fp32 partial tiles the product needs in the workspace (0 if every tile writes y directly)
size_t layer_gemm_partial_bytes(uint64_t M, uint32_t in_features, uint32_t out_features)
{
    const GemmShape s = gemm_shape(M, in_features, out_features);
    return align256(size_t(s.cut_tiles) * s.f * BM * BN * 4);
}

// bytes of the weight in fragment layout (whole fragments: columns padded to 32, in-features to 16)
size_t layer_weight_frag_bytes(uint32_t in_features, uint32_t out_features)
{
    return align256(size_t((out_features + 31) / 32) * ((in_features + 15) / 16) * kFragHalves * 2);
}

hipError_t launch_layer_weight_frag(const void* codebook, int bits, int dtype, uint32_t K, uint32_t g, const uint16_t* codes, uint32_t in_features,
                                    uint32_t out_features, void* wf, void* room, size_t room_bytes, hipStream_t s)
{
    if (dtype != 1 && dtype != 2) return hipErrorInvalidValue;
    const uint32_t per_row = (out_features + g - 1) / g, KB = (in_features + 15) / 16, NB = (out_features + 31) / 32;
    const uint32_t J = K * 8 <= kColumnLds ? 4 : (K * 4 <= kColumnLds ? 2 : 1), sets = (g + J - 1) / J;
    // By columns, unless the matrix is small: the columns' way into LDS costs more than it saves. us a call of 520 rows, row by row / by columns: 512 x 512, g = 4
    // 23.8 / 25.5, 1024 x 1024 26.4 / 27.9, 2048 x 2048 39.5 / 39.2, 4096 x 4096 70.7 / 62.8; g = 8: 2048 x 2048 37.6 / 39.8, 4096 x 4096 64.9 / 63.2.
    // Other lengths (rows that no single load fetches): g = 6, 1024 x 1024 29.2 / 28.5, g = 9, 2048 x 2048 51.6 / 41.2.
    const uint64_t weights = uint64_t(in_features) * out_features;
    const bool columns = weights > (g == 4 || g == 8 ? 1u << 22 : 1u << 19) && in_features % 8 == 0 && in_features <= (1u << 20) && per_row >= 2;
    const uint16_t* book = static_cast<const uint16_t*>(codebook);
    const uint32_t stride = columns ? (K * 2 * J + 15) / 16 * 16 : 0;   // bytes
    const bool laid = columns && (K >= 8192 || bits != 16) && size_t(sets) * stride <= room_bytes;   // a small one is as soon read row by row
    if (bits != 16 || laid) {
        const uint32_t n = K * g;
        const auto lay = dtype == 1 ? codebook_columns_kernel<1> : codebook_columns_kernel<2>;
        hipLaunchKernelGGL(lay, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, s, static_cast<const uint8_t*>(codebook), bits, n, g,
                           laid ? J : g, stride / 2, static_cast<uint16_t*>(room));
        book = static_cast<const uint16_t*>(room);
    }
    if (columns) {
        const uint32_t k_steps = (in_features + 31) / 32, items = (per_row + 32 * kBand - 1) / (32 * kBand) * kBand * k_steps;
        const uint32_t parts = std::min(std::max(1u, kUnits / sets), items), per_job = (items + parts - 1) / parts;
        const uint32_t jobs = (items + per_job - 1) / per_job * sets, lds = std::max(stride, K * 2 * J);
        auto go = [&](auto kernel) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kernel, dim3((jobs + 7) / 8 * 8), dim3(kColumnThreads), lds, s, book,
                               laid ? static_cast<const uint8_t*>(room) : static_cast<const uint8_t*>(nullptr), stride, K, g, codes, per_row, in_features,
                               out_features, NB, KB, static_cast<uint16_t*>(wf), sets, jobs, k_steps, items, per_job);
            return hipGetLastError();
        };
        return J == 4 ? go(layer_weight_frag_columns_kernel<4>) : (J == 2 ? go(layer_weight_frag_columns_kernel<2>) : go(layer_weight_frag_columns_kernel<1>));
    }
    const dim3 grid((out_features + 63) / 64, (in_features + 63) / 64);
    if (grid.y > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(layer_weight_frag_kernel, grid, dim3(kThreads), 0, s, book, K, g, codes, per_row, in_features, out_features, NB, KB,
                       static_cast<uint16_t*>(wf));
    return hipGetLastError();
}

// y [M][out] = x [M][in] . W, W as written by launch_layer_weight_frag; scale (device, may be NULL) multiplies the
// finished sum; `partial` holds layer_gemm_partial_bytes(...) bytes
hipError_t launch_layer_gemm(const void* x, uint32_t M, const void* wf, int dtype, uint32_t in_features, uint32_t out_features,
                             const float* scale, const void* bias, void* y, float* partial, uint32_t group, hipStream_t s)
{
    const GemmShape g = gemm_shape(M, in_features, out_features);
    const auto kernel = dtype == 1 ? gemm_frag_kernel<1> : gemm_frag_kernel<2>;
    if (const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(kGemmLdsBytes)); e != hipSuccess) return e;
    const dim3 grid(8 * ((g.whole + 7) / 8) + 8 * ((g.jobs - g.whole + 7) / 8));
    const uint16_t* xs = static_cast<const uint16_t*>(x);
    const uint16_t* ws = static_cast<const uint16_t*>(wf);
    const uint16_t* bs = static_cast<const uint16_t*>(bias);
    uint16_t* ys = static_cast<uint16_t*>(y);
    const uint32_t NB = (out_features + 31) / 32, KB = (in_features + 15) / 16;
    if (dtype != 1 && dtype != 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel, grid, dim3(kGemmThreads), kGemmLdsBytes, s, xs, ws, M, out_features, in_features, NB,
                       KB, scale, bs, ys, partial, g.m_tiles, g.whole, g.f, g.k_per_split, g.jobs, group);
    if (g.cut_tiles > 0) {
        const dim3 fgrid(BM * BN / 8 / kThreads, g.cut_tiles);
        if (dtype == 1)
            hipLaunchKernelGGL(gemm_finish_kernel<1>, fgrid, dim3(kThreads), 0, s, partial, M, out_features, g.m_tiles, g.whole,
                               g.f, scale, bs, ys);
        else
            hipLaunchKernelGGL(gemm_finish_kernel<2>, fgrid, dim3(kThreads), 0, s, partial, M, out_features, g.m_tiles, g.whole,
                               g.f, scale, bs, ys);
    }
    return hipGetLastError();
}

}  // namespace cc
