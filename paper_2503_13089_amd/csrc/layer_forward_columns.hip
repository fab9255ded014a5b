// Forward pass of the compressed linear layer for decoding-sized and small prefill batches: y = x . W (+ bias), codebook rows of
// 4 .. 9 elements of 16, 8 or 4 bits, with no copy of W anywhere.
//
// What bounds such a call is a random codebook access per code. L2 serves one 128-byte line per clock and channel, 0.3 to 0.4
// rows per clock and compute unit, whatever the kernel does; LDS serves 64 numbers in 5 to 10 clocks. A codebook of 65536 rows
// does not fit LDS (160 KB), one of its columns does: a workgroup (one per compute unit, 16 waves) keeps columns j .. j + J - 1
// of the whole codebook, an "entry" of 2, 4 or 8 bytes per row, and computes the outputs that those columns belong to, for
// some of the code columns. The codes are read once per set of columns; every lookup hits, at one per weight (J = 1) or fewer.
// What a lane looks up ARE its matrix-core operands: lane (n, q) of v_mfma_f32_16x16x32 holds 8 consecutive in-features of
// output n, which are the entries of 8 codes below one another. No wave needs another one until their sums are added.
// Tried and slower: whole rows in LDS, a part of the codebook per workgroup and a row of zeros for the codes of the others
// (g = 4 as fast, g = 6: 60 us where this takes 27); rows gathered from L2 straight into the operands (67 us).
//
// Measured, us a call, before (rows from L2 through LDS tiles; the codebook in four parts through LDS; integers by plain
// multiply-adds) and now. K = 65536, 16 bits: 4096 x 4096, g = 4, M = 1 22.6 / 13.3, M = 16 24.2 / 13.9; 4096 x 11008, M = 1 39.1 / 22.5,
// M = 16 59.1 / 24.2, M = 64 69.8 / 37.8, M = 256 116 / 93; 4096 x 10997, g = 6, M = 23 49.1 / 27.2; 8192 x 28672, M = 1 144 / 69; g = 9,
// 4096 x 11008, M = 4 52.3 / 25.2. K = 4096, g = 8: 4096 x 4096, M = 16 15.8 / 13.2, 2048 x 2048, M = 64 14.6 / 12.6. 4 bits: 8192 x 8192, g = 4,
// M = 4 42.7 / 16.3, M = 16 113 / 18.2; 4096 x 11008, g = 6, M = 9 210 / 25.6.
// A call of 4096 x 4096, M = 1: 2.8 us for the copies, then 2.5 us until the codes are requested (their loads, 8 of 2 bytes a step,
// take the address unit 10 clocks each), 2 for the column, 3 for the lookups, 1 for the sums.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "half_types.h"

namespace cc {

namespace {

constexpr uint32_t kStep = 32;             // in-features of a matrix instruction
constexpr uint32_t kLds = 160 * 1024;
constexpr int kWaves = 16, kThreads = 64 * kWaves;
constexpr uint32_t kUnits = 256;           // compute units
constexpr int kSumFloats = 4 * 64 + 8;     // sums of a matrix instruction, and 8 for lanes that read 8 of them to meet 64 banks

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32_2 __attribute__((aligned(2)));
typedef uint64_t u64_2 __attribute__((aligned(2)));
typedef uint64_t u64_1 __attribute__((aligned(1)));

template <int DT>
__device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c)
{
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// J elements of BITS bits: an entry. Integers of 4 bits are held as q + 8.
template <int BITS, int J>
constexpr int kEntryBytes = BITS * J / 8;

// The entry of row k that begins with element j0; elements from g on are zero (16 bits) or anything. One load each, of bytes of
// the codebook only: loads of 2 bytes 16 apart take 24 clocks a wave, whole rows of 16 bytes 16.
template <int BITS, int J>
__device__ __forceinline__ uint64_t make_entry(const uint8_t* __restrict__ book, uint32_t book_bytes, uint32_t g, uint32_t k, uint32_t j0)
{
    uint64_t e = 0;
    if constexpr (BITS == 16 && J == 1) {
        if (g == 8) {   // (j0 is the same for every lane)
            const u32x4 row = reinterpret_cast<const u32x4*>(book)[k];
            const uint32_t w = j0 < 4 ? (j0 < 2 ? row[0] : row[1]) : (j0 < 6 ? row[2] : row[3]);
            e = uint16_t(w >> (16 * (j0 % 2)));
        } else {
            e = reinterpret_cast<const uint16_t*>(book)[size_t(k) * g + j0];
        }
    } else if constexpr (BITS == 16) {
        const uint32_t j1 = min(j0, g - J);   // the row's last J elements, moved down: J <= 4 <= g
        const uint16_t* from = reinterpret_cast<const uint16_t*>(book) + size_t(k) * g + j1;
        if constexpr (J == 2) e = *reinterpret_cast<const u32_2*>(from);
        else e = *reinterpret_cast<const u64_2*>(from);
        e >>= 16 * (j0 - j1);
    } else {
        const uint64_t bit = (uint64_t(k) * g + j0) * BITS;
        const uint32_t at = uint32_t(bit / 8), shift = uint32_t(bit % 8);   // shift: 0 or 4
        if (book_bytes >= 8) {
            const uint32_t at1 = min(at, book_bytes - 8);   // what the codebook ends before is not used
            e = *reinterpret_cast<const u64_1*>(book + at1) >> (8 * (at - at1));
        } else {
#pragma unroll
            for (uint32_t b = 0; b <= kEntryBytes<BITS, J>; ++b) e |= uint64_t(book[min(at + b, book_bytes - 1)]) << (8 * b);
        }
        e = (e >> shift) ^ (BITS == 8 ? 0ull : 0x8888888888888888ull);
    }
    return e;
}

template <int BITS, int J>
__device__ __forceinline__ void put_entry(uint8_t* dst, uint32_t k, uint64_t e)
{
    constexpr int E = kEntryBytes<BITS, J>;
    if constexpr (E == 2) reinterpret_cast<uint16_t*>(dst)[k] = uint16_t(e);
    else if constexpr (E == 4) reinterpret_cast<uint32_t*>(dst)[k] = uint32_t(e);
    else reinterpret_cast<uint64_t*>(dst)[k] = e;
}

// The in-features of lanes (., q) in the step that begins at k0: base + 8 q .. + 7. A last step that in_features does not fill begins
// earlier instead; what it has twice, or beyond a matrix of less than one step, is cleared in both operands.
__device__ __forceinline__ uint32_t step_base(uint32_t k0, uint32_t in_features) { return in_features >= kStep ? min(k0, in_features - kStep) : 0u; }
__device__ __forceinline__ uint32_t lane_features(uint32_t q, uint32_t in_features) { return min(8 * q, in_features - 8); }
__device__ __forceinline__ bool lane_dead(uint32_t k0, uint32_t q, uint32_t in_features)
{
    return step_base(k0, in_features) + 8 * q < k0 || 8 * q >= in_features;
}

// Ahead of the product: the codebook by sets of J columns, [sets][stride] bytes, and the rows of x as operands, [row tiles][steps]
// [MT][64 lanes] of 16 bytes, zero past the last row. Row by row, a load of x would touch 64 cache lines instead of 8.
template <int BITS, int J>
__global__ __launch_bounds__(256) void forward_columns_layout_kernel(const uint8_t* __restrict__ book, uint32_t book_bytes, uint32_t g,
                                                                     uint32_t K, uint32_t sets, uint32_t stride, uint8_t* __restrict__ out,
                                                                     uint32_t book_blocks, const uint16_t* __restrict__ x, uint32_t M,
                                                                     uint32_t MT, uint32_t in_features, u32x4* __restrict__ x_out)
{
    if (blockIdx.x < book_blocks) {
        const uint32_t set = blockIdx.x % sets, k = blockIdx.x / sets * 256 + threadIdx.x;
        if (k < K) put_entry<BITS, J>(out + size_t(set) * stride, k, make_entry<BITS, J>(book, book_bytes, g, k, set * J));
        return;
    }
    const uint32_t t = (blockIdx.x - book_blocks) * 256 + threadIdx.x;   // read in the order of x
    const uint32_t eights = (in_features + kStep - 1) / kStep * 4, m = t / eights, e = t % eights, k0 = e / 4 * kStep;
    const uint32_t tile = m / (16 * MT), tiles = (M + 16 * MT - 1) / (16 * MT);
    if (tile >= tiles) return;
    const int k = int(step_base(k0, in_features)) + int(lane_features(e % 4, in_features));
    u32x4 v = {0u, 0u, 0u, 0u};
    if (m < M) v = *reinterpret_cast<const u32x4*>(x + size_t(m) * in_features + k);
    x_out[(size_t(tile * (eights / 4) + e / 4) * MT + m / 16 % MT) * 64 + (e % 4) * 16 + m % 16] = v;
}

struct ColumnArgs {
    const uint16_t* x;
    uint32_t M;
    const uint8_t* book;
    uint32_t book_bytes, K, g, sets;
    const uint8_t* laid;         // NULL, or the codebook by sets of columns, laid_stride bytes each (multiples of 16)
    uint32_t laid_stride;
    const u32x4* x_laid;         // NULL, or x as operands
    const uint16_t* codes;
    uint32_t per_row, in_features, out_features;
    const float* scale;          // NULL, or what multiplies the sum
    const uint16_t* bias;
    uint16_t* y;
    float* partial;              // [slices][M][out_features] if there is more than one
    uint32_t CW, tiles;          // column groups of a workgroup; workgroups side by side
    uint32_t row_tiles;          // of 16 * MT rows of x
    uint32_t slices, slice_rows; // of the in-features, in multiples of kStep
};

// The operand of element j from the words of 8 entries (two entries a word where they are of 2 bytes). Integers become operands with
// their sign: with an offset left in and taken off the finished sum, the fp32 sum would round at the size of the offset's
// share, several times its own. Signed bytes convert in one instruction, as unsigned ones do; nibbles become signed bytes four at a
// time (8192 x 8192, g = 4, M = 4: 16.3 us, with an offset of 8 for up to 16 rows 17.5).
template <int DT, int BITS, int J, int RW>
__device__ __forceinline__ u32x4 operand(const uint32_t (&w)[RW], int j)
{
    u32x4 b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (BITS == 16 && J == 1) {
            b[i] = w[i];
        } else if constexpr (BITS == 16) {
            b[i] = __builtin_amdgcn_perm(w[(2 * i + 1) * (J / 2) + j / 2], w[2 * i * (J / 2) + j / 2], j % 2 ? 0x07060302u : 0x05040100u);
        } else {
            float f[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t v = kEntryBytes<BITS, J> == 2 ? w[i] : w[2 * i + e];
                const int first = kEntryBytes<BITS, J> == 2 ? 2 * e : 0;   // byte
                if constexpr (BITS == 8) {
                    f[e] = float(int8_t(v >> (8 * (first + j))));
                } else {   // 0 .. 15 + 0x78 carries into no other byte
                    const uint32_t q = (((j % 2 ? v >> 4 : v) & 0x0f0f0f0fu) + 0x78787878u) ^ 0x80808080u;
                    f[e] = float(int8_t(q >> (8 * (first + j / 2))));
                }
            }
            if constexpr (DT == 1) b[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(f[0], f[1]));   // exact, as
            else b[i] = __builtin_amdgcn_perm(__float_as_uint(f[1]), __float_as_uint(f[0]), 0x07060302u);         // is this
        }
    }
    return b;
}

// One workgroup: a set of J columns of the codebook, 16 * NC * CW code columns and a slice of the in-features; wave (ks, cw)
// takes every KW-th step of 32 in-features of column group cw, lane (n, q) the code columns NC * n .. of the group.
template <int DT, int BITS, int J, int MT, int NC>
__global__ __launch_bounds__(kThreads, kWaves / 4) void layer_forward_columns_kernel(const ColumnArgs p)
{
    constexpr int E = kEntryBytes<BITS, J>, RW = E == 2 ? 4 : 2 * E;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane = threadIdx.x & 63, n16 = lane & 15, kg = lane >> 4;
    const uint32_t wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    // consecutive workgroup ids go to different XCDs: XCD q takes the q-th share of the jobs (sets of the same codes are
    // neighbours, then tiles of the same x)
    const uint32_t total = p.sets * p.tiles * p.slices * p.row_tiles;
    uint32_t job = blockIdx.x;
    if (total % 8 == 0) job = (blockIdx.x % 8) * (total / 8) + blockIdx.x / 8;
    const uint32_t set = job % p.sets, tile = job / p.sets % p.tiles, rest = job / p.sets / p.tiles, slice = rest % p.slices;
    const uint32_t row_tile = rest / p.slices, row0 = row_tile * 16 * MT, rows = min(p.M - row0, uint32_t(16 * MT));
    const uint32_t CW = p.CW, KW = kWaves / CW, cw = wave % CW, ks = wave / CW;   // ks == KW: nothing to do
    const uint32_t k_begin = slice * p.slice_rows, k_end = min(k_begin + p.slice_rows, p.in_features);
    auto column = [&](uint32_t group, uint32_t n) { return min((tile * CW + group) * (16 * NC) + n * NC, p.per_row - NC); };   // the first of NC

    f32x4 acc[MT][NC][J];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < J; ++j) acc[mt][c][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    const uint32_t stride = KW * kStep, k_first = k_begin + ks * kStep;
    const uint32_t steps = ks < KW && k_first < k_end ? (k_end - k_first + stride - 1) / stride : 0u;   // of this wave
    uint32_t code[2][8];   // of this step and the next; two neighbouring ones in a register where NC is 2
    u32x4 xs[2][MT];
    const uint32_t lane_k = lane_features(kg, p.in_features), lane_code = 2 * (lane_k * p.per_row + column(cw, n16));   // bytes
    auto load_codes = [&](uint32_t base, uint32_t (&c)[8]) {
        const char* from = reinterpret_cast<const char*>(p.codes + size_t(base) * p.per_row);
        if constexpr (MT == 4) {
            // Sums of 64 rows leave no registers for eight 64-bit addresses: 24 bytes a lane went through scratch memory, whose loads wait for all the others. A scalar and
            // 32 bits instead: M = 64, 4096 x 11008 36.8 -> 32.2 us, M = 200, 4096 x 4096 37.0 -> 32.2, 4 bits, M = 64, 4096 x 4096 22.0 -> 20.1
            // (37 of its registers still go through scratch, 51 before; 8 and 16 bits none). With fewer rows it is up to 6 % slower.
            typedef const __attribute__((address_space(1))) char* Global;
            uint32_t off = lane_code;
            asm volatile("" : "+v"(off));
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) {
                Global q = reinterpret_cast<Global>(reinterpret_cast<uintptr_t>(from + size_t(2 * i) * p.per_row));
                asm volatile("" : "+s"(q));
                if constexpr (NC == 1) c[i] = *reinterpret_cast<const __attribute__((address_space(1))) uint16_t*>(q + off);
                else c[i] = *reinterpret_cast<const __attribute__((address_space(1))) u32_2*>(q + off);
            }
        } else {
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) {
                const char* q = from + size_t(2 * i) * p.per_row + lane_code;
                if constexpr (NC == 1) c[i] = *reinterpret_cast<const uint16_t*>(q);
                else c[i] = *reinterpret_cast<const u32_2*>(q);
            }
        }
    };
    const char* x_at[MT];   // the lane's part of x
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)   // rows past M repeat the last one
        x_at[mt] = p.x_laid != nullptr ? reinterpret_cast<const char*>(p.x_laid + size_t(row_tile) * ((p.in_features + kStep - 1) / kStep) * MT * 64 + 64 * mt + lane)
                                       : reinterpret_cast<const char*>(p.x + size_t(row0 + min(uint32_t(16 * mt + n16), rows - 1)) * p.in_features + lane_k);
    auto load_x = [&](uint32_t k0, uint32_t base, u32x4 (&a)[MT]) {
        const size_t off = p.x_laid != nullptr ? size_t(k0) * (32 * MT) : size_t(base) * 2;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[mt] = *reinterpret_cast<const u32x4*>(x_at[mt] + off);
    };
    auto request = [&](uint32_t at, int i) {   // step `at` of the wave, or its last one again
        const uint32_t k0 = k_first + min(at, steps - 1) * stride, base = step_base(k0, p.in_features);
        load_x(k0, base, xs[i]);
        load_codes(base, code[i]);
    };
    if (steps > 0) {
        request(0, 0);
        if (steps > 1) request(1, 1);
    }
    // ---- the columns into LDS. Every workgroup starts at another place, so that they do not all ask the same cache channels
    if (p.laid != nullptr || (p.sets == 1 && uint32_t(E) * 8 == p.g * BITS)) {
        const uint8_t* src = p.laid != nullptr ? p.laid + size_t(set) * p.laid_stride : p.book;
        const uint32_t offset = p.laid != nullptr || BITS != 4 ? 0u : 0x88888888u;   // to q + 8
        const uint32_t bytes = p.K * E, pieces = bytes / 16, turn = pieces > 0 ? (blockIdx.x / 8 * 331u + blockIdx.x) % pieces : 0u;
        constexpr int U = 8;
        for (uint32_t i0 = threadIdx.x; i0 < pieces; i0 += U * kThreads) {
            u32x4 t[U];
            uint32_t at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                at[u] = min(i0 + u * kThreads, pieces - 1) + turn;
                at[u] = at[u] >= pieces ? at[u] - pieces : at[u];
                t[u] = *reinterpret_cast<const u32x4*>(src + 16 * size_t(at[u]));
            }
#pragma unroll
            for (int u = 0; u < U; ++u) *reinterpret_cast<u32x4*>(smem + 16 * at[u]) = t[u] ^ offset;
        }
        for (uint32_t i = pieces * 8 + threadIdx.x; i < bytes / 2; i += kThreads)
            reinterpret_cast<uint16_t*>(smem)[i] = reinterpret_cast<const uint16_t*>(src)[i] ^ uint16_t(offset);
    } else {
        constexpr int U = 4;
        for (uint32_t k0 = threadIdx.x; k0 < p.K; k0 += U * kThreads) {
            uint64_t e[U];
#pragma unroll
            for (int u = 0; u < U; ++u) e[u] = make_entry<BITS, J>(p.book, p.book_bytes, p.g, min(k0 + u * kThreads, p.K - 1), set * J);
#pragma unroll
            for (int u = 0; u < U; ++u) put_entry<BITS, J>(smem, min(k0 + u * kThreads, p.K - 1), e[u]);
        }
    }
    __syncthreads();

    if (steps > 0) {
        const u16x2 last = {uint16_t(p.K - 1), uint16_t(p.K - 1)};
        auto step = [&](uint32_t at, int i, auto more) {
            const uint32_t k0 = k_first + at * stride;
            uint32_t (&c)[8] = code[i];
            uint32_t w[NC][RW];
#pragma unroll
            for (int v = 0; v < NC; ++v)
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const u16x2 both = __builtin_elementwise_min(__builtin_bit_cast(u16x2, c[r]), last);   // never outside the codebook
                    const uint32_t from = uint32_t(both[v]) * E;
                    if constexpr (E == 2) {
                        u16x2 pair = __builtin_bit_cast(u16x2, w[v][r / 2]);
                        pair[r % 2] = *reinterpret_cast<const uint16_t*>(smem + from);
                        w[v][r / 2] = __builtin_bit_cast(uint32_t, pair);
                    } else if constexpr (E == 4) {
                        w[v][r] = *reinterpret_cast<const uint32_t*>(smem + from);
                    } else {
                        const uint2 t = *reinterpret_cast<const uint2*>(smem + from);
                        w[v][2 * r] = t.x; w[v][2 * r + 1] = t.y;
                    }
                }
            u32x4 a[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[mt] = xs[i][mt];
            if constexpr (more) request(at + 2, i);
            if (step_base(k0, p.in_features) != k0 || p.in_features < kStep) {
                const bool dead = lane_dead(k0, kg, p.in_features);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) a[mt][r] = dead ? 0u : a[mt][r];
                if constexpr (BITS == 16) {   // integers are finite
#pragma unroll
                    for (int v = 0; v < NC; ++v)
#pragma unroll
                        for (int r = 0; r < RW; ++r) w[v][r] = dead ? 0u : w[v][r];
                }
            }
#pragma unroll
            for (int v = 0; v < NC; ++v)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const u32x4 b = operand<DT, BITS, J, RW>(w[v], j);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[mt][v][j] = mma<DT>(a[mt], b, acc[mt][v][j]);
                }
        };
        uint32_t at = 0;
        for (; at + 2 < steps; at += 2) {
            step(at, 0, std::true_type{});
            step(at + 1, 1, std::true_type{});
        }
        step(at, 0, std::false_type{});
        if (at + 1 < steps) step(at + 1, 1, std::false_type{});
    }

    // ---- the waves of a column group are added and stored, as many rows at a time as there is room for
    constexpr int Q = NC * J, T = MT * Q > 8 ? MT / 2 : MT;
    float (*red)[Q][kSumFloats] = reinterpret_cast<float (*)[Q][kSumFloats]>(smem);   // [kWaves * T], [4][64] each
    const float scale = p.scale != nullptr && p.slices == 1 ? *p.scale : 1.0f;
#pragma unroll
    for (int t0 = 0; t0 < MT; t0 += T) {
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < T; ++mt)
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[wave * T + mt][q][64 * i + lane] = acc[t0 + mt][q / J][q % J][i];
        __syncthreads();
        const uint32_t width = CW * 16 * Q, here = min(rows > uint32_t(16 * t0) ? rows - 16 * t0 : 0u, uint32_t(16 * T)), count = here * width;
#pragma unroll 1
        for (uint32_t e = threadIdx.x; e < count; e += kThreads) {
            const uint32_t mm = e / width, rest = e % width, q = rest % Q, c16 = rest / Q % 16, cg = rest / (16 * Q), mt = mm / 16, m = row0 + 16 * t0 + mm;
            const uint32_t at = 64 * (mm % 4) + 16 * (mm % 16 / 4) + c16;
            float part[kWaves], v = 0.0f;
#pragma unroll
            for (uint32_t s = 0; s < kWaves; ++s) part[s] = red[min(s * CW + cg, uint32_t(kWaves - 1)) * T + mt][q][at];
#pragma unroll
            for (uint32_t s = 0; s < kWaves; ++s) v += s < KW ? part[s] : 0.0f;
            const uint32_t j = set * J + q % J, n = p.g * (column(cg, c16) + q / J) + j;
            if (j < p.g && n < p.out_features) {
                if (p.slices > 1) {
                    p.partial[(size_t(slice) * p.M + m) * p.out_features + n] = v;
                } else {
                    v *= scale;
                    p.y[size_t(m) * p.out_features + n] = from_f32<DT>(p.bias ? v + to_f32<DT>(p.bias[n]) : v);
                }
            }
        }
    }
}

// How a call is cut: estimated clocks of a workgroup times rounds over the chip. The constants are fitted to measured calls. Against the
// best of all cuts (NC, CW and 12 numbers of slices, all timed) over 34 shapes of 1 to 256 rows, 512 x 512 to 8192 x 28672, 27 are within 3 %;
// 6 take 6 to 25 % longer (layers of less than 1100 outputs, and 1 and 2 rows of 4 bits: too many slices), and one of 930 outputs, K = 4096,
// 8 bits twice as long (17 us with 44 slices, 8.5 with 8).
struct Cut {
    uint32_t CW, tiles, slices, slice_rows;
    float clocks;
};

Cut choose_cut(uint32_t M, uint32_t in_features, uint32_t out_features, uint32_t per_row, uint32_t jobs, uint32_t nc, float step_clocks, float fixed,
               uint32_t most_slices)
{
    const uint32_t groups = (per_row + 16 * nc - 1) / (16 * nc), steps = (in_features + kStep - 1) / kStep;
    Cut best{};
    best.clocks = 1e30f;
    for (uint32_t cw = 1; cw <= uint32_t(kWaves); ++cw) {
        const uint32_t kw = kWaves / cw, tiles = (groups + cw - 1) / cw;
        for (uint32_t full = 0; full <= 2; ++full) {   // no slices, or as many as fill the chip once or twice
            const uint32_t sl = std::max<uint32_t>(1, std::min({full * kUnits / (tiles * jobs), most_slices, steps}));
            const uint32_t rounds = (tiles * sl * jobs + kUnits - 1) / kUnits, per_slice = (steps + sl - 1) / sl, per_wave = (per_slice + kw - 1) / kw;
            const float clocks = rounds * (fixed + per_wave * std::max(float(kw * cw) * step_clocks, 900.0f)) +
                                 (sl > 1 ? 6000.0f + float(sl) * M * out_features * 0.003f : 0.0f);
            if (clocks < best.clocks) best = Cut{cw, tiles, (steps + per_slice - 1) / per_slice, per_slice * kStep, clocks};
        }
    }
    return best;
}

template <int DT, int BITS, int J, int MT, int NC>
hipError_t launch_t(ColumnArgs p, const Cut& c, hipStream_t s)
{
    p.CW = c.CW; p.tiles = c.tiles; p.slices = c.slices; p.slice_rows = c.slice_rows;
    const uint32_t lds = std::max<uint32_t>(p.K * kEntryBytes<BITS, J>, kWaves * std::min(MT * NC * J, 8) * kSumFloats * 4);
    const auto kernel = layer_forward_columns_kernel<DT, BITS, J, MT, NC>;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(p.sets * p.tiles * p.slices * p.row_tiles), dim3(kThreads), lds, s, p);
    if (p.slices > 1) return launch_layer_forward_reduce(p.partial, p.M, p.out_features, p.slices, p.scale, p.bias, p.y, DT, s);
    return hipGetLastError();
}

// Rows of x (in 16) and code columns per lane that a kernel exists for: their sums fit the registers of four waves per SIMD
template <int BITS, int J>
constexpr bool cut_exists(uint32_t mt, uint32_t nc) { return mt * nc * J <= 8 || (BITS == 4 && mt == 4 && nc == 1 && J == 4); }

template <int BITS, int J>
hipError_t launch_entries(ColumnArgs p, int dtype, uint32_t most_slices, size_t room, hipStream_t s)
{
    constexpr int E = kEntryBytes<BITS, J>;
    p.sets = (p.g + J - 1) / J;
    const uint32_t stride = (p.K * E + 15) / 16 * 16, steps = (p.in_features + kStep - 1) / kStep;
    const bool as_it_is = (p.sets == 1 && uint32_t(E) * 8 == p.g * BITS) || p.K < 8192;   // the columns come from the codebook itself
    const uint32_t mt = p.M <= 16 ? 1 : (p.M <= 32 ? 2 : 4);
    p.row_tiles = (p.M + 16 * mt - 1) / (16 * mt);
    // clocks of a step of one wave: address unit (codes, x as it is or laid out), lookups, arithmetic (integers: fitted; with the instructions
    // that they take, 12 a column for 8 bits and 19 for 4, three shapes of 90 got slower by 9 to 17 %, two faster)
    const float x_rows = p.M <= 16 ? std::min(64.0f, 12.0f + 4.0f * p.M) : 64.0f * mt;
    // x laid out: where a launch for the codebook is needed anyway, or the lines saved are worth one
    const float x_saved = float(p.sets) * p.row_tiles * p.per_row * p.in_features / (16.0f * kStep * kUnits) * (x_rows - 16.0f * mt);
    bool x_laid = x_saved > (as_it_is ? 12000.0f : 1000.0f);
    const size_t x_bytes = size_t(p.row_tiles) * steps * mt * 1024, book_bytes = as_it_is ? 0 : size_t(p.sets) * stride;
    auto step_clocks = [&](uint32_t nc) {
        const float lines = 80.0f + (x_laid ? 16.0f * mt : x_rows), lookups = nc * (E == 8 ? 90.0f : 60.0f);
        const float alu = 20.0f + nc * (18.0f + (BITS == 16 ? (J == 1 ? 0.0f : 4.0f * J) : (mt == 1 && BITS == 4 ? 15.0f : 22.0f) * J));
        return 1.1f * std::max(std::max(lookups, alu), lines);
    };
    const float fixed = float(p.K) * E * 0.035f + 8000.0f;
    Cut best{};
    best.clocks = 1e30f;
    uint32_t nc_best = 1;
    for (uint32_t nc : {1u, 2u}) {
        if (!cut_exists<BITS, J>(mt, nc) || nc > p.per_row) continue;
        const Cut c = choose_cut(p.M, p.in_features, p.out_features, p.per_row, p.sets * p.row_tiles, nc, step_clocks(nc), fixed, most_slices);
        if (c.clocks < best.clocks) { best = c; nc_best = nc; }
    }
    // behind the partial sums, if there is room
    const size_t partial_bytes = best.slices > 1 ? align256(size_t(best.slices) * p.M * p.out_features * 4) : 0;
    // Without room for the codebook's copy (one row or a few through a workspace of the sums' size) every workgroup takes its columns
    // out of whole rows: 16 bits, M = 1, us with room / without / rows gathered tile by tile, as every length was before: K = 65536, g = 4, 1024 x 1024
    // 9.0 / 12.0 / 12.2, 2048 x 2048 9.7 / 13.5 / 12.1, 4096 x 4096 12.3 / 16.4 / 21.9; g = 6, 4096 x 4096 16.5 / 20.1 / 19.2; g = 8, 1024 x 1024 9.7 / 15.2 / 11.9,
    // 4096 x 4096 13.1 / 19.5 / 15.3, 4096 x 11008 21.3 / 27.3 / 34.3; g = 9, 2048 x 2048 10.9 / 14.6 / 12.0. K = 20000, g = 9, 4096 x 4096 12.6 / 12.2 / 21.0.
    if (room < partial_bytes + align256(book_bytes) + x_bytes) x_laid = false;
    const bool laid = !as_it_is && room >= partial_bytes + book_bytes;
    if (laid || x_laid) {
        uint8_t* at = reinterpret_cast<uint8_t*>(p.partial) + partial_bytes;
        p.laid = laid ? at : nullptr;
        p.laid_stride = stride;
        p.x_laid = x_laid ? reinterpret_cast<const u32x4*>(at + align256(book_bytes)) : nullptr;
        const uint32_t book_blocks = laid ? (p.K + 255) / 256 * p.sets : 0, x_blocks = x_laid ? uint32_t((uint64_t(steps) * 4 * 16 * mt * p.row_tiles + 255) / 256) : 0;
        hipLaunchKernelGGL((forward_columns_layout_kernel<BITS, J>), dim3(book_blocks + x_blocks), dim3(256), 0, s, p.book, p.book_bytes, p.g, p.K,
                           p.sets, stride, at, book_blocks, p.x, p.M, mt, p.in_features, const_cast<u32x4*>(p.x_laid));
    }
#define CC_C(MT, NC)                                                                                       \
    if constexpr (cut_exists<BITS, J>(MT, NC))                                                                   \
        if (mt == MT && nc_best == NC) return dtype == 1 ? launch_t<1, BITS, J, MT, NC>(p, best, s) : launch_t<2, BITS, J, MT, NC>(p, best, s)
    CC_C(1, 1);
    CC_C(1, 2);
    CC_C(2, 1);
    CC_C(2, 2);
    CC_C(4, 1);
    CC_C(4, 2);
#undef CC_C
    return hipErrorInvalidValue;
}

}  // namespace

size_t layer_forward_columns_room(uint64_t M, uint32_t in_features)
{
    const uint64_t mt = M <= 16 ? 1 : (M <= 32 ? 2 : 4), steps = (uint64_t(in_features) + kStep - 1) / kStep;
    return align256(size_t(65536) * kMostColumns * 2) + align256((M + 16 * mt - 1) / (16 * mt) * steps * mt * 1024);
}

hipError_t launch_layer_forward_columns(const void* x, uint32_t M, const void* book, int bits, const float* scale, uint32_t K, uint32_t g,
                                        const uint16_t* codes, uint32_t in_features, uint32_t out_features, const void* bias, void* y,
                                        int dtype, void* workspace, size_t workspace_bytes, uint32_t most_slices, hipStream_t s)
{
    ColumnArgs p{};
    p.x = static_cast<const uint16_t*>(x); p.M = M;
    p.book = static_cast<const uint8_t*>(book); p.K = K; p.g = g;
    p.book_bytes = uint32_t((uint64_t(K) * g * bits + 7) / 8);
    p.codes = codes; p.in_features = in_features; p.out_features = out_features;
    p.per_row = (out_features + g - 1) / g;
    p.scale = scale;
    p.bias = static_cast<const uint16_t*>(bias); p.y = static_cast<uint16_t*>(y);
    p.partial = static_cast<float*>(workspace);
    const size_t room = workspace != nullptr ? workspace_bytes : 0;
    // as wide entries as fit
    if (bits == 16) {
        if (K * 8 <= kLds && M <= 32) return launch_entries<16, 4>(p, dtype, most_slices, room, s);
        if (K * 4 <= kLds) return launch_entries<16, 2>(p, dtype, most_slices, room, s);
        return launch_entries<16, 1>(p, dtype, most_slices, room, s);
    }
    if (bits == 8) {
        if (K * 4 <= kLds && M <= 32) return launch_entries<8, 4>(p, dtype, most_slices, room, s);
        return launch_entries<8, 2>(p, dtype, most_slices, room, s);
    }
    if (K * 4 <= kLds && g > 4 && M <= 16) return launch_entries<4, 8>(p, dtype, most_slices, room, s);
    return launch_entries<4, 4>(p, dtype, most_slices, room, s);
}

}  // namespace cc
