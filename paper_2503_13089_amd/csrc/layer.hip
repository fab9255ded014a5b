// Data movement of the compressed linear layer (Section 3.1 footnote, Section 3.2, the paper's layer
// listing): the reshape that produces the vectors to cluster, the 16-bit storage formats, and the
// reconstruction of the weight from (codebook, codes) with the padding columns cut off.
#include <type_traits>

#include "common.h"

namespace cc {

constexpr int kThreads = 256;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---- element conversions -----------------------------------------------------------------------
// bf16 is the upper half of the fp32 pattern; rounding to nearest even adds 0x7fff + (lowest kept bit).
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float v)
{
    const uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN
    return uint16_t((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }
__device__ __forceinline__ uint16_t f32_to_f16_bits(float v)
{
    const _Float16 h = _Float16(v);  // round to nearest even
    return *reinterpret_cast<const uint16_t*>(&h);
}
__device__ __forceinline__ float f16_bits_to_f32(uint16_t b) { return float(*reinterpret_cast<const _Float16*>(&b)); }

template <int DT>
__device__ __forceinline__ float load_as_f32(const void* p, size_t i)
{
    if constexpr (DT == 0) return static_cast<const float*>(p)[i];
    else if constexpr (DT == 1) return f16_bits_to_f32(static_cast<const uint16_t*>(p)[i]);
    else return bf16_bits_to_f32(static_cast<const uint16_t*>(p)[i]);
}

// ---- vectors to cluster: transpose [out, in] -> [in, out + deficiency] with zero padding, as fp32.
// 64 x 64 tiles through LDS so that both the reads (along in) and the writes (along out) are contiguous.
template <int DT>
__global__ __launch_bounds__(kThreads) void layer_vectors_kernel(const void* __restrict__ weight, uint32_t out_features,
                                                                 uint32_t in_features, uint32_t width,
                                                                 float* __restrict__ vectors)
{
    __shared__ float tile[64][65];
    const uint32_t c0 = blockIdx.x * 64;  // first out-feature (column of the transpose) of this tile
    const uint32_t r0 = blockIdx.y * 64;  // first in-feature (row of the transpose)
    const uint32_t tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (uint32_t j = ty; j < 64; j += 4) {  // weight rows c0 + j, columns r0 + tx
        const uint32_t c = c0 + j, r = r0 + tx;
        tile[j][tx] = (c < out_features && r < in_features) ? load_as_f32<DT>(weight, size_t(c) * in_features + r) : 0.0f;
    }
    __syncthreads();
    for (uint32_t j = ty; j < 64; j += 4) {  // transposed rows r0 + j, columns c0 + tx (padding columns get the zeros)
        const uint32_t r = r0 + j, c = c0 + tx;
        if (r < in_features && c < width) vectors[size_t(r) * width + c] = tile[tx][j];
    }
}

hipError_t launch_layer_vectors(const void* weight, int dtype, uint32_t out_features, uint32_t in_features, uint32_t g,
                                float* vectors, hipStream_t s)
{
    const uint32_t width = (out_features + g - 1) / g * g;
    const dim3 grid((width + 63) / 64, (in_features + 63) / 64);
    switch (dtype) {
        case 0: hipLaunchKernelGGL(layer_vectors_kernel<0>, grid, dim3(kThreads), 0, s, weight, out_features, in_features, width, vectors); break;
        case 1: hipLaunchKernelGGL(layer_vectors_kernel<1>, grid, dim3(kThreads), 0, s, weight, out_features, in_features, width, vectors); break;
        case 2: hipLaunchKernelGGL(layer_vectors_kernel<2>, grid, dim3(kThreads), 0, s, weight, out_features, in_features, width, vectors); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---- storage formats
template <int DT>
__global__ __launch_bounds__(kThreads) void pack_codebook_kernel16(const float* __restrict__ in, size_t n,
                                                                  uint16_t* __restrict__ out)
{
    const size_t i = size_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) out[i] = DT == 1 ? f32_to_f16_bits(in[i]) : f32_to_bf16_bits(in[i]);
}

hipError_t launch_layer_pack_codebook(const float* centroids, size_t n, void* codebook, int dtype, hipStream_t s)
{
    const dim3 grid(uint32_t((n + kThreads - 1) / kThreads));
    uint16_t* out = static_cast<uint16_t*>(codebook);
    switch (dtype) {
        case 1: hipLaunchKernelGGL(pack_codebook_kernel16<1>, grid, dim3(kThreads), 0, s, centroids, n, out); break;
        case 2: hipLaunchKernelGGL(pack_codebook_kernel16<2>, grid, dim3(kThreads), 0, s, centroids, n, out); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void pack_codes_kernel(const uint32_t* __restrict__ idx, uint64_t n, uint32_t K,
                                                              uint16_t* __restrict__ codes)
{
    const uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) codes[i] = uint16_t(min(idx[i], K - 1));
}

hipError_t launch_layer_pack_codes(const uint32_t* idx, uint64_t n, uint32_t K, uint16_t* codes, hipStream_t s)
{
    hipLaunchKernelGGL(pack_codes_kernel, dim3(uint32_t((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, idx, n, K,
                       codes);
    return hipGetLastError();
}

// ---- reconstruction: weight[r][c .. c + g) = codebook[code of (r, c / g)] minus the padding.
// Consecutive codes fill consecutive elements, across the ends of rows too: element j of code v goes to v g + j less the padding of
// the rows before. A wave takes 64 P codes, puts their rows (one load of up to 16 bytes, or two) side by side in LDS where the
// 16-byte pieces of the output begin, and stores whole pieces; up to 7 elements at either end singly. G is the row in 16-bit units
// (fp32: 2 g), `padding` and out_features too. No wave needs another one.
// Element by element the loads and stores are what counts (2 G + 1 an instruction each). 4096 x 11005, K = 65536, us, before and
// now: g = 4 108 / 49, g = 5 (K = 35000) 119 / 45, g = 6 105 / 38, g = 8 109 / 31, g = 9 121 / 39; 512 x 700 9.3 / 6.6.
// Now bound by a codebook line from L2 per code (0.3 to 0.4 a clock and compute unit) where K = 65536; K = 4096, g = 4 26.
template <int G>
constexpr int kCodesPerLane = G <= 9 ? 4 : (G <= 18 ? 2 : 1);

template <int G>
struct CodeRow {
    uint16_t e[G];
    __device__ __forceinline__ void load(const uint16_t* p)
    {
        constexpr int A = G % 8 == 0 ? 16 : (G % 4 == 0 ? 8 : (G % 2 == 0 ? 4 : 2));   // of every row: the codebook begins at 16 bytes
        __builtin_memcpy(e, __builtin_assume_aligned(p, A), G * 2);
    }
};

template <int G, bool EVEN>
__global__ __launch_bounds__(kThreads) void layer_weight_kernel(const uint16_t* __restrict__ codebook, uint32_t K, const uint16_t* __restrict__ codes,
                                                                uint64_t num_codes, uint32_t per_row, uint32_t padding, uint16_t* __restrict__ weight)
{
    constexpr int P = kCodesPerLane<G>;
    constexpr uint32_t C = 64 * P;
    __shared__ __attribute__((aligned(16))) uint16_t lds[kThreads / 64][C * G + 8];
    const uint32_t lane = threadIdx.x & 63, wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    const uint64_t first = (uint64_t(blockIdx.x) * (kThreads / 64) + wave) * C;
    if (first >= num_codes) return;
    const uint32_t n = uint32_t(min(num_codes - first, uint64_t(C)));
    const uint64_t r0 = first / per_row;
    const uint32_t c0 = uint32_t(first - r0 * per_row);
    uint32_t code[P];
#pragma unroll
    for (int p = 0; p < P; ++p) code[p] = codes[first + min(lane + 64 * p, n - 1)];
    CodeRow<G> row[P];
#pragma unroll
    for (int p = 0; p < P; ++p) row[p].load(codebook + size_t(min(code[p], K - 1)) * G);   // never read outside the codebook
    const uint64_t begin = first * G - r0 * padding;        // of the wave's elements
    const uint32_t shift = uint32_t(begin % 8);
    uint16_t* out = lds[wave];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t i = lane + 64 * p, c = c0 + i;
        const uint32_t ends = per_row >= C ? (c >= per_row ? 1u : 0u) : c / per_row;   // rows that end before this code
        const uint32_t keep = c - ends * per_row == per_row - 1 ? G - padding : uint32_t(G);
        uint16_t* at = out + shift + i * G - ends * padding;
        if (i < n) {
            if (EVEN) {
#pragma unroll
                for (int j = 0; j < G / 2; ++j)
                    if (uint32_t(2 * j) < keep)
                        reinterpret_cast<uint32_t*>(at)[j] = uint32_t(row[p].e[2 * j]) | uint32_t(row[p].e[2 * j + 1]) << 16;
            } else {
#pragma unroll
                for (int j = 0; j < G; ++j)
                    if (uint32_t(j) < keep) at[j] = row[p].e[j];
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // one wave's LDS accesses are served in order: nothing to wait for
    const uint32_t last_c = c0 + n - 1, rows_ended = last_c / per_row + (last_c % per_row == per_row - 1 ? 1 : 0);
    const uint32_t end = shift + n * G - rows_ended * padding;
    uint16_t* to = weight + (begin - shift);
    const uint32_t whole_begin = (shift + 7) / 8, whole_end = end / 8;   // pieces
    for (uint32_t t = whole_begin + lane; t < whole_end; t += 64)
        __builtin_nontemporal_store(reinterpret_cast<const u32x4*>(out)[t], reinterpret_cast<u32x4*>(to) + t);
    // the ends, lanes 0 .. 7 and 8 .. 15; one piece may be both
    const uint32_t e = lane < 8 ? lane : end / 8 * 8 + lane - 8;
    const bool mine = lane < 8 ? e >= shift && e < min(8 * whole_begin, end) : lane < 16 && e >= max(8 * whole_begin, shift) && e < end;
    if (mine) to[e] = out[e];
}

// g = 8 with no padding and 16-bit elements: whole rows as one piece
__global__ __launch_bounds__(kThreads) void layer_weight_vec_kernel(const u32x4* __restrict__ codebook, uint32_t K, const uint16_t* __restrict__ codes,
                                                                    uint64_t num_codes, u32x4* __restrict__ weight)
{
    const uint64_t v = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (v >= num_codes) return;
    const uint32_t k = min(uint32_t(codes[v]), K - 1);
    __builtin_nontemporal_store(codebook[k], &weight[v]);
}

// g = 4, no padding, 16-bit elements, by parts of the codebook. What bounds the general kernel is a line from L2 per code. Here a
// workgroup (16 waves, one per compute unit) holds up to 38 codes and their rows per thread in registers; the parts of the codebook pass
// through its LDS one after the other, every thread picks the rows that are there, and whole rows leave at the end, past the caches (plain
// stores of more than the memory-side cache holds run at 2 TB/s). Bound: the parts' way into LDS (512 KB a workgroup and round at K = 65536) and
// the lookups, 10 us of 35 each at 4096 x 11008, then the stores.
// Tried: a workgroup per part that stores the 8 bytes of each of its codes (L2 puts the lines together): 47 us there, as the general kernel.
constexpr int kPartThreads = 1024;
constexpr uint32_t kPartRows = 160 * 1024 / 8 - 16;
constexpr int kLeastPairs = 4, kMostPairs = 19;   // of codes of a thread: 76 registers of rows, 19 of codes; at 22 it spills, and one round for two gains nothing
typedef uint32_t u32_2 __attribute__((aligned(2)));

template <int PAIRS>
__global__ __launch_bounds__(kPartThreads, 4) void layer_weight_parts_kernel(const u32x4* __restrict__ codebook, uint32_t K, const uint16_t* __restrict__ codes,
                                                                          uint64_t num_codes, u32x4* __restrict__ weight, uint32_t parts,
                                                                          uint32_t part_rows, uint64_t per_share)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u32x2* table = reinterpret_cast<const u32x2*>(smem);
    const uint32_t lane = threadIdx.x & 63, wave = uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
    const uint64_t begin = blockIdx.x * per_share, end = min(begin + per_share, num_codes);   // per_share and num_codes are even
    const u16x2 last = {uint16_t(K - 1), uint16_t(K - 1)};
    constexpr uint64_t round = PAIRS * 2 * kPartThreads;
    for (uint64_t at = begin; at < end; at += round) {
        const uint32_t n = uint32_t(min(end - at, uint64_t(round)));
        uint32_t code[PAIRS];
        u32x4 row[PAIRS];
#pragma unroll
        for (int q = 0; q < PAIRS; ++q) {
            const uint32_t i = min(2 * (q * kPartThreads + threadIdx.x), n - 2);   // past the end the last pair again
            const uint32_t pair = *reinterpret_cast<const u32_2*>(codes + at + i);
            code[q] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, pair), last));   // never outside the codebook
        }
        for (uint32_t part = 0; part < parts; ++part) {
            const uint32_t low = part * part_rows, rows = min(part_rows, K - low);   // part_rows is even
            // into LDS, each workgroup from another place on; a row of zeros behind
            const u32x4* from = codebook + low / 2;
            const uint32_t pieces = rows / 2, chunks = (pieces + 63) / 64, turn = (blockIdx.x / 8 * 7u + blockIdx.x) % chunks;   // of 1 KB
            if (part > 0 || at > begin) __syncthreads();
            for (uint32_t i = wave; i < chunks; i += kPartThreads / 64) {
                uint32_t chunk = i + turn;
                chunk = chunk >= chunks ? chunk - chunks : chunk;
                if (chunk * 64 + lane < pieces)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(from + chunk * 64 + lane),
                                                     (__attribute__((address_space(3))) void*)(smem + chunk * 1024), 16, 0, 0);
            }
            if (threadIdx.x == 0) {
                if (rows % 2 != 0) reinterpret_cast<u32x2*>(smem)[rows - 1] = reinterpret_cast<const u32x2*>(from)[rows - 1];
                reinterpret_cast<u32x2*>(smem)[rows] = u32x2{0u, 0u};
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // what this wave requested has landed: the others read it behind the barrier
            __syncthreads();
            auto look = [&](auto first) {
#pragma unroll
                for (int q = 0; q < PAIRS; ++q) {
                    asm volatile("" : "+v"(code[q]));   // its halves are not kept over the parts: registers
                    const u32x2 x = table[min((code[q] & 0xffffu) - low, rows)], y = table[min((code[q] >> 16) - low, rows)];
                    const u32x4 here = {x[0], x[1], y[0], y[1]};
                    row[q] = decltype(first)::value ? here : row[q] | here;
                    if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // few reads at a time: registers
                }
            };
            if (part == 0) look(std::true_type{});
            else look(std::false_type{});
        }
        uint32_t thread = threadIdx.x;
        asm volatile("" : "+v"(thread));   // nor are the places of the loads
#pragma unroll
        for (int q = 0; q < PAIRS; ++q) {
            const uint32_t i = q * kPartThreads + thread;
            if (2 * i < n) __builtin_nontemporal_store(row[q], weight + at / 2 + i);
        }
    }
}

template <int PAIRS>
hipError_t launch_weight_parts(int pairs, uint32_t shares, const u32x4* codebook, uint32_t K, const uint16_t* codes, uint64_t num_codes, u32x4* weight,
                               uint32_t parts, uint32_t part_rows, uint64_t per_share, hipStream_t s)
{
    if constexpr (PAIRS <= kMostPairs) {
        if (pairs > PAIRS) return launch_weight_parts<PAIRS + 1>(pairs, shares, codebook, K, codes, num_codes, weight, parts, part_rows, per_share, s);
        if (const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&layer_weight_parts_kernel<PAIRS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, int(kPartRows + 16) * 8);
            e != hipSuccess)
            return e;
        hipLaunchKernelGGL(layer_weight_parts_kernel<PAIRS>, dim3(shares), dim3(kPartThreads), size_t(part_rows + 1) * 8, s, codebook, K, codes, num_codes,
                           weight, parts, part_rows, per_share);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

// us, general kernel / by parts, 16-bit, g = 4. K = 65536 (4 parts): 1024 x 8192 11.1 / 11.4, 2048 x 11008 25.8 / 19.4, 4096 x 11008 47 / 35, 8192 x 14336
// 117 / 72. K = 50000 (3): 10.5 / 9.2, 25 / 17, 47 / 30, 116 / 64. K = 20000 (1): 1024 x 4096 6.1 / 6.4, 1024 x 8192 9.7 / 6.4, 4096 x 11008 42 / 20; K = 4096
// 25.5 / 20, and where the general kernel's rows lie in L1, 21 / 20 at K = 2000 and 6.7 / 6.9 for 1024 x 8192.
bool weight_parts_pay(uint32_t K, uint64_t num_codes) { return K >= 4096 && num_codes >= (K > 3 * kPartRows ? 3u << 20 : 1u << 21); }

template <int G>
hipError_t launch_weight(uint32_t units, const void* codebook, uint32_t K, const uint16_t* codes, uint64_t num_codes, uint32_t per_row, uint32_t padding,
                         void* weight, hipStream_t s)
{
    if constexpr (G <= 32) {
        if (units != G) return launch_weight<(G < 16 ? G + 1 : G + 2)>(units, codebook, K, codes, num_codes, per_row, padding, weight, s);
        constexpr uint32_t kCodes = kThreads * kCodesPerLane<G>;
        const bool even = G % 2 == 0 && padding % 2 == 0;   // every row of the codebook and of the weight begins at 4 bytes
        const auto kernel = even || G > 16 ? layer_weight_kernel<G, G % 2 == 0> : layer_weight_kernel<(G <= 16 ? G : 16), false>;
        hipLaunchKernelGGL(kernel, dim3(uint32_t((num_codes + kCodes - 1) / kCodes)), dim3(kThreads), 0, s, static_cast<const uint16_t*>(codebook), K,
                           codes, num_codes, per_row, padding, static_cast<uint16_t*>(weight));
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

hipError_t launch_layer_weight(const void* codebook, int dtype, uint32_t K, uint32_t g, const uint16_t* codes,
                               uint32_t in_features, uint32_t out_features, void* weight, hipStream_t s)
{
    const uint32_t per_row = (out_features + g - 1) / g;
    const uint64_t num_codes = uint64_t(in_features) * per_row;
    const dim3 grid(uint32_t((num_codes + kThreads - 1) / kThreads));
    const bool whole = out_features % g == 0;
    if (dtype != 0 && whole && g == 8) {   // 28.2 us at 4096 x 11008, K = 65536, where the general kernel takes 30.5
        hipLaunchKernelGGL(layer_weight_vec_kernel, grid, dim3(kThreads), 0, s, static_cast<const u32x4*>(codebook), K, codes, num_codes,
                           static_cast<u32x4*>(weight));
        return hipGetLastError();
    }
    if (dtype != 0 && whole && g == 4 && num_codes % 2 == 0 && weight_parts_pay(K, num_codes)) {
        const uint32_t parts = (K + kPartRows - 1) / kPartRows, part_rows = ((K + parts - 1) / parts + 1) & ~1u;
        const uint64_t per_share = (num_codes + 511) / 512 * 2;
        const uint32_t shares = uint32_t((num_codes + per_share - 1) / per_share);
        constexpr uint64_t kUnit = 2 * kPartThreads;
        // rounds of equal length, each length an instance of the kernel: with every third one 8192x10240 takes 57.9 us instead of 55.4, 2048x11008 18.4 instead of
        // 17.9 (K = 65536), others 0 to 2 % more
        const uint64_t rounds = (per_share + kMostPairs * kUnit - 1) / (kMostPairs * kUnit);
        const int pairs = int((per_share + rounds * kUnit - 1) / (rounds * kUnit));
        return launch_weight_parts<kLeastPairs>(pairs, shares, static_cast<const u32x4*>(codebook), K, codes, num_codes, static_cast<u32x4*>(weight), parts,
                                                part_rows, per_share, s);
    }
    const uint32_t unit = dtype == 0 ? 2 : 1;
    return launch_weight<1>(g * unit, codebook, K, codes, num_codes, per_row, (per_row * g - out_features) * unit, weight, s);
}

// ---- codebook gradient, first step: the gradient of the weight as fp32 vectors in the layout of the
// clustering (padding columns and padding components zero), and the codes widened for the M-step kernels.
template <int DT>
__global__ __launch_bounds__(kThreads) void layer_grad_vectors_kernel(const void* __restrict__ grad, uint32_t out_features,
                                                                      uint32_t width, uint32_t g, uint32_t d_pad,
                                                                      const uint16_t* __restrict__ codes,
                                                                      uint64_t num_codes, float* __restrict__ vectors,
                                                                      uint32_t* __restrict__ idx)
{
    const uint64_t t = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
    if (t >= num_codes * d_pad) return;
    const uint64_t v = t / d_pad;
    const uint32_t j = uint32_t(t % d_pad);
    float val = 0.0f;
    if (j < g) {
        const uint64_t flat = v * g + j;  // position in the padded transpose
        const uint64_t r = flat / width;
        const uint32_t c = uint32_t(flat % width);
        if (c < out_features) val = load_as_f32<DT>(grad, r * out_features + c);
    }
    vectors[t] = val;
    if (j == 0) idx[v] = codes[v];
}

hipError_t launch_layer_grad_vectors(const void* grad, int dtype, uint32_t in_features, uint32_t out_features,
                                     uint32_t g, uint32_t d_pad, const uint16_t* codes, uint64_t num_codes, float* vectors,
                                     uint32_t* idx, hipStream_t s)
{
    (void)in_features;
    const uint32_t width = (out_features + g - 1) / g * g;
    const uint64_t n = num_codes * d_pad;
    const dim3 grid(uint32_t((n + kThreads - 1) / kThreads));
    switch (dtype) {
        case 0: hipLaunchKernelGGL(layer_grad_vectors_kernel<0>, grid, dim3(kThreads), 0, s, grad, out_features, width, g, d_pad, codes, num_codes, vectors, idx); break;
        case 1: hipLaunchKernelGGL(layer_grad_vectors_kernel<1>, grid, dim3(kThreads), 0, s, grad, out_features, width, g, d_pad, codes, num_codes, vectors, idx); break;
        case 2: hipLaunchKernelGGL(layer_grad_vectors_kernel<2>, grid, dim3(kThreads), 0, s, grad, out_features, width, g, d_pad, codes, num_codes, vectors, idx); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cc
