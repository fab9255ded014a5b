// Forward pass of the compressed linear layer for few rows of x (decode-time M <= 4), g = 4, 16-bit elements: the codebook
// goes through LDS in parts of 16384 rows (128 KB).
//
// What bounds a decoding row is one random codebook row per code. From L2 these come at about 3 clocks each per compute
// unit, whatever the kernel does; from LDS a wave gets 64 of them in about 10. So a workgroup - one per compute unit,
// 16 waves - keeps the codes of its columns in registers and lets the parts of the codebook come by: every code is looked
// at in every part and meets a row of zeros in all but the one it falls into. That is 12 to 14 vector instructions per
// code and part (what bounds large layers); the parts, prefetched into registers while the one before is worked on, cost
// about 2.8 us each (what bounds small ones).
// A workgroup owns whole columns, all in-features of them: no partial sums in memory, no second launch, sums in a fixed
// order. Thread t takes column t % C and every R-th pair of in-features from pair t / C on.
// Measured, M = 1, K = 65536: 4096 x 4096 40.0 -> 21.5 us a call, 4096 x 11008 57.8 -> 38.3, 8192 x 28672 332 -> 126.
#include <algorithm>

#include "common.h"
#include "half_types.h"

namespace cc {

namespace {

constexpr int kThreads = 1024;
constexpr uint32_t kPart = 16384;          // codebook rows in LDS
template <int MB>
constexpr int kPairs = MB == 1 ? 36 : (MB == 2 ? 28 : 20);   // pairs of codes a thread holds
constexpr uint32_t kXBytes = 28 * 1024;    // x values in LDS

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ float hi_to_f32(uint32_t v)   // high 16 bits
{
    if constexpr (DT == 1) return float(__builtin_bit_cast(_Float16, uint16_t(v >> 16)));
    else return __uint_as_float(v & 0xffff0000u);
}

template <int DT, int MB>
__global__ __launch_bounds__(kThreads) void layer_forward_book_kernel(const uint16_t* __restrict__ x, uint32_t M,
                                                                      const uint16_t* __restrict__ codebook, uint32_t K,
                                                                      const uint16_t* __restrict__ codes, uint32_t per_row,
                                                                      uint32_t in_features, uint32_t out_features,
                                                                      const uint16_t* __restrict__ bias, uint16_t* __restrict__ y,
                                                                      uint32_t C, uint32_t chunk)
{
    constexpr int U = MB == 4 ? 2 : 4;                      // pairs of codes worked on together
    constexpr int kPieces = kPart * 8 / 16 / kThreads;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint2* book = reinterpret_cast<uint2*>(smem);                              // [kPart + 1], the last row zero
    uint32_t* xs = reinterpret_cast<uint32_t*>(smem + (kPart + 1) * 8);        // [chunk / 2][MB], two in-features each
    // slots: R of them per column, each with two neighbouring in-features at a time
    const uint32_t R = kThreads / C;
    // consecutive workgroup ids go to different XCDs: XCD q takes the q-th share of the columns (lines of codes are shared)
    const uint32_t job = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (job * C >= per_row) return;
    const uint32_t col = threadIdx.x % C, slot = threadIdx.x / C;   // slot >= R: idle, reads what slot R - 1 reads
    const uint32_t cn = min(job * C + col, per_row - 1), pair0 = min(slot, R - 1);
    const uint32_t parts = (K + kPart - 1) / kPart;
    if (threadIdx.x == 0) book[kPart] = make_uint2(0u, 0u);

    // part of the codebook on its way; each workgroup starts at another place of it, so that they do not all ask the same
    // cache channels at once
    u32x4 next[kPieces];
    auto place = [&](int i) { return threadIdx.x + ((uint32_t(i) + job) % kPieces) * kThreads; };   // in 16 bytes
    auto request = [&](uint32_t q) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const uint32_t r = q * kPart + 2 * place(i);   // rows r, r + 1
            next[i] = u32x4{0u, 0u, 0u, 0u};
            if (r + 1 < K) {
                next[i] = *reinterpret_cast<const u32x4*>(codebook + size_t(r) * 4);
            } else if (r < K) {
                const uint2 last = *reinterpret_cast<const uint2*>(codebook + size_t(r) * 4);
                next[i] = u32x4{last.x, last.y, 0u, 0u};
            }
        }
    };
    request(0);
    float acc[MB][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j] = 0.0f;

    for (uint32_t k0 = 0; k0 < in_features; k0 += chunk) {
        const uint32_t rows = min(chunk, in_features - k0), pairs = rows / 2;   // in-features come in eights
        uint32_t word[kPairs<MB>];   // two codes each
        uint32_t first = pair0, step = R;
        asm volatile("" : "+v"(first), "+s"(step));   // as below
#pragma unroll
        for (int i0 = 0; i0 < kPairs<MB>; i0 += U) {
            if (i0 * step >= pairs) continue;   // uniform
            uint32_t c[U][2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t r = k0 + 2 * min((i0 + u) * step + first, pairs - 1);
                c[u][0] = codes[size_t(r) * per_row + cn];
                c[u][1] = codes[size_t(r + 1) * per_row + cn];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) word[i0 + u] = min(c[u][0], K - 1) | (min(c[u][1], K - 1) << 16);  // never outside the codebook
            __builtin_amdgcn_sched_barrier(0);   // a batch of loads at a time
        }
        __syncthreads();   // the chunk before has been worked on
        bool odd = false;   // Inf or NaN among this thread's share of x
        for (uint32_t i = threadIdx.x; i < pairs; i += kThreads) {
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const uint32_t v = m < int(M) ? reinterpret_cast<const uint32_t*>(x + size_t(m) * in_features + k0)[i] : 0u;
                constexpr uint32_t kExp = DT == 1 ? 0x7c00u : 0x7f80u;
                odd = odd || (v & kExp) == kExp || ((v >> 16) & kExp) == kExp;
                xs[i * MB + m] = v;
            }
        }
        const bool finite = __syncthreads_or(odd) == 0;
        for (uint32_t q = 0; q < parts; ++q) {
            if (q > 0) __syncthreads();   // the part before has been worked on
#pragma unroll
            for (int i = 0; i < kPieces; ++i) *reinterpret_cast<u32x4*>(smem + 16 * place(i)) = next[i];
            __syncthreads();
            if (parts > 1 || k0 + chunk < in_features) request(q + 1 < parts ? q + 1 : 0u);
            const uint32_t shift = 0u - q * kPart * 8;
            // hide from the compiler that codes and places are those of the part before: it would keep everything it can
            // derive from them in registers that are not there
            asm volatile("" : "+v"(first), "+s"(step));
#pragma unroll
            for (int i = 0; i < kPairs<MB>; ++i) asm volatile("" : "+v"(word[i]));
#pragma unroll
            for (int i0 = 0; i0 < kPairs<MB>; i0 += U) {
                if (i0 * step >= pairs) continue;   // uniform
                uint2 row[U][2];
                uint32_t at[U][2], xw[U][MB];
                const bool whole = (i0 + U) * step <= pairs;   // uniform
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t w = word[i0 + u];
                    uint32_t r = (i0 + u) * step + first;
                    at[u][0] = min(((w & 0xffffu) << 3) + shift, kPart * 8);   // the zero row for codes of other parts
                    at[u][1] = min(((w >> 16) << 3) + shift, kPart * 8);
                    if (!whole) {
                        at[u][0] = r < pairs ? at[u][0] : kPart * 8;
                        at[u][1] = r < pairs ? at[u][1] : kPart * 8;
                        r = min(r, pairs - 1);
                    }
                    row[u][0] = *reinterpret_cast<const uint2*>(smem + at[u][0]);
                    row[u][1] = *reinterpret_cast<const uint2*>(smem + at[u][1]);
#pragma unroll
                    for (int m = 0; m < MB; ++m) xw[u][m] = xs[r * MB + m];
                }
                if (!finite) {   // zero times zero where the code lies in another part
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int m = 0; m < MB; ++m)
                            xw[u][m] = (at[u][0] != kPart * 8 ? xw[u][m] & 0xffffu : 0u) | (at[u][1] != kPart * 8 ? xw[u][m] & 0xffff0000u : 0u);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const uint2 w = row[u][e];
                        const float f[4] = {to_f32<DT>(uint16_t(w.x)), hi_to_f32<DT>(w.x), to_f32<DT>(uint16_t(w.y)), hi_to_f32<DT>(w.y)};
#pragma unroll
                        for (int m = 0; m < MB; ++m) {
                            const float xf = e == 0 ? to_f32<DT>(uint16_t(xw[u][m])) : hi_to_f32<DT>(xw[u][m]);
#pragma unroll
                            for (int j = 0; j < 4; ++j) acc[m][j] = __builtin_fmaf(xf, f[j], acc[m][j]);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // sums over the R threads of a column: S of 4 C outputs each add every S-th, then one adds those
    const uint32_t outs = 4 * C, S = kThreads / outs;
    float* red = reinterpret_cast<float*>(smem);           // [kThreads][4]
    float* red2 = red + kThreads * 4;                      // [S][outs]
    const uint32_t o = threadIdx.x % outs, part = threadIdx.x / outs;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        if (m >= int(M)) break;
        __syncthreads();
        *reinterpret_cast<float4*>(red + 4 * threadIdx.x) = make_float4(acc[m][0], acc[m][1], acc[m][2], acc[m][3]);
        __syncthreads();
        if (part < S) {
            float v = 0.0f;
            for (uint32_t r = part; r < R; r += S) v += red[(r * C + o / 4) * 4 + o % 4];
            red2[part * outs + o] = v;
        }
        __syncthreads();
        const uint32_t n = job * outs + threadIdx.x;
        if (threadIdx.x < outs && n < out_features) {
            float v = 0.0f;
            for (uint32_t p = 0; p < S; ++p) v += red2[p * outs + threadIdx.x];
            y[size_t(m) * out_features + n] = from_f32<DT>(bias ? v + to_f32<DT>(bias[n]) : v);
        }
    }
}

constexpr uint32_t kLds = (kPart + 1) * 8 + kXBytes;
static_assert(kThreads * 4 * 4 + kThreads * 4 <= kPart * 8, "sums fit where the codebook was");

// Code columns per workgroup: one workgroup per compute unit
uint32_t book_columns(uint32_t per_row) { return (per_row + 255) / 256; }

template <int DT, int MB>
hipError_t launch_t(const uint16_t* x, uint32_t M, const uint16_t* codebook, uint32_t K, const uint16_t* codes, uint32_t in_features,
                    uint32_t out_features, const uint16_t* bias, uint16_t* y, hipStream_t s)
{
    const uint32_t per_row = (out_features + 3) / 4, C = book_columns(per_row);
    const uint32_t chunk = std::min<uint32_t>({in_features, 2 * kPairs<MB> * (kThreads / C), kXBytes / (2 * MB)});
    const auto kernel = layer_forward_book_kernel<DT, MB>;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, int(kLds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((per_row + 8 * C - 1) / (8 * C) * 8), dim3(kThreads), kLds, s, x, M, codebook, K, codes, per_row, in_features,
                       out_features, bias, y, C, chunk);
    return hipGetLastError();
}

}  // namespace

// The parts pay where there are enough codes for the time they take (2048 x 2048 with K = 65536, 16 codes per row: 18 against
// 14 us; 3072 x 3000, 35: 22.6 against 27.5), and with M = 3, 4 rows of x, whose values do not all fit beside a part, up
// to two parts (K = 32768, 8192 x 8192: 51 against 77 us; K = 65536, 4096 x 11008: 63 against 59).
bool layer_forward_book(uint64_t M, uint32_t g, uint32_t K, uint32_t in_features, uint32_t out_features)
{
    const uint64_t per_row = (uint64_t(out_features) + 3) / 4;
    return g == 4 && M <= (K <= 2 * kPart ? 4u : 2u) && K <= 65536 && per_row <= 256 * 256 &&
           uint64_t(in_features) * per_row >= 32ull * K;
}

hipError_t launch_layer_forward_book(const uint16_t* x, uint32_t M, const uint16_t* codebook, int dtype, uint32_t K,
                                     const uint16_t* codes, uint32_t in_features, uint32_t out_features, const uint16_t* bias,
                                     uint16_t* y, hipStream_t s)
{
#define CC_BOOK(DT, MB) launch_t<DT, MB>(x, M, codebook, K, codes, in_features, out_features, bias, y, s)
    if (dtype == 1) return M == 1 ? CC_BOOK(1, 1) : (M == 2 ? CC_BOOK(1, 2) : CC_BOOK(1, 4));
    if (dtype == 2) return M == 1 ? CC_BOOK(2, 1) : (M == 2 ? CC_BOOK(2, 2) : CC_BOOK(2, 4));
#undef CC_BOOK
    return hipErrorInvalidValue;
}

}  // namespace cc
