// Internal declarations shared by the translation units of libcluscomp (not part of the public ABI).
#pragma once
#include <type_traits>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace cc {

// bytes of the radix sort's histogram buffer for n elements (sort.hip)
size_t sort_hist_bytes(uint64_t n);
// per-workgroup cluster sums of a small problem (small_fit.hip); 0 where that form is not used
size_t small_partials_bytes(uint64_t N, uint32_t d, uint32_t K);
// E-step by cells (cells.hip): room for the entries of a cell's list
uint32_t cell_list_cap(uint32_t d);
// Operands of 32 centroids for the lists; d = 8: whole pairs of them
__host__ __device__ constexpr uint32_t list_tiles(uint32_t d, uint32_t K) { return d == 4 ? (K + 31) / 32 : (K + 63) / 64 * 2; }
constexpr uint32_t kCellItem = 192;       // vectors of one wave (d = 4)
struct CellHead {
    uint32_t start, members;   // the cell's vectors
    uint32_t n1, n2;           // list entries within r1, between r1 and r2 (more than there is room for: not all stored)
    float r1, r2;
    uint32_t tmax;             // largest t(x) of the last E-step, fp32 bits
    uint32_t mids;             // d = 8: vectors of the cell between r1 and r2
};
// Whether a fit of this shape runs its E-steps by cells (d as padded; codes of 16 bits; the bounds do not prune at
// d = 16). The line lies where grouping, lists and the extra launches pay, with few iterations as with many. Times with
// windows alone over times by cells, random weights, after 3 / 5 / 20 iterations:
//   d = 4: (N, K) = (1.6 M, 4096) 1.01 / 1.01 / 1.2, (1.6 M, 65500) 1.01 / 1.06 / 1.2, (2 M, 20000) 1.04 / 1.13 / 1.3,
//     (3.5 M, 65500) 1.1 / 1.2 / 1.5, (11 M, 65536, 20) 1.3; one side below: (1.06 M, 4096) 1.01 / 0.91 / 1.1
//   d = 8: (1.6 M, 1100) 1.00 / 1.12 / 1.4, (1.6 M, 12000) 1.15 / 1.23 / 1.5, (1.6 M, 65500) 1.29 / 1.40 / 1.7; and below:
//     (0.8 M, 12000) 0.93 / 0.96 / 1.0
// Rows of differing scales (0.3 in the logarithm) move both sides: (0.8 M, 12000) 0.76 / 0.79 / 0.81 after 10,
// (1.1 M, 65500) 0.90 / 0.94 / 1.02, but (1.6 M, 65500) 1.03 / 1.10 / 1.19 and (1.6 M, 12000) 0.96 / 1.03 / 1.11.
inline bool cells_possible(uint64_t N, uint32_t d, uint32_t K)
{
    return d <= 8 && K >= 1024 && K <= 65536 && N >= 24ull * K && N >= (3u << 19) && N < (1ull << 31);
}

constexpr uint32_t kMaxK = 1u << 24;

// Device time of the library's own kernels, for callers that ask for it (cc_profile in the public header): a pool
// of HIP events created once; a scope records one event before and one after the launches it brackets, on the
// stream of the call. Slots follow cc_profile_slot. A NULL profile, a slot outside the caller's mask or a full pool
// turns a scope into a no-op.
struct Profile;
struct ProfileScope {
    ProfileScope(Profile* p, int slot, hipStream_t s);
    ~ProfileScope();
    ProfileScope(const ProfileScope&) = delete;
    ProfileScope& operator=(const ProfileScope&) = delete;
    Profile* p_;
    hipStream_t s_;
    int record_;
};
enum ProfileSlot : int { kProfEstepF16 = 0, kProfEstepF32 = 1, kProfEstepDirect = 2, kProfRefine = 3, kProfMstep = 4,
                         kProfOrder = 5, kProfSlots = 6 };

// Device-side bookkeeping at the start of the workspace (one 256-byte slot).
struct WsHeader {
    uint32_t absmax_bits;      // max over all inputs of the fp32 bit pattern of |x|
    uint32_t refine_count;     // length of the refine list written by the last matrix-core assign
    uint32_t x_not_f16;        // != 0: some |x| >= 2^15, or some |x| >= 2^-14 is not an fp16 number
    uint32_t cmax_bits;        // max over the current codebook of the fp32 bit pattern of |c|
    unsigned long long refined_vectors;
    unsigned long long skipped_vectors;
    unsigned long long assign_calls;
    unsigned long long window_stages;   // sum over 512-vector tiles of the codebook stages they had to score
    unsigned long long window_total;    // what that sum would be without pruning
    int32_t fixed_point_exp;
    uint32_t x_nonfinite;      // != 0: some input is Inf or NaN (the sums then skip such components)
    uint32_t far_count;        // E-step by cells: vectors that go through the windowed pass
    unsigned long long list_stages;     // E-steps by cells: the part of window_stages that was scored on lists
};

// Survives between calls on the same workspace (not touched by the per-call header reset): whether the
// codes of the previous E-step may serve as a hint, and where they lie. A hint never affects results, only
// how much of the codebook has to be scored.
enum Hint : int { kHintNone = 0, kHintByNorm = 1,   // in the norm order, in idx_sorted
                  kHintByCells = 2 };               // in the order of the cells, in idx_prev; that of norm rank r at cell_position[r]
struct WsPersist {
    unsigned long long magic;
    uint32_t N, d, K;
    uint32_t hint_valid;       // a Hint
};

// Carved view of the caller's workspace.
struct Workspace {
    uint32_t d;                // sub-vector length the kernels run at: the caller's, rounded up to 4, 8 or 16
    bool padded;               // the caller's length differs: the kernels see zero-padded copies
    float* xpad;               // [N*d]  padded vectors   (only if padded)
    float* cpad;               // [K*d]  padded centroids (only if padded)
    WsHeader* hdr;
    float* cnorm;              // [K]    ||c_k||^2
    long long* sums;           // [K*d]  fixed-point cluster sums
    uint32_t* counts;          // [K]
    double* partials;          // [partial_slots] per-block partial objective
    float* dmin;               // [N]    ||x_i - c_idx_i||^2 of the last assign (fp32, direct form)
    float* packed;             // codebook re-laid out as matrix-core operand tiles (+ ||c||^2)
    uint32_t* refine_list;     // [refine_cap] ids of vectors to re-decide in direct form
    // norm ordering for the pruned E-step
    WsPersist* persist;
    float* xsorted;            // [N*d]  the vectors in ascending-norm order
    uint32_t* idx_sorted;      // [N]    codes in that order (also the next call's hint)
    uint32_t* idx_prev;        // [N]    the previous iteration's code of every vector flagged in `changed` (incremental M-step)
    uint32_t* changed;         // [ceil(N/32)] one bit per ordered vector: its code may differ from the previous iteration's
    uint32_t* vperm;           // [N]    input position of the p-th vector in norm order
    uint32_t* vperm_tmp;       // [N]
    uint16_t* vkeys;           // [N]    norm keys (sorted after the sort)
    uint16_t* vkeys_tmp;       // [N]
    float* csorted;            // [K*d]  the centroids in ascending-norm order
    uint32_t* cperm;           // [K]    centroid index of the p-th centroid in norm order
    uint32_t* cperm_tmp;       // [K]    rank of each centroid among those of its key; most moved of each list (cells)
    uint32_t* cinv;            // [K]    position of centroid k in norm order (inverse of cperm)
    uint16_t* ckeys;           // [K]
    uint16_t* ckeys_tmp;       // [K]    moves (cells)
    uint32_t* key_starts;      // [65537] first norm-ordered centroid position with ordering key >= v
    uint32_t* sort_hist;       // [256 * sort blocks of the vectors]
    uint2* windows;            // [ceil(N/512)][kWinStride] window list (runs of codebook stages) per 512-vector tile
    // M-step by buckets (K <= kMaxBuckets * kBucketClusters)
    char* records;             // [2N] x (4d + 16) bytes: the vectors, each with its code, grouped by bucket
    uint32_t* bucket_hist;     // [blocks][buckets] members of each bucket in each block of kBucketChunk vectors
    uint32_t* bucket_gtot;     // [groups of kBucketGroup blocks][buckets]
    uint32_t* bucket_base;     // [buckets + 1] first record of each bucket
    bool bucket_ok;
    // E-step by cells
    uint32_t* cell_order;      // [N]    scratch of the grouping
    uint32_t* cell_rank;       // [N]    norm rank of the vector at each position
    uint32_t* cell_position;   // [N]    inverse of cell_rank: where the vector is far, and after the last grouping
    uint32_t* far_bits;        // [ceil(N/32)] by norm rank
    CellHead* cell_heads;      // [K]
    uint32_t* cell_hist;       // [65536] centroids per ordering key; zero between E-steps
    uint32_t* cell_cursor;     // [65536] next position of each key
    char* cell_flat;           // [K + 1] x 64 bytes: operand pieces of each centroid (d = 8)
    char* cell_operands;       // one matrix-core operand per 32 centroids (d = 4: ordered ones), for the lists
    uint16_t* cell_lists;      // [K][cap] centroids (d = 4: positions in their norm order; an E-step's own); NULL: no room for cells
    char* small_partials;      // small problems: one set of cluster sums per workgroup; NULL: no room
    uint32_t refine_cap;
    uint32_t partial_slots;
    uint32_t packed_tiles;     // number of 32-centroid tiles in `packed` (K rounded up, padded)
    size_t least;              // bytes without which no call runs: cells and the form for small problems go without
    size_t bytes;              // bytes for the fastest form of every call
};

constexpr uint32_t kTileCentroids = 32;   // centroids per matrix-core tile
constexpr uint32_t kGroupTiles = 2;       // tiles per tracking group of the matrix-core E-step
constexpr uint32_t kStageTilesMax = 8;    // the packed codebook is padded to whole LDS stages of this many tiles
constexpr uint32_t kStageTiles = 4;       // tiles per LDS stage of the matrix-core E-step kernels
constexpr uint32_t kWinQuad = kTileCentroids;  // window lists count runs in tiles = 32 positions; runs never share a stage
constexpr int kWinSlots = 32;             // most runs a window list can hold (one per norm shell)
// Vectors (neighbours in the norm order) that share one window list: what one workgroup of the windowed kernels
// scores (4 waves x 4 tiles of 32). Half of that gives tighter hulls but halves the work per staged codebook tile:
// measured 29.0 -> 31.9 ms per cfg3 fit.
constexpr uint32_t kWinTile = 512;
constexpr int kWinStride = kWinSlots + 1; // uint2 entries per 512-vector tile: (count, -), then the runs
// The far vectors of an E-step by cells have windows of their own: up to two octaves of shells, for those that share a workgroup.
constexpr int kFarWinSlots = 64;
constexpr int kFarWinStride = kFarWinSlots + 1;
constexpr uint32_t kBucketClusters = 64;  // M-step by buckets: consecutive clusters summed by one workgroup
constexpr uint32_t kMaxBuckets = 1024;    // so K <= 65536 for that path
constexpr uint32_t kBucketGroup = 64;     // blocks per group in the two-level scan of the bucket histogram
constexpr uint32_t kBucketChunk = 4096;   // vectors per workgroup in its counting and scatter passes
constexpr uint32_t kDeltaChunk = 16384;   // the same for an incremental pass, which looks only at the flagged vectors

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// E-step by cells: the far vectors lie at the start of the M-step's record buffer, which is free during an E-step
inline size_t far_bytes(uint64_t N, uint32_t d) { return align256(size_t(N) * d * 4) + 3 * align256(size_t(N) * 4); }

// Lays the arrays out behind `base` (which may be NULL for a pure size query); `have` bytes are there. Calls take a workspace
// of w.least bytes; the arrays of cells and of small problems share space with others where those are idle, and are left out
// (NULL) where `have` does not reach them.
inline Workspace carve(void* base, uint64_t N, uint32_t d_caller, uint32_t K, size_t have = ~size_t(0))
{
    Workspace w{};
    const uint32_t d = d_caller <= 4 ? 4u : (d_caller <= 8 ? 8u : 16u);
    w.d = d;
    w.padded = d != d_caller;
    char* p = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) { char* q = p ? p + off : nullptr; off += align256(bytes); return q; };
    static_assert(sizeof(WsHeader) <= 128 && sizeof(WsPersist) <= 128, "header slot layout");
    char* slot = take(256);
    w.hdr = reinterpret_cast<WsHeader*>(slot);
    w.persist = reinterpret_cast<WsPersist*>(slot ? slot + 128 : nullptr);
    w.cnorm = reinterpret_cast<float*>(take(size_t(K) * 4));
    w.sums = reinterpret_cast<long long*>(take(size_t(K) * d * 8));
    w.counts = reinterpret_cast<uint32_t*>(take(size_t(K) * 4));
    w.partial_slots = 1024;
    w.partials = reinterpret_cast<double*>(take(size_t(w.partial_slots) * 8));
    w.dmin = reinterpret_cast<float*>(take(size_t(N) * 4));
    if (w.padded) {
        w.xpad = reinterpret_cast<float*>(take(size_t(N) * d * 4));
        w.cpad = reinterpret_cast<float*>(take(size_t(K) * d * 4));
    }
    const size_t small_at = off;   // a small problem uses none of what follows
    const uint32_t stage = kTileCentroids * kStageTilesMax;
    w.packed_tiles = uint32_t((uint64_t(K) + stage - 1) / stage) * kStageTilesMax;
    // per centroid: fp32 operands + norm take 4(d+1) bytes; the fp16-split operands take up to 6d+4 bytes
    w.packed = reinterpret_cast<float*>(take(size_t(w.packed_tiles) * kTileCentroids * (6 * d + 16)));
    w.refine_cap = uint32_t(N / 8 + 4096);
    w.refine_list = reinterpret_cast<uint32_t*>(take(size_t(w.refine_cap) * 4));
    w.xsorted = reinterpret_cast<float*>(take(size_t(N) * d * 4));
    w.idx_sorted = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    w.idx_prev = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    w.changed = reinterpret_cast<uint32_t*>(take((size_t(N) / 32 + 1) * 4));
    w.vperm = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    w.vperm_tmp = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    w.vkeys = reinterpret_cast<uint16_t*>(take(size_t(N) * 2));
    w.vkeys_tmp = reinterpret_cast<uint16_t*>(take(size_t(N) * 2));
    w.csorted = reinterpret_cast<float*>(take(size_t(K) * d * 4));
    w.cperm = reinterpret_cast<uint32_t*>(take(size_t(K) * 4));
    w.cperm_tmp = reinterpret_cast<uint32_t*>(take(size_t(K) * 4));
    w.cinv = reinterpret_cast<uint32_t*>(take(size_t(K) * 4));
    w.ckeys = reinterpret_cast<uint16_t*>(take(size_t(K) * 2));
    w.ckeys_tmp = reinterpret_cast<uint16_t*>(take(size_t(K) * 2));
    w.key_starts = reinterpret_cast<uint32_t*>(take(size_t(65537) * 4));
    // histogram rows + 256 totals of the vectors' sort
    w.sort_hist = reinterpret_cast<uint32_t*>(take(sort_hist_bytes(N)));
    w.windows = reinterpret_cast<uint2*>(take((size_t(N) / kWinTile + 1) * kWinStride * 8));
    w.bucket_ok = K <= kMaxBuckets * kBucketClusters && N < (uint64_t(1) << 31);  // record positions are 32-bit
    if (w.bucket_ok) {
        const size_t buckets = (size_t(K) + kBucketClusters - 1) / kBucketClusters;
        w.bucket_hist = reinterpret_cast<uint32_t*>(take(buckets * (size_t(N) / kBucketChunk + 1) * 4));
        w.bucket_gtot = reinterpret_cast<uint32_t*>(take(buckets * (size_t(N) / kBucketChunk / kBucketGroup + 1) * 4));
        w.bucket_base = reinterpret_cast<uint32_t*>(take((buckets + 1) * 4));
        // 2N records: every vector with a trailer needs N, an incremental M-step 8 bytes a vector and its runs, the far vectors of a fit by cells and
        // the lists behind them what is there; the rest is room for more ranges of partial sums, of which small calls want many
        w.records = take(size_t(N) * 2 * (4 * d + 16));
    }
    w.least = w.bytes = off;
    if (cells_possible(N, d, K)) {
        // the lists live from the start of an E-step to its end: behind the far vectors, past the records' end if need be
        const size_t lists_at = off - align256(size_t(N) * 2 * (4 * d + 16)) + far_bytes(N, d);
        off = std::max(off, lists_at + align256(size_t(K) * cell_list_cap(d) * 2));
        w.cell_order = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
        w.cell_rank = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
        w.cell_position = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
        w.far_bits = reinterpret_cast<uint32_t*>(take((size_t(N) / 32 + 1) * 4));
        w.cell_heads = reinterpret_cast<CellHead*>(take(size_t(K) * sizeof(CellHead)));
        w.cell_hist = reinterpret_cast<uint32_t*>(take(65536 * 4));
        w.cell_cursor = reinterpret_cast<uint32_t*>(take(65536 * 4));
        w.cell_operands = take(size_t(list_tiles(d, K)) * 1024);
        w.cell_flat = take((size_t(K) + 1) * 64);
        w.cell_lists = have >= off && p ? reinterpret_cast<uint16_t*>(p + lists_at) : nullptr;
        w.bytes = off;
    }
    if (const size_t n = small_partials_bytes(N, d, K); n > 0) {
        const size_t end = small_at + align256(n);
        w.small_partials = have >= end && p ? p + small_at : nullptr;
        w.bytes = std::max(w.bytes, end);
    }
    return w;
}

// ---- launchers (each enqueues on `s` and returns the launch status) -------------------------------

// Direct-form E-step over all N vectors; dmin may be NULL. With gate != NULL the kernel does nothing
// unless *gate > gate_limit (used as the overflow path of the matrix-core E-step).
hipError_t launch_assign_direct(const float* X, uint32_t N, uint32_t d, const float* C, uint32_t K,
                                uint32_t* idx, float* dmin, const uint32_t* gate, uint32_t gate_limit,
                                hipStream_t s, Profile* profile = nullptr);

// Up to so many far vectors, 32, 64 and 128 of them share a workgroup: the first two give each of 256 compute units one, and 256 vectors
// (d = 8), whose operand loads and start values serve twice the products (27.3 instead of 31.8 ms of the 29 M fit), take four rounds
// to be worth it (2.8 M: 26.7 ms with 256 at any number, 25.5 with 128, 25.0 with this rule).
constexpr uint32_t kFarFew1 = 32 * 256, kFarFew2 = 64 * 256, kFarFew4 = 4 * 128 * 256;
// How many far vectors, neighbours in their list, share a window: those of a workgroup. 512 of them lie far apart, and so their windows held 64 % of the codebook
// at d = 8 (29 M, K = 65536) and 10 % at d = 4 (11 M) where those of 256 and 128 with room for two octaves of shells hold 38 % and 6 % (fits of
// 10 and 20 iterations 87.9 -> 81.2 and 12.98 -> 12.67 ms). 512 where the windows would need more room than there is.
// Inputs that are no fp16 numbers, on the fp32 matrix cores: 128 to a workgroup up to 2^17 of them, else 512, whose tiles come through LDS for four times the
// products. Fits of 10 iterations with 512 always / this rule, ms: (4 M, d = 4, K = 30000) 6.94 / 5.20, (16 M, 4, 65536) 19.7 / 17.6,
// (2 M, 8, 8192) 10.9 / 10.0; up to 2^19 of them (4 M, 8, 30000) 32.0 / 30.0, (16 M, 4, 65536) 17.6 / 17.3, but (16 M, 8, 40000) 121 / 123.
constexpr uint32_t kFarFewF32 = 1u << 17;
__device__ __forceinline__ uint32_t far_window_tile(const WsHeader* hdr, uint32_t d, uint32_t N)
{
    const uint32_t far = hdr->far_count;
    if (far > N / 2 || (hdr->x_not_f16 != 0 && far > kFarFewF32)) return kWinTile;
    if (hdr->x_not_f16 != 0) return 128u;
    return far <= kFarFew1 ? 32u : (far <= kFarFew2 ? 64u : (d == 4 || far <= kFarFew4 ? 128u : 256u));
}

// Which inputs a gated kernel runs for (decided on the device from WsHeader::x_not_f16).
// kGateNoHint (a flag on top of the three) additionally requires that the workspace holds no usable hint.
enum Gate : int { kGateIfF16 = 0, kGateIfNotF16 = 1, kGateAlways = 2, kGateNoHint = 4 };
__device__ __forceinline__ bool gate_open(const WsHeader* hdr, int gate)
{
    if (gate & kGateNoHint) {
        // the persistent state sits in the second half of the header's 256-byte slot
        const WsPersist* persist = reinterpret_cast<const WsPersist*>(reinterpret_cast<const char*>(hdr) + 128);
        if (persist->hint_valid != 0) return false;
    }
    const int base = gate & 3;
    return base == kGateAlways || (base == kGateIfF16) == (hdr->x_not_f16 == 0);
}

// One scoring pass of a matrix-core E-step kernel.
struct EStep {
    const float* X;             // vectors to score (input order, or the norm-ordered copy)
    uint32_t N;
    const float* pack_rows;     // centroid rows, where the packed codebook is not there already
    const float* rows;          // centroid rows in packed order, for the direct-form index recovery ...
    const uint32_t* row_ids;    // ... and the centroid index of each packed position (NULL = identity)
    uint32_t K;                 // rows in this codebook
    void* packed;               // operand tiles ...
    bool packed_already;        // ... which hold the codebook (the fp16 variant's always do)
    uint32_t packed_tiles;
    const uint2* windows;       // per 512-vector tile window list (NULL = whole codebook)
    uint32_t* idx;              // codes out
    bool accumulate;            // also add every vector to the cluster sums/counts of its provisional code
    bool hint_only;             // only write codes: no guard band, no distances, no refine list
    uint32_t* prev_out;         // with `changed`: where the code that idx held before goes, for every vector flagged there
    uint32_t* changed;          // NULL, or one bit per vector, set where the code differs from what idx held or is not final yet
    int gate;
    const uint32_t* n_dev;      // NULL, or where the device keeps the number of vectors, at most N (fp32 variant)
    const uint32_t* out_pos;    // NULL, or the position of each vector in idx and the distances (fp32 variant)
    Profile* profile;           // NULL, or where the scoring kernel's device time is recorded
};

// Matrix-core E-step, fp32 MFMA: packs the codebook and runs the scoring kernel (provisional idx,
// w.dmin and the refine list). Must be followed by launch_refine.
hipError_t launch_assign_mfma_f32(const EStep& e, uint32_t d, const Workspace& w, hipStream_t s);

// Matrix-core E-step for fp16-representable inputs: centroids split into three fp16 parts so that
// every product is exact, scored with the fp16 MFMA. Same outputs as the fp32 variant.
hipError_t launch_assign_mfma_f16(const EStep& e, uint32_t d, const Workspace& w, hipStream_t s);

// Small problems (small_fit.hip): E-step on the vector ALUs with the codebook and the cluster sums in LDS. One Lloyd
// iteration (C updated in place; idx, dmin and counts may be NULL), and the E-step alone.
bool small_problem(uint64_t N, uint32_t d, uint32_t K);
struct SmallCut {           // how the vectors of an iteration are dealt out
    uint32_t blocks, per_block;
    int32_t slices, lane;   // ways to split the codebook; vectors of a lane
    int32_t direct;         // every distance in direct form
};
SmallCut small_cut(uint32_t N, uint32_t d, uint32_t K, bool sums);   // sums: an iteration, else an E-step alone
hipError_t launch_small_iter(const float* X, uint32_t N, uint32_t d, float* C, uint32_t K, const SmallCut& cut, uint32_t* idx, float* dmin,
                             uint32_t* counts, const Workspace& w, hipStream_t s);
hipError_t launch_small_assign(const float* X, uint32_t N, uint32_t d, const float* C, uint32_t K, uint32_t* idx, float* dmin,
                               const Workspace& w, hipStream_t s);

// Norm ordering (pruned E-step): vectors once per call, centroids + per-tile windows once per E-step,
// and the codes back to input order afterwards.
// drop_hint = true forgets the codes a previous call left in the workspace (a fit starts cold).
hipError_t launch_sort_vectors(const float* X, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, bool drop_hint,
                               hipStream_t s);
// the centroids in the norm order (w.cperm, w.cinv, w.csorted, w.key_starts) and as operands (w.packed); after launch_sort_vectors
hipError_t launch_sort_centroids(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s);
// the centroids as operands where they are; zero_sums: the cluster sums are cleared too
hipError_t launch_pack_codebook(const float* C, uint32_t d, uint32_t K, const Workspace& w, bool zero_sums, hipStream_t s);
hipError_t launch_key_starts(const uint32_t* hist, uint32_t* starts, uint32_t* cursor, uint32_t K, hipStream_t s);
hipError_t launch_windows(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, float guess, hipStream_t s);
hipError_t launch_gather_rows(const float* in, const uint32_t* ids, uint32_t n, uint32_t d, float* out, hipStream_t s);
// by_cells: the vectors are grouped by cells
hipError_t launch_unpermute(uint32_t N, uint32_t* idx, const Workspace& w, bool by_cells, hipStream_t s);

// E-step by cells inside a fit (cells.hip), after a first E-step in the norm order. launch_cells_order groups the
// vectors by their codes (w.idx_sorted; swaps buffers of w; `first`: they lie in the norm order, and the codes change
// places with w.idx_prev: at the end a next call can put them into the norm order, kHintByCells; `last`: no grouping follows); launch_cells_centroids
// orders the current centroids and makes their operands and the lists of the cells; launch_cells_near decides the near
// vectors; launch_cells_compact leaves the far ones as a list of hdr->far_count entries in the arrays of far_view, with their windows
// (far_windows); launch_cells_far decides those (fp16 inputs) within their windows, up to the entries it leaves on the refine list.
hipError_t launch_cells_order(const float* X, const float* C, uint32_t N, uint32_t d, uint32_t d_caller, uint32_t K, Workspace& w,
                              bool first, bool last, hipStream_t s);
enum Radii : int { kRadiiStay, kRadiiFollow, kRadiiJump };   // towards the lists' target lengths: not, a step, all the way (same centroids)
hipError_t launch_cells_centroids(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, Radii radii, bool bounded, hipStream_t s);
hipError_t launch_cells_near(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, bool track, bool bounded, hipStream_t s);
hipError_t launch_cells_hints(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s);
hipError_t launch_cells_compact(const float* C, uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s);
hipError_t launch_cells_far(uint32_t N, uint32_t d, uint32_t K, const Workspace& w, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* dst, size_t n, uint32_t value, hipStream_t s);
struct FarView {
    float* x;        // [N * d] rows
    uint32_t* pos;   // [N]     positions
    uint32_t* idx;   // [N]     previous codes
    uint32_t* refine;  // [N]   those to be re-decided in direct form
};
// Work items of the near vectors, N / kCellItem + K (d = 4) or N / 64 + K of them: the cell (none: ~0), its first vector, the item's place among its vectors and how
// many these are, in one load. Where the sort by code had its second buffer (K <= N / 24: at most 0.92 N of 2 N bytes).
inline uint4* cell_items(const Workspace& w) { return reinterpret_cast<uint4*>(w.vkeys_tmp); }
// Windows of the far vectors, kFarWinStride entries for each far_window_tile of them: between groupings nobody uses that buffer of theirs
// (at most N / 256 + 257 windows of 520 bytes in 4 N of the 1.5 M vectors or more of such a fit).
inline uint2* far_windows(const Workspace& w) { return reinterpret_cast<uint2*>(w.vperm_tmp); }
inline FarView far_view(const Workspace& w, uint32_t N, uint32_t d)   // far_bytes(N, d) bytes
{
    FarView f;
    char* p = w.records;
    auto take = [&](size_t bytes) { char* q = p; p += align256(bytes); return q; };
    f.x = reinterpret_cast<float*>(take(size_t(N) * d * 4));
    f.pos = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    f.idx = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    f.refine = reinterpret_cast<uint32_t*>(take(size_t(N) * 4));
    return f;
}

// Re-decides the listed guard-band vectors over all K centroids in direct form; if the list
// overflowed, re-decides everything in direct form. With fix_sums = true the cluster sums/counts that
// the scoring kernel accumulated are corrected for every vector whose code changed (or rebuilt from
// scratch on overflow).
// With norm_ordered = true (X = w.xsorted, idx = w.idx_sorted) only each vector's window is searched and
// the codes are flagged as a usable hint for the next call.
// out_pos != NULL (norm_ordered only): where each of the listed vectors keeps its code and distance; the list then holds
// everything there is to refine (w.refine_cap vectors at most exist).
hipError_t launch_refine(const float* X, uint32_t N, uint32_t d, const float* C, uint32_t K, uint32_t* idx,
                         const Workspace& w, bool fix_sums, bool norm_ordered, hipStream_t s, const uint32_t* out_pos = nullptr);

// Scans the inputs: max |x| and whether every x is exactly representable in fp16.
hipError_t launch_scan_inputs(const float* X, uint64_t n_floats, WsHeader* hdr, hipStream_t s);

// *out = sum_i dmin[i] in fp64 with a fixed reduction shape.
hipError_t launch_reduce_dmin(const float* dmin, uint32_t N, double* partials, uint32_t partial_slots,
                              double* out, hipStream_t s);

// Header bookkeeping.
hipError_t launch_reset_header(WsHeader* hdr, hipStream_t s);
hipError_t launch_bump_assign_calls(WsHeader* hdr, hipStream_t s);

// M-step = zero the accumulators, accumulate, finalize. With gate != NULL a gated launch does nothing
// unless *gate > gate_limit (the refine-overflow path).
hipError_t launch_zero_accumulators(const Workspace& w, uint32_t K, uint32_t d, const uint32_t* gate,
                                    uint32_t gate_limit, hipStream_t s);
hipError_t launch_accumulate(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, uint32_t K,
                             const Workspace& w, const uint32_t* gate, uint32_t gate_limit, hipStream_t s);
// M-step by buckets (K <= 65536): counts, scatter into per-bucket records, LDS sums, means (and counts_out if
// not NULL) in one go. Codes >= K are skipped and counted in WsHeader::skipped_vectors. norm_order = true
// buckets the clusters by their position in the norm order left by launch_sort_centroids (w.cinv, w.cperm).
// mean = false writes the plain sums (0 for an empty cluster) instead of the means. The integer sums and the
// counts are left in w.sums / w.counts.
hipError_t launch_update_buckets(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, const float* prev,
                                 uint32_t K, float* out, uint32_t* counts_out, const Workspace& w, bool norm_order,
                                 bool mean, hipStream_t s);
// Incremental M-step (update_delta.hip): w.sums and w.counts hold the sums and counts of the codes w.idx_prev; only the vectors whose code
// differs are moved (bit-identical to a recomputation from idx). w.changed has one bit per vector: w.idx_prev is only read, and only
// needs to be valid, where the bit is set, and a vector whose bit is clear must have kept its code. Needs update_delta_applies.
bool update_delta_applies(uint32_t N, uint32_t d, uint32_t K, const Workspace& w);
hipError_t launch_update_delta(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, const float* prev, uint32_t K, float* out,
                               uint32_t* counts_out, const Workspace& w, hipStream_t s);
// M-step by cluster slices (update_sliced.hip): each chunk's codes sorted by slice, then one LDS accumulation per slice of the
// clusters; for K <= 65536 and not too few N. Same integer sums (left in w.sums / w.counts) and the same
// result bits as the other formulations. `out` may alias `prev`.
bool update_sliced_applies(uint32_t N, uint32_t d, uint32_t K, const Workspace& w);
// Whether all clusters fit one slice, i.e. the pass needs neither lists nor a second look at a code.
inline bool update_one_slice(uint32_t d, uint32_t K) { return K <= 16384 / d; }
// Sums (not means) of the sub-vectors of a 16-bit gradient [in][out_features] (dtype 1 = fp16, 2 = bf16) by 16-bit code, both read in
// place; out [K][g]. Header as after a reset and a scan of the rows.
bool sum_rows16_applies(uint32_t N, uint32_t d, uint32_t K, const Workspace& w);
hipError_t launch_sum_rows16(const void* grad, int dtype, uint32_t N, uint32_t out_features, uint32_t g, const uint16_t* codes, uint32_t K,
                             float* out, const Workspace& w, hipStream_t s);
// fresh: instead of launch_reset_header and launch_scan_inputs too
hipError_t launch_update_sliced(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, const float* prev, uint32_t K,
                                float* out, uint32_t* counts_out, const Workspace& w, bool mean, bool fresh, hipStream_t s);
// out[i][j] = j < d_in ? in[i][j] : 0 for rows of d_out >= d_in floats, and the reverse (drop the tail).
hipError_t launch_pad_rows(const float* in, uint32_t n, uint32_t d_in, uint32_t d_out, float* out, hipStream_t s);
hipError_t launch_unpad_rows(const float* in, uint32_t n, uint32_t d_in, uint32_t d_out, float* out, hipStream_t s);
hipError_t launch_finalize(const float* prev, float* out, uint32_t* counts_out, uint32_t K, uint32_t d, uint32_t N,
                           const Workspace& w, bool mean, hipStream_t s);
hipError_t launch_update(const float* X, uint32_t N, uint32_t d, const uint32_t* idx, const float* prev,
                         uint32_t K, float* out, uint32_t* counts_out, const Workspace& w, bool mean, hipStream_t s);

// ---- the compressed linear layer (layer.hip); dtype: 0 = fp32, 1 = fp16, 2 = bf16
hipError_t launch_layer_vectors(const void* weight, int dtype, uint32_t out_features, uint32_t in_features, uint32_t g,
                                float* vectors, hipStream_t s);
hipError_t launch_layer_pack_codebook(const float* centroids, size_t n, void* codebook, int dtype, hipStream_t s);
hipError_t launch_layer_pack_codes(const uint32_t* idx, uint64_t n, uint32_t K, uint16_t* codes, hipStream_t s);
hipError_t launch_layer_weight(const void* codebook, int dtype, uint32_t K, uint32_t g, const uint16_t* codes,
                               uint32_t in_features, uint32_t out_features, void* weight, hipStream_t s);
// y = x . W(codebook, codes) (+ bias); `partial` holds layer_forward_splits(...) * M * out_features floats if that
// count is above 1
uint32_t layer_forward_splits(uint64_t M, uint32_t in_features, uint32_t out_features);
// The sum of slices (times a scale if it is not NULL) + bias
hipError_t launch_layer_forward_reduce(const float* partial, uint32_t M, uint32_t out_features, uint32_t splits, const float* scale,
                                       const uint16_t* bias, uint16_t* y, int dtype, hipStream_t s);
// Rows of 4 .. 9 elements of 16, 8 or 4 bits, each column of the codebook through LDS (layer_forward_columns.hip). The workspace
// holds most_slices * M * out_features floats (none are needed if that is 1); what it has beyond the slices in use, up to
// layer_forward_columns_room bytes, holds copies of codebook and x in the layout of the kernel, without which it is slower.
// `scale` multiplies the sum if it is not NULL.
constexpr uint32_t kLeastColumns = 4, kMostColumns = 9;
inline bool layer_forward_columns(uint32_t g) { return g >= kLeastColumns && g <= kMostColumns; }
size_t layer_forward_columns_room(uint64_t M, uint32_t in_features);
hipError_t launch_layer_forward_columns(const void* x, uint32_t M, const void* book, int bits, const float* scale, uint32_t K, uint32_t g,
                                        const uint16_t* codes, uint32_t in_features, uint32_t out_features, const void* bias, void* y,
                                        int dtype, void* workspace, size_t workspace_bytes, uint32_t most_slices, hipStream_t s);
// The other lengths: rows gathered from memory tile by tile (layer_forward.hip)
hipError_t launch_layer_forward(const void* x, uint32_t M, const void* codebook, int dtype, uint32_t K, uint32_t g,
                                const uint16_t* codes, uint32_t in_features, uint32_t out_features, const void* bias,
                                void* y, float* partial, hipStream_t s);
// ---- codebook gradient from a prepared order of the codes (layer_grad_plan.hip); sort helpers from sort.hip
hipError_t launch_sort_u16(uint16_t* keys_a, uint32_t* ids_a, uint16_t* keys_b, uint32_t* ids_b, uint32_t n, uint32_t* hist,
                           hipStream_t s);
size_t layer_grad_plan_bytes(uint64_t num_codes, uint32_t K);
size_t layer_grad_plan_build_bytes(uint64_t num_codes);
size_t layer_grad_planned_bytes(uint64_t num_codes, uint32_t K, uint32_t g);
hipError_t launch_layer_grad_plan(const uint16_t* codes, uint32_t n, uint32_t K, void* plan, void* workspace, hipStream_t s);
hipError_t launch_layer_grad_planned(const void* grad, int dtype, uint32_t in_features, uint32_t out_features, uint32_t K,
                                     uint32_t g, uint32_t n, const void* plan, float* grad_codebook, void* workspace,
                                     hipStream_t s);
// ---- prefill-sized batches (layer_gemm.hip): W rebuilt into memory, then one dense product on the matrix cores
// Rows from which on a call brings room for the rebuilt weight: what a workspace is checked against. Which route a call takes is
// decided by rebuild_pays where the room allows both.
inline bool brings_rebuilt(uint64_t M, uint32_t g, uint32_t in_features, uint32_t out_features)
{
    const uint64_t weights = uint64_t(in_features) * out_features;
    if (g < 4) return M > 128;
    if (g != 4 && g != 8) return M > 384;
    return M > (weights >= (1ull << 25) ? 128u : (weights >= (1ull << 22) ? 256u : 384u));
}
inline bool brings_rebuilt_q(uint64_t M, uint32_t in_features, uint32_t out_features)
{
    const uint64_t weights = uint64_t(in_features) * out_features;
    if (weights < (1ull << 24)) return M > 64;
    if (weights >= (1ull << 25) && out_features >= 2 * uint64_t(in_features)) return M >= 16;
    return M > 32;
}
// From where on the rebuilt-weight route is the faster one: the others repeat their lookups for every 64 (by columns) or 128 rows
// of x, the rebuild takes the same for any number of rows. bf16, K = 65536, us, by columns / rebuilt + product:
//   g = 4, 4096 x 4096 at 256 rows 39 / 62, at 320 56 / 59, at 384 63 / 62; 4096 x 11008 at 256 90 / 91, at 320 117 / 107; 8192 x 16384 at 256
//   208 / 208, at 320 290 / 235; 8192 x 28672 at 128 226 / 317, at 192 367 / 320. g = 8: the same within 5 %. g = 6: 4096 x 11008 at 256 100 /
//   94, at 320 129 / 112; 2048 x 2048 at 384 26 / 37; 512 x 28672 at 256 60 / 53, at 320
//   77 / 44. g = 9: 4096 x 11008 97 / 96, 121 / 113; 8192 x 8192 at 128 91 / 119, at 160 141 / 123.
//   8 bits: g = 4, 4096 x 4096 at 384 63 / 61; 8192 x 28672 at 128 237 / 310, at 192 374 / 330.
//   4 bits (more arithmetic a lookup): 4096 x 4096 at 192 48 / 54, at 320 83 / 59; 8192 x 8192 at 128 91 / 111, at 192 153 / 121; g = 6, 2048 x
//   5000 at 128 30 / 38, at 192 49 / 40; g = 9, 4096 x 4096 at 128 47 / 48, at 192 82 / 57; 2048 x 2048 at 384 29 / 39.
// Row by row (up to 127 rows of smaller layers the query asks for the sums' room only: the rebuilt weight is taken where that holds it or the
// caller brings more): g = 12, 4096 x 4096 at 64 rows 39 / 48, at 96 59 / 50; g = 16, 4096 x 11008 62 / 85, 101 / 88; g = 2, 4096 x 4096 at 4 rows 40 / 36, at
// 48 46 / 42; integers: g = 12 at 4 rows 71 / 43, g = 3, 2048 x 2048 30 / 25, g = 12, 1024 x 4096 at 32 26 / 27, at 48 32 / 27.
inline bool rebuild_pays(uint64_t M, uint32_t g, int bits, uint32_t in_features, uint32_t out_features)
{
    const uint64_t weights = uint64_t(in_features) * out_features;
    if (!layer_forward_columns(g)) {
        if (bits != 16) return M > 32 || weights >= (1ull << 22);
        return M > (g < 4 ? 32u : 64u);
    }
    if (bits == 4) return M > (weights <= (1ull << 22) ? 384u : 128u);
    if (weights <= (1ull << 24) && out_features <= 8192) return M > 384;
    return M > (weights < (1ull << 26) || (weights <= (1ull << 27) && (g == 4 || g == 8)) ? 256u : 128u);
}
// layer_gemm.hip: the weight rebuilt in the register layout of the matrix cores' B operand (layer_weight_frag_bytes
// bytes; codebook of 16, 8 or 4 bits, the integers themselves in `dtype`; room: for the codebook as 16-bit numbers, needed for
// integers only, K * g * 2 bytes, and one more 16-byte piece per column to spare) and y [M][out] = x [M][in] . W
// (scale: device pointer or NULL, multiplies the finished sum; partial: layer_gemm_partial_bytes(...) bytes of fp32
// tiles for the tiles whose contraction is cut into slices)
size_t layer_gemm_partial_bytes(uint64_t M, uint32_t in_features, uint32_t out_features);
size_t layer_weight_frag_bytes(uint32_t in_features, uint32_t out_features);
hipError_t launch_layer_weight_frag(const void* codebook, int bits, int dtype, uint32_t K, uint32_t g, const uint16_t* codes, uint32_t in_features,
                                    uint32_t out_features, void* wf, void* room, size_t room_bytes, hipStream_t s);
hipError_t launch_layer_gemm(const void* x, uint32_t M, const void* wf, int dtype, uint32_t in_features, uint32_t out_features,
                             const float* scale, const void* bias, void* y, float* partial, uint32_t g, hipStream_t s);
// ---- uniformly quantised codebook (layer_quant.hip); bits = 8 or 4
hipError_t launch_codebook_quantize(const float* centroids, size_t n, int bits, void* qbook, float* scale,
                                    uint32_t* absmax_scratch, hipStream_t s);
hipError_t launch_layer_weight_q(const void* qbook, int bits, const float* scale, uint32_t K, uint32_t g,
                                 const uint16_t* codes, uint32_t in_features, uint32_t out_features, int dtype, void* weight,
                                 hipStream_t s);
uint32_t layer_forward_q_max_splits(uint64_t M, uint32_t in_features, uint32_t out_features);
hipError_t launch_layer_forward_q(const void* x, uint32_t M, const void* qbook, int bits, const float* scale, uint32_t K,
                                  uint32_t g, const uint16_t* codes, uint32_t in_features, uint32_t out_features,
                                  const void* bias, void* y, int dtype, float* partial, hipStream_t s);
// grad_weight [in, out] (dtype) -> fp32 vectors [num_codes][d_pad] (zero padding columns and components) and
// codes widened to 32 bits
hipError_t launch_layer_grad_vectors(const void* grad, int dtype, uint32_t in_features, uint32_t out_features,
                                     uint32_t g, uint32_t d_pad, const uint16_t* codes, uint64_t num_codes, float* vectors,
                                     uint32_t* idx, hipStream_t s);

// Diagnostic (probe.hip): the fp16 matrix-core instructions of the E-step on caller-chosen operands.
hipError_t launch_mfma_f16_probe16(const uint16_t* A, const uint16_t* B, const float* C, float* D, uint32_t tiles, uint32_t km,
                                   hipStream_t s);
hipError_t launch_mfma_f16_probe(const uint16_t* A, const uint16_t* B, const float* C, float* D, uint32_t tiles, uint32_t km,
                                 hipStream_t s);

// Reconstruction.
hipError_t launch_decode(const float* C, uint32_t K, uint32_t d, const uint32_t* idx, uint64_t N, float* out,
                         hipStream_t s);

hipError_t launch_copy_f32(const float* src, float* dst, size_t n, hipStream_t s);

// log2 of the centroid scale sigma: max|c| * sigma <= 2^15 and d * max|c|^2 * sigma <= 2^23
__device__ __forceinline__ int centroid_scale_log2(uint32_t cmax_bits, int d)
{
    if (cmax_bits == 0) return 0;
    const int ec = int(cmax_bits >> 23) - 127;  // max|c| < 2^(ec+1)
    const int ld = 32 - __clz(uint32_t(d - 1)); // d <= 2^ld
    int s = min(14 - ec, 21 - 2 * ec - ld);
    return max(-100, min(100, s));
}

// Fixed-point exponent e of the cluster sums: inputs satisfy |x| < 2^(EM+1) with EM the unbiased
// exponent of the largest magnitude M, and N < 2^LN, so |sum of N terms| < 2^(EM+1+e+LN) <= 2^62.
__device__ __forceinline__ int fixed_point_exp(uint32_t absmax_bits, uint32_t N)
{
    const int em = int(absmax_bits >> 23) - 127;   // -127 for zero/subnormal M: fine, just a large e
    const int ln = 32 - __clz(N);                  // N < 2^ln
    const int e = 62 - ln - (em + 1);
    return e < 100 ? e : 100;                      // keep ldexp away from fp64 overflow for tiny inputs
}

// A finite input as a fixed-point term of the cluster sums: x * 2^e rounded to the nearest integer, ties to even; e in -98 .. 100
// from fixed_point_exp, |x * 2^e| < 2^62. In fp32: the scaling and the split at 2^32 are exact (what 2^e x loses below the
// normal range is far below 1/2), and rounding a number of 24 bits is the same in any format. In fp64 the same takes ten
// instructions at a quarter of the rate: 8 M vectors of 16 numbers 140 us.
__device__ __forceinline__ long long fixed_point_finite(float x, int e)
{
    const float r = __builtin_rintf(x * __uint_as_float(uint32_t(e + 127) << 23)), a = __builtin_fabsf(r);
    const float hi = __builtin_truncf(a * 2.3283064365386963e-10f), lo = __builtin_fmaf(hi, -4294967296.0f, a);
    const long long v = static_cast<long long>((static_cast<unsigned long long>(uint32_t(hi)) << 32) | uint32_t(lo));
    const long long s = static_cast<int>(__float_as_uint(x)) >> 31;   // 0 or -1
    return (v ^ s) - s;
}

// The same terms where they have at most 30 bits above a common unit, 2^(k - e): x in that unit is a whole number t, and the term t * 2^k. Multiplication, fraction, conversion
// and two shifts, 18 clocks of a SIMD where fixed_point_finite takes 45. Non-finite numbers have no fraction of zero.
struct ShortTerms {
    float scale;   // 2^(e - k)
    uint32_t k;    // 1 .. 31
};
__device__ __forceinline__ ShortTerms short_terms(uint32_t absmax_bits, int e)   // |x| < 2^(em + 1): |t| < 2^29
{
    const int em = int(absmax_bits >> 23) - 127, s = max(min(28 - em, e - 1), e - 31);
    return {__uint_as_float(uint32_t(s + 127) << 23), uint32_t(e - s)};
}
// Bits other than zero: not a whole number
__device__ __forceinline__ uint32_t not_whole(float t) { return __float_as_uint(__builtin_amdgcn_fractf(t)); }
__device__ __forceinline__ unsigned long long short_term(float t, uint32_t k)
{
    const int v = int(t);
    return static_cast<unsigned long long>(uint32_t(v) << k) | static_cast<unsigned long long>(uint32_t(v >> (32 - k))) << 32;
}

// The same for any input: a non-finite one (which the input scan flags in WsHeader::x_nonfinite) contributes nothing.
__device__ __forceinline__ long long fixed_point_term(float x, int e)
{
    return (__float_as_uint(x) & 0x7f800000u) == 0x7f800000u ? 0ll : fixed_point_finite(x, e);
}

// One centroid (c = 0 and norm = +inf past K) at position `pos` of the fp32 variant's packed codebook.
template <int D>
__device__ __forceinline__ void put_f32_operand(float* packed, uint32_t pos, const float (&c)[D], float norm)
{
    constexpr uint32_t KS = D / 2, TF = 64 * KS + 32;
    const uint32_t q = pos & 31u, m = 4 * (q >> 4) + (q & 3u) + 8 * ((q & 15u) >> 2);   // the operand row whose results lie at q
    float* tile = packed + size_t(pos >> 5) * TF;
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h)
#pragma unroll
        for (uint32_t ks = 0; ks < KS; ++ks) tile[(32 * h + m) * KS + ks] = c[2 * ks + h];
    tile[64 * KS + q] = norm;
}

// Adds (sign = +1) or removes (sign = -1) one vector to/from cluster k's fixed-point sums and count.
// Integer adds commute, so the totals do not depend on the order in which these atomics land.
template <int D>
__device__ __forceinline__ void accumulate_vector(const float (&x)[D], uint32_t k, long long* sums, uint32_t* counts,
                                                  int e, int sign)
{
    unsigned long long* dst = reinterpret_cast<unsigned long long*>(sums + size_t(k) * D);
#pragma unroll
    for (int j = 0; j < D; ++j) {
        const long long f = fixed_point_term(x[j], e);
        if (f != 0) atomicAdd(dst + j, static_cast<unsigned long long>(sign > 0 ? f : -f));
    }
    atomicAdd(counts + k, sign > 0 ? 1u : 0xffffffffu);
}

// ||x - c||^2 in fp32, direct form: first square, then one fused multiply-add per further component.
// Every kernel that needs a distance uses this exact operation order, so that a vector decided by
// one kernel and re-decided by another sees identical values.
template <int D>
__device__ __forceinline__ float direct_sqdist(const float (&x)[D], const float (&c)[D])
{
    const float t0 = x[0] - c[0];
    float acc = t0 * t0;
#pragma unroll
    for (int j = 1; j < D; ++j) {
        const float t = x[j] - c[j];
        acc = __builtin_fmaf(t, t, acc);
    }
    return acc;
}

template <int D>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&v)[D]);

// The value of lane V of a lane's four neighbours
template <int V>
__device__ __forceinline__ uint32_t of_quad(uint32_t v) { return uint32_t(__builtin_amdgcn_mov_dpp(int(v), V * 0x55, 0xf, 0xf, true)); }
template <int V>
__device__ __forceinline__ float of_quad(float v) { return __uint_as_float(of_quad<V>(__float_as_uint(v))); }

// Index recovery of the matrix-core E-step: direct-form argmin over the codebook positions
// 32*(group*GT+g) + 16*h + r, g in [g_begin, g_end), r in [0, 16), of a winning group (the two lanes that
// share a vector split the group's tiles between them). `rows` holds the centroids in packed
// order (the codebook itself, or its norm-ordered copy together with `cperm`, which maps a position
// to the centroid index). Among exactly equal distances the lowest centroid index wins. Called by whole waves; neighbouring lanes have the same
// range of tiles. Four lanes take the candidates of their four vectors one vector after the other, four neighbouring rows at a time, which are one or two accesses
// of L1: with a lane to a vector every lane was one, and the windowed kernels, whose bound they were, made 0.9 per clock. Fits, ms: 29 M x 8, K = 65536
// 92.0 -> 88.9; 1.7 M x 8, K = 2000 6.56 -> 6.16; 3 M x 16, K = 20000, 3 iterations 16.4 -> 14.7; 11 M x 4, K = 65536 13.1 -> 12.9.
// ROWS of a lane at once: four, or at D = 16 two where four (64 registers) cost a kernel its fourth wave per SIMD or make it spill. Four / two, us, d = 16: fp32 numbers,
// 450000, K = 20000, 10 iterations 26062 / 24968, one iteration of 4.4 M, K = 8068 9138 / 8705; fp16 numbers, 90000, K = 2600, 10 1095 / 822; by windows 3 M, K = 20000, 3
// 16172 / 15732. Elsewhere two are slower: whole codebook, 4.2 M, K = 7872, 2 iterations 8623 / 9102.
template <int D, int GT, int ROWS>
__device__ __forceinline__ void recover_group(const float (&x)[D], const float* __restrict__ rows,
                                              const uint32_t* __restrict__ cperm, uint32_t K, uint32_t group, int h,
                                              int g_begin, int g_end, float& best_d, uint32_t& best_k)
{
    const uint32_t in_quad = threadIdx.x & 3u, first = 32 * GT * group + 16 * uint32_t(h);
    auto before = [&](uint32_t pos, uint32_t other) { return cperm != nullptr ? cperm[pos] < cperm[other] : pos < other; };   // among equal distances
    float best = INFINITY;
    uint32_t at = 0;
    auto vector = [&](auto of) {
        constexpr int V = decltype(of)::value;
        float y[D];
#pragma unroll
        for (int j = 0; j < D; ++j) y[j] = of_quad<V>(x[j]);
        const uint32_t k0 = of_quad<V>(first) + in_quad;
        float bd = INFINITY;
        uint32_t bpos = 0;
        for (int g = g_begin; g < g_end; ++g) {
#pragma unroll
            for (int u0 = 0; u0 < 4; u0 += ROWS) {
                float c[ROWS][D];
#pragma unroll
                for (int u = 0; u < ROWS; ++u) load_row<D>(rows + size_t(min(k0 + 32 * g + 4 * (u0 + u), K - 1)) * D, c[u]);
#pragma unroll
                for (int u = 0; u < ROWS; ++u) {
                    const uint32_t pos = k0 + 32 * g + 4 * (u0 + u);
                    const float dk = direct_sqdist<D>(y, c[u]);
                    if (pos < K) {
                        if (dk < bd) {
                            bd = dk;
                            bpos = pos;
                        } else if (dk == bd && before(pos, bpos)) {
                            bpos = pos;  // exact tie in norm order: keep the lower centroid index
                        }
                    }
                }
            }
        }
        auto meet = [&](auto ctrl) {   // with a neighbour's
            const float od = __uint_as_float(uint32_t(__builtin_amdgcn_mov_dpp(int(__float_as_uint(bd)), decltype(ctrl)::value, 0xf, 0xf, true)));
            const uint32_t opos = uint32_t(__builtin_amdgcn_mov_dpp(int(bpos), decltype(ctrl)::value, 0xf, 0xf, true));
            if (od < bd || (od == bd && opos != bpos && before(opos, bpos))) {
                bd = od;
                bpos = opos;
            }
        };
        meet(std::integral_constant<int, 0xb1>{});   // 1 0 3 2
        meet(std::integral_constant<int, 0x4e>{});   // 2 3 0 1
        best = in_quad == uint32_t(V) ? bd : best;
        at = in_quad == uint32_t(V) ? bpos : at;
    };
    vector(std::integral_constant<int, 0>{});
    vector(std::integral_constant<int, 1>{});
    vector(std::integral_constant<int, 2>{});
    vector(std::integral_constant<int, 3>{});
    best_d = best;
    best_k = (cperm != nullptr && best < INFINITY) ? cperm[min(at, K - 1)] : at;
}

template <int D>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&v)[D])
{
    const float4* s = reinterpret_cast<const float4*>(p);
#pragma unroll
    for (int q = 0; q < D / 4; ++q) {
        const float4 t = s[q];
        v[4 * q + 0] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
    }
}

}  // namespace cc
