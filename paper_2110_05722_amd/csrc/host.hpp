// Host-side helpers shared by the entry points: argument checks, dropout
// parameter packing, launch bookkeeping.  Nothing here touches device memory.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/lsq.h"
#include "device.hpp"

namespace lsq {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#define LSQ_REQUIRE(cond) do { if (!(cond)) return LSQ_INVALID_ARG; } while (0)
#define LSQ_ALIGNED(ptr) do { if ((ptr) && !::lsq::aligned16(ptr)) return LSQ_MISALIGNED; } while (0)

inline bool valid_dtype(int dt) { return dt == LSQ_F16 || dt == LSQ_BF16 || dt == LSQ_F32; }

// p must lie in [0, 1).  T16 = round(p * 65536) in double, clamped to [0, 65535].
inline bool make_dropout(float p, uint64_t seed, uint64_t offset, DropoutParams* d)
{
    if (!(p >= 0.0f) || !(p < 1.0f)) return false;
    double t = floor(static_cast<double>(p) * 65536.0 + 0.5);
    if (t < 0.0) t = 0.0;
    if (t > 65535.0) t = 65535.0;
    d->key0 = static_cast<uint32_t>(seed);
    d->key1 = static_cast<uint32_t>(seed >> 32);
    d->ctr2 = static_cast<uint32_t>(offset);
    d->ctr3 = static_cast<uint32_t>(offset >> 32);
    d->t16 = p == 0.0f ? 0u : static_cast<uint32_t>(t);
    d->on = p > 0.0f ? 1u : 0u;
    d->scale = static_cast<float>(1.0 / (1.0 - static_cast<double>(p)));
    return true;
}

inline lsq_status launch_status()
{
    return hipGetLastError() == hipSuccess ? LSQ_OK : LSQ_LAUNCH_FAILED;
}

// Zero fill by a kernel (a memset node inside a captured graph is avoided on purpose).
template <int = 0>
__global__ __launch_bounds__(256) void zero_f32_kernel(float* p, int64_t n)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

inline lsq_status zero_fill(float* p, int64_t n, hipStream_t s)
{
    if (n <= 0) return LSQ_OK;
    hipLaunchKernelGGL((zero_f32_kernel<0>), dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, p, n);
    return launch_status();
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The streamed inputs of a call are loaded past the caches (nontemporal) unless a tensor has 2 (heads, padding) or 4 to 16 MiB: what the kernel ahead has just written, or the same
// pass will read again, is then in the 256 MB Infinity Cache, and a load past the caches gives the line up.  It is a choice between states. us, 16 bits, past the caches
// and the change through them, in the order: passes over 100 MB that stay there / inputs written by the kernel ahead, outputs in far memory (its time counted too) / all in far
// memory.  Backward of bias+dropout+residual, 8 MB 9.0 - 1.0 / 12.3 + 0.9 / 9.5 + 0.6; of the feed-forward 11.2 - 0.3 / 16.1 + 0.8 / 11.7 + 0.8; padding restored, 8 MB 5.9 - 1.2 / 8.1 + 1.3 / 6.3
// + 0.5; head split backward, three of 8 MB 15.3 - 1.6 / 27.0 - 1.6 / 16.6 + 0.2.  Whole calls that take several of them gain: a captured layer of 128 x 32 tokens, hidden 512, 90.3 us with the
// forwards and the feed-forward past the caches, 85.5 like this (about half of that on inputs that no pass has read), the four calls of a sub-layer boundary of 8192 x 1024 51.7 and 50.2.
// Below, nothing gains in any state and a call from far memory loses: 1 MB 2.4 + 0.6 head merge backward, 5.6 + 0.8 feed-forward backward; of bias+dropout+residual and feed-forward up to 4 MiB
// (2048 x 512 bf16 forward 2.36 + 0.24 / 2.64 + 0.41 in the Infinity Cache and far, 3 MB feed-forward 3.1 + 0.2 / 3.4 + 0.4, backward 7.1 + 0.1 / 7.3 + 0.7).
// The head split's backward with its bias sum, a serial walk without loads ahead, gains from 1 MiB in all heads on (three of 1 MB 5.9 - 0.2 / 11.5 + 0.2 / 6.0 + 0.6, of 1.5 MB 6.5 - 0.4 / 12.1 + 0.2 / 6.6 + 0.6).
// Beyond, far memory costs more: 24 MB heads 27.5 + 0.6 split, 10.2 + 0.9 merge backward, 20 MB feed-forward backward 16.8 + 0.8.
constexpr int64_t kCachedLeast = 2ll << 20, kCachedLeastRows = 4ll << 20, kCachedLeastSums = 1ll << 20, kCachedMost = 16ll << 20;
inline bool stays_cached(int64_t elements, size_t elem_bytes, int64_t least = kCachedLeast)
{
    const int64_t bytes = elements * static_cast<int64_t>(elem_bytes);
    return bytes >= least && bytes <= kCachedMost;
}

// Division of a row index (below 2^32) by a launch constant: multiply-high by a host-made reciprocal, two shifts
// (Granlund and Montgomery's round-up form) -- 5 integer instructions where the 64-bit division the compiler emits
// for an int64 row index takes about 40 per row (a tenth of a short softmax row's vector-ALU work).
struct FastDiv {
    uint32_t m;
    int sh1, sh2;
};
inline FastDiv make_fastdiv(uint32_t d)
{
    if (d == 0) d = 1;
    int l = 0;
    while ((1ull << l) < d) ++l;                                   // ceil(log2 d)
    FastDiv f;
    f.m = static_cast<uint32_t>(((1ull << 32) * ((1ull << l) - d)) / d + 1);
    f.sh1 = l < 1 ? l : 1;
    f.sh2 = l - f.sh1;
    return f;
}
__device__ __forceinline__ uint32_t fastdiv(uint32_t n, const FastDiv& f)
{
    const uint32_t t = __umulhi(f.m, n);
    return (t + ((n - t) >> f.sh1)) >> f.sh2;
}

// Second stage of the column reductions: out[c] = sum over the P partial rows of
// partial[y][c], C columns, in a fixed order (reproducible).  Columns below `split`
// go to out0, those below `split2` to out1, the rest to out2.  A workgroup owns 32 columns; its 8 row slices each
// sum a contiguous chunk of rows with the loads of 32 rows in flight at a time (a
// plain loop would pay one memory latency per row; 256 partial rows are one batch per thread), then the
// slices are combined in slice order through LDS.  Measured behind a 21 MB producer kernel, 256 x 2560
// partials: 2.5 us against 2.7 us as 32 slices x 8 loads in a 1024-thread workgroup (an empty dependent
// kernel: 1.4 us).
constexpr int kFinalizeSlices = 8, kFinalizeLoads = 32;

// WHOLE: P is a whole number of batches (256 partial rows).  Otherwise a batch that runs past the slice's rows reads its last
// row again and drops it: a loop over the left-over rows paid one latency each (170 x 1536: 4.2 us, now 2.4).  LOADS: the batch, no larger than
// a slice of few partial rows needs; its sums round the same (feed-forward backward of 8 x 1024 with the batch of 32 0.25 us more, LayerNorm backward
// of 512 x 264, 64 partial rows, 0.3 us).
template <bool WHOLE, int LOADS>
__global__ __launch_bounds__(32 * kFinalizeSlices) void colsum_finalize_kernel(float* __restrict__ out0,
                                                                               float* __restrict__ out1,
                                                                               float* __restrict__ out2, int split,
                                                                               int split2,
                                                                               const float* __restrict__ partial,
                                                                               int P, int C)
{
    __shared__ float sm[kFinalizeSlices][33];
    const int lane = threadIdx.x & 31, slice = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + lane;
    const int chunk = (P + kFinalizeSlices - 1) / kFinalizeSlices;
    const int y0 = slice * chunk, y1 = min(P, y0 + chunk);
    float s = 0.0f;
    if (c < C) {
        for (int y = y0; y < y1; y += LOADS) {
            float t[LOADS];
#pragma unroll
            for (int k = 0; k < LOADS; ++k) t[k] = partial[static_cast<int64_t>(WHOLE ? y + k : min(y + k, y1 - 1)) * C + c];
#pragma unroll
            for (int k = 0; k < LOADS; ++k) t[k] = WHOLE || y + k < y1 ? t[k] : 0.0f;
            // pairwise: five roundings on a batch's way into the sum instead of up to 32
#pragma unroll
            for (int w = LOADS / 2; w > 0; w /= 2)
#pragma unroll
                for (int k = 0; k < w; ++k) t[k] += t[k + w];
            s += t[0];
        }
    }
    sm[slice][lane] = s;
    __syncthreads();
    if (slice == 0 && c < C) {
        float t = sm[0][lane];
#pragma unroll
        for (int w = 1; w < kFinalizeSlices; ++w) t += sm[w][lane];
        if (c < split) out0[c] = t;
        else if (c < split2) out1[c - split] = t;
        else out2[c - split2] = t;
    }
}

inline void launch_colsum_finalize(float* out0, float* out1, int split, const float* partial, int P, int C, hipStream_t s,
                                   float* out2 = nullptr, int split2 = 0x7FFFFFFF)
{
    const dim3 grid(static_cast<unsigned>((C + 31) / 32)), block(32 * kFinalizeSlices);
    if (P % (kFinalizeSlices * kFinalizeLoads) == 0)
        hipLaunchKernelGGL((colsum_finalize_kernel<true, kFinalizeLoads>), grid, block, 0, s, out0, out1, out2, split, split2, partial, P, C);
    else if (P <= kFinalizeSlices * 4)
        hipLaunchKernelGGL((colsum_finalize_kernel<false, 4>), grid, block, 0, s, out0, out1, out2, split, split2, partial, P, C);
    else if (P <= kFinalizeSlices * 8)
        hipLaunchKernelGGL((colsum_finalize_kernel<false, 8>), grid, block, 0, s, out0, out1, out2, split, split2, partial, P, C);
    else if (P <= kFinalizeSlices * 16)
        hipLaunchKernelGGL((colsum_finalize_kernel<false, 16>), grid, block, 0, s, out0, out1, out2, split, split2, partial, P, C);
    else
        hipLaunchKernelGGL((colsum_finalize_kernel<false, kFinalizeLoads>), grid, block, 0, s, out0, out1, out2, split, split2, partial, P, C);
}

// ---- short rows (up to 256 columns) of the element-wise operators
// The tensor is walked as ONE flat array in aligned packs (a pack may straddle two rows), so every
// access stays a 128-bit one and a pack still costs one Philox call (the dropout contract counts
// packs over the flat tensor).  F supplies the operator:
//   void  pack(int64_t e0, int c0, float (&g)[8])   loads, computes and stores the pack at element e0,
//                                                   whose first column is c0; g = the fp32 results
//   float one(int64_t e, int c)                      the same for one element of the ragged last pack
// With COLS the fp32 results also feed column sums (a bias gradient): a workgroup parks the
// results of a trip (256 threads x 4 packs, consecutive) in LDS, then every thread adds up, in
// ascending element order, the entries of the columns it owns (c = thread, thread + 256, ...); the
// owner alone touches a column's accumulator, so no atomics and a fixed order.  One partial row per workgroup, summed
// by colsum_finalize_kernel.
constexpr int kFlatPacks = 4;                                    // packs per thread and trip
constexpr int kFlatChunk = 256 * kFlatPacks * kPack;             // elements per trip
constexpr int kFlatMaxBlocks = 512;                              // partial rows at most

struct FlatPlan { int blocks, trips; };
inline FlatPlan flat_plan(int64_t total, bool cols)
{
    const int64_t chunks = ceil_div(total, kFlatChunk);
    FlatPlan p;
    if (!cols) { p.blocks = static_cast<int>(chunks); p.trips = 1; return p; }
    p.trips = static_cast<int>(ceil_div(chunks, kFlatMaxBlocks));
    if (p.trips < 1) p.trips = 1;
    p.blocks = static_cast<int>(ceil_div(chunks, p.trips));
    if (p.blocks < 1) p.blocks = 1;
    return p;
}

template <typename F, bool COLS>
__global__ __launch_bounds__(256) void flat_packs_kernel(F f, float* __restrict__ partial, int64_t total, int hidden, int trips)
{
    extern __shared__ float flat_lds[];        // COLS: [kFlatChunk] results of the trip, [hidden] accumulators
    const int tid = threadIdx.x;
    float* acc = nullptr;
    if constexpr (COLS) {
        acc = flat_lds + kFlatChunk;
        for (int c = tid; c < hidden; c += 256) acc[c] = 0.0f;     // read again by this thread only
    }
    for (int t = 0; t < trips; ++t) {
        const int64_t base = (static_cast<int64_t>(blockIdx.x) * trips + t) * kFlatChunk;
        if (base >= total) break;                                  // uniform over the workgroup
        const int cb = static_cast<int>(base % hidden);            // column of the trip's first element
#pragma unroll
        for (int u = 0; u < kFlatPacks; ++u) {
            const int off = (u * 256 + tid) * kPack;
            const int64_t e0 = base + off;
            float g[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (e0 + kPack <= total) {
                f.pack(e0, static_cast<int>(static_cast<uint32_t>(cb + off) % static_cast<uint32_t>(hidden)), g);
            } else if (e0 < total) {
                int c = static_cast<int>(static_cast<uint32_t>(cb + off) % static_cast<uint32_t>(hidden));
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (e0 + j < total) g[j] = f.one(e0 + j, c);
                    c = c + 1 == hidden ? 0 : c + 1;
                }
            }
            if constexpr (COLS) store8<float>(flat_lds + off, g);
        }
        if constexpr (COLS) {
            __syncthreads();
            const int64_t left = total - base;
            const int n = left < kFlatChunk ? static_cast<int>(left) : kFlatChunk;
            if (hidden >= 256) {
                for (int c = tid; c < hidden; c += 256) {
                    int i = c - cb;
                    if (i < 0) i += hidden;
                    float a = acc[c];
                    for (; i < n; i += hidden) a += flat_lds[i];
                    acc[c] = a;
                }
                __syncthreads();                                   // the next trip overwrites the results
            } else {
                // short rows: 256 / hidden threads share a column (every slices-th entry each, ascending), their
                // sums are added in slice order by the column's owner
                const int slices = 256 / hidden, c = tid % hidden, sl = tid / hidden;
                float a = 0.0f;
                if (sl < slices) {
                    int i = c - cb;
                    if (i < 0) i += hidden;
                    for (i += sl * hidden; i < n; i += slices * hidden) a += flat_lds[i];
                }
                __syncthreads();                                   // all entries read: the results' place is reused
                if (sl < slices) flat_lds[sl * hidden + c] = a;
                __syncthreads();
                if (tid < hidden) {
                    float tsum = acc[tid];
                    for (int k = 0; k < slices; ++k) tsum += flat_lds[k * hidden + tid];
                    acc[tid] = tsum;
                }
                __syncthreads();
            }
        }
    }
    if constexpr (COLS) {
        float* prow = partial + static_cast<int64_t>(blockIdx.x) * hidden;
        for (int c = tid; c < hidden; c += 256) prow[c] = acc[c];
    }
}

// dbias == nullptr: the element-wise part only.  workspace: flat_plan(total, true).blocks rows of hidden floats.
template <typename F>
inline void launch_flat_packs(const F& f, float* dbias, void* workspace, int64_t rows, int hidden, hipStream_t s)
{
    const int64_t total = rows * hidden;
    const FlatPlan pl = flat_plan(total, dbias != nullptr);
    const dim3 grid(static_cast<unsigned>(pl.blocks)), block(256);
    if (!dbias) {
        hipLaunchKernelGGL((flat_packs_kernel<F, false>), grid, block, 0, s, f, nullptr, total, hidden, 1);
        return;
    }
    float* partial = static_cast<float*>(workspace);
    hipLaunchKernelGGL((flat_packs_kernel<F, true>), grid, block, (kFlatChunk + hidden) * sizeof(float), s, f, partial, total, hidden, pl.trips);
    launch_colsum_finalize(dbias, dbias, hidden, partial, pl.blocks, hidden, s);
}

inline size_t flat_workspace_bytes(int64_t rows, int32_t hidden)
{
    return static_cast<size_t>(flat_plan(rows * hidden, true).blocks) * static_cast<size_t>(hidden) * sizeof(float);
}
// of the largest call of up to `rows` rows (at most one partial row per chunk, kFlatMaxBlocks in all)
inline size_t flat_workspace_bytes_upto(int64_t rows, int32_t hidden)
{
    const int64_t chunks = ceil_div(rows * hidden, kFlatChunk);
    return static_cast<size_t>(chunks < kFlatMaxBlocks ? chunks : kFlatMaxBlocks) * static_cast<size_t>(hidden) * sizeof(float);
}

// LayerNorm backward, launch shape of the kernel whose rows span several waves (512..8192 columns in whole packs, 129..8191 others): lanes per
// row, rows a workgroup holds at a time, workgroups (= partial rows of the column sums).
constexpr int kLnSpanThreads = 768;          // three waves per SIMD; wider rows take up to 1024 threads
struct LnBwdPlan { int lanes, slots, blocks; };
// rows that are not whole packs: both directions, from 129 columns on
inline bool ln_rag_spans(int32_t hidden) { return hidden % kPack != 0 && hidden > 128 && hidden < 8192; }
inline bool ln_bwd_spans(int32_t hidden) { return ln_rag_spans(hidden) || (hidden % kPack == 0 && hidden >= 512 && hidden <= 8192); }
inline int ln_span_lanes(int32_t hidden) { return ((hidden + kPack - 1) / kPack + 31) / 32 * 32; }
inline LnBwdPlan ln_bwd_span_plan(int64_t rows, int32_t hidden)
{
    constexpr int kMaxBlocks = 256;          // one per compute unit (8192 x 1280 fused: 26.0 us with the second stage, 512 of half the rows: 28.6)
    LnBwdPlan p;
    p.lanes = ln_span_lanes(hidden);
    const bool half_wave = p.lanes % 64 != 0;                     // then rows come in pairs
    // Of the slot counts that give 384..768 threads, the one that leaves the fewest slots idle in the last trip, the larger
    // among equals (8192 x 1024: 4 slots 21.5, 6 slots 23.2 us; 16000 x 640: 8 slots 25.9, 4 slots 27.3 us).  Short batches: no more
    // than leave three trips, which the loads ahead can overlap (2200 x 512: 3 slots 8.8, 8 slots 9.4 us).
    const int most = kLnSpanThreads / p.lanes;
    int64_t cap = ceil_div(rows, static_cast<int64_t>(kMaxBlocks) * 3);
    if (half_wave && cap == 3) cap = 4;      // pairs: two would leave five trips (2100 x 520 fp16 9.6 -> 8.9 us)
    if (cap > most) cap = most;
    p.slots = 0;
    int64_t best = 0;
    for (int n = 1; n <= cap; ++n) {
        if (half_wave && n % 2 != 0) continue;
        if (n * p.lanes < kLnSpanThreads / 2 && n + (half_wave ? 2 : 1) <= cap) continue;
        const int64_t cost = ceil_div(rows, static_cast<int64_t>(kMaxBlocks) * n) * n;
        if (p.slots == 0 || cost <= best) { p.slots = n; best = cost; }
    }
    if (p.slots == 0) {                       // one row at a time, in whole waves
        p.slots = 1;
        p.lanes = (p.lanes + 63) / 64 * 64;
    }
    // partial rows: at least 8 rows each where 256 of them would be more than 8 MiB (rows of more than 4096 columns)
    int64_t b = (8 << 20) / (2 * static_cast<int64_t>(sizeof(float)) * hidden);
    if (b < ceil_div(rows, 8)) b = ceil_div(rows, 8);
    if (b > kMaxBlocks) b = kMaxBlocks;
    if (b > ceil_div(rows, p.slots)) b = ceil_div(rows, p.slots);
    p.blocks = static_cast<int>(b < 1 ? 1 : b);
    return p;
}

// Number of partial-sum rows LayerNorm backward writes to the workspace: one per workgroup, so that the grid fills the 256
// compute units while the partials stay a small fraction of the tensor traffic.
inline int ln_bwd_blocks(int64_t rows, int32_t hidden)
{
    if (ln_bwd_spans(hidden)) return ln_bwd_span_plan(rows, hidden).blocks;
    int64_t b = ceil_div(rows, 8);       // at least 8 rows per workgroup
    if (b > 256) b = 256;   // one workgroup per compute unit: measured best at 8192 rows
    if (b < 1) b = 1;
    return static_cast<int>(b);
}

// ---- bias + dropout + residual: launch shapes (shared with the workspace sizing)
// Measured at 8192 x 1280 / 8192 x 1024 (fp16, p = 0.1): forward one row per lane 11.4 / 9.9 us, two 11.5 / 10.8, four
// 13.4 / 10.6; backward (without the column sums) 4 waves per workgroup 8.9 / 7.6 us, 8 waves 9.2 / 7.3, 16 waves 9.5 / 8.0;
// column blocks of 32 packs against 16: forward 11.4 / 9.7 against 11.5 / 10.2.
constexpr int kBdrFwdWaves = 4;                   // waves per forward workgroup; each takes its own rows
constexpr int kBdrFwdUnroll = 1;                  // rows a lane has in flight in forward
constexpr int kBdrBwdWaves = 4;                   // waves per backward workgroup
constexpr int kBdrMaxLanes = 32;                  // widest column block (packs) the kernels are built for

// Lanes of a wave that share a row: 32 or 16, the wider that divides the packs of a row; 16 with a
// ragged last column block if none does.
inline int bdr_lanes_per_row(int ppr)
{
    for (int w = kBdrMaxLanes; w >= 16; w >>= 1)
        if (ppr % w == 0) return w;
    return 16;
}

// Rows that are not whole packs run in packs of their own (RowPackIO) from 257 columns on; shorter ones, and rows of very few packs, take the
// flat walk.  Rows of few packs leave most lanes of a 16-lane row segment idle (measured at 32 Mi elements: forward
// 187 / 94 / 63 us at 8 / 16 / 24 columns against 47 us flat; backward 860 / 439 / 175 / 83 / 80 us at 8 / 16 / 24 / 64 / 72
// columns against 48 us flat), bias + activation + dropout works in column blocks of 64 packs
// (8 columns: 1629 / 10103 us in column blocks at 32 Mi elements, 51 / 95 us flat; 256 columns: 56 / 138 us).  For odd rows the same line:
// 257 columns in packs of their own against flat, 64 to 65536 rows, 0.43-1.12 in the four forward and backward kernels, 1.12 once.
constexpr int kFlatColumns = 256;
inline bool odd_in_packs(int hidden) { return hidden % kPack != 0 && hidden > kFlatColumns; }
inline bool bdr_fwd_is_flat(int hidden) { return hidden % kPack != 0 ? hidden <= kFlatColumns : hidden <= 32; }
inline bool bdr_bwd_is_flat(int hidden) { return hidden % kPack != 0 ? hidden <= kFlatColumns : hidden < 128; }
inline bool bad_is_flat(int hidden) { return hidden <= kFlatColumns; }
// A wave holds 64 packs of an odd row, 63 with dropout (dropout_factors8_row) and in bias + activation + dropout.  Rows of a few
// packs more leave a second column block with as good as nothing to do, and long tensors of them are faster flat.  Packs of
// their own against flat: bias + activation + dropout forward, 16 bits with dropout 505 columns 8192 / 24000 / 65536 rows 1.14 / 1.20 /
// 1.12, 513 columns 12000 / 24000 1.15 / 1.20, 545 24000 / 65536 0.93 / 1.10 (4096: 0.91, 0.90; 593 columns 0.78-0.96; fp32 0.83-1.06);
// bias + dropout + residual fp32, forward 505 with dropout 12000 / 16384 / 65536 0.76 / 1.10 / 1.12, without 513 16384 / 65536 0.93 / 1.06, 545 24000 /
// 65536 0.92 / 1.08, backward 505 / 513 / 593 / 641 at 24000 1.20 / 1.20 / 1.07 / 1.09 (16384 rows 0.71-0.95; 700 columns 1.00).
inline int odd_second_block(int hidden, int lanes) { return (hidden + kPack - 1) / kPack - lanes; }       // packs of it
inline bool bad_fwd_is_flat(int64_t rows, int hidden, int elem_bytes, bool drop)
{
    const int n = odd_second_block(hidden, kRagLanes);
    return bad_is_flat(hidden) ||
           (odd_in_packs(hidden) && elem_bytes == 2 && drop && n >= 1 && n <= 6 && rows * hidden >= (n == 1 ? 4000000 : n == 2 ? 6000000 : 30000000));
}
inline bool bdr_fwd_is_flat(int64_t rows, int hidden, int elem_bytes, bool drop)
{
    const int n = odd_second_block(hidden, drop ? kRagLanes : kWave);
    return bdr_fwd_is_flat(hidden) || (odd_in_packs(hidden) && elem_bytes == 4 && n >= 1 && n <= 6 && rows * hidden >= (n == 1 && drop ? 8000000 : 20000000));
}
inline bool bdr_bwd_is_flat(int64_t rows, int hidden, int elem_bytes, bool drop)
{
    const int n = odd_second_block(hidden, drop ? kRagLanes : kWave);
    return bdr_bwd_is_flat(hidden) || (odd_in_packs(hidden) && elem_bytes == 4 && n >= 1 && n <= 18 && rows * hidden >= (n <= 6 ? 10000000 : 14000000));
}
// column blocks of bias + activation + dropout: 64 packs, 63 where rows are not whole packs
inline int bad_col_blocks(int hidden) { return static_cast<int>(ceil_div(ceil_div(hidden, kPack), hidden % kPack == 0 ? 64 : kRagLanes)); }

// Backward launch shape: column blocks of w packs; row blocks (= partial rows of the column sums) of
// `trips` consecutive groups of waves * 64 / w rows.
constexpr int kBdrBwdWorkgroups = 1280;           // about five per compute unit: fewer (640, 768) cost 0.5-1.5 us at 8192 rows
constexpr int kBdrBwdMaxPartials = 256;           // partial rows the second stage sums
struct BdrBwdPlan { int w, col_blocks, row_blocks, trips; };
inline BdrBwdPlan bdr_bwd_plan(int64_t rows, int32_t hidden)
{
    BdrBwdPlan p;
    const int ppr = hidden / kPack;
    p.w = bdr_lanes_per_row(ppr);
    p.col_blocks = static_cast<int>(ceil_div(ppr, p.w));
    const int64_t units = ceil_div(rows, static_cast<int64_t>(kBdrBwdWaves) * (64 / p.w));     // row groups of one trip
    int64_t rb_max = kBdrBwdWorkgroups / p.col_blocks;
    if (rb_max > kBdrBwdMaxPartials) rb_max = kBdrBwdMaxPartials;
    if (rb_max < 1) rb_max = 1;
    const int64_t trips = ceil_div(units, rb_max);
    p.trips = static_cast<int>(trips < 1 ? 1 : trips);
    const int64_t rb = ceil_div(units, p.trips);
    p.row_blocks = static_cast<int>(rb < 1 ? 1 : rb);
    return p;
}

// Row blocks of the column-blocked backward kernels that leave one partial row of column sums per row block
// (feed-forward bias+activation+dropout, head merge): as many as give about `target` workgroups over the
// hidden / 512 column blocks.  Measured at 8192 x 5120 (GELU, dropout) and 4096 x 4096 (ReLU): 512 workgroups, two per
// compute unit, 45.2 / 35.2 us; 384: 49.8 / 40.7; 640: 47.5 / 37.9; 1024: 46.9 / 36.8; 2560 (one row block per
// 32 rows, the earlier choice): 49.8 / 38.4 -- totals that are not a multiple of the 256 compute units leave some
// of them with one workgroup more, and fewer, longer workgroups pay prologue, LDS epilogue and partial row less often.
// The head merge (no arithmetic, 128-byte pieces) wants more loads in flight: 1024 workgroups 26.5 us at
// 8192 x 3840, 768: 28.4, 1536: 27.6, 2048: 29.2, 512: 34.
constexpr int kBadBwdWorkgroups = 512, kHeadsBwdWorkgroups = 1024;
inline int colsum_row_blocks(int64_t rows, int32_t hidden, int target)
{
    const int64_t col_blocks = ceil_div(hidden, 64 * kPack);
    int64_t b = target / col_blocks;
    // at least 16 rows each, 8 in short calls, which leave compute units idle otherwise (512 x 2048 f32 8.7 -> 7.1 us, head merge of
    // 512 x 1536 f32 7.4 -> 6.3); more partial rows than one batch of the second stage cost more (3133 x 1152: 196 8.4 us, 341 8.8)
    const int64_t most = ceil_div(rows, rows <= 2048 ? 8 : 16);
    if (b > most) b = most;
    return static_cast<int>(b < 1 ? 1 : b);
}
// the largest of colsum_row_blocks over the calls of up to `rows` rows (it falls from 256 to 129 behind 2048 rows)
inline int colsum_row_blocks_upto(int64_t rows, int32_t hidden, int target)
{
    const int here = colsum_row_blocks(rows, hidden, target), at = rows > 2048 ? colsum_row_blocks(2048, hidden, target) : 0;
    return here > at ? here : at;
}
inline int bdr_rag_row_blocks(int64_t rows, int32_t hidden)
{
    const int b = colsum_row_blocks(rows, hidden, kBdrBwdWorkgroups);
    return b < kBdrBwdMaxPartials ? b : kBdrBwdMaxPartials;
}
inline int bad_bwd_row_blocks(int64_t rows, int32_t hidden) { return colsum_row_blocks(rows, hidden, kBadBwdWorkgroups); }
// (fp32 from 3.2 M elements on: 16 rows each in short calls too, 2048 x 1920 12.2 us against 14.1 with 8; 2048 x 1536 and 16 bits 8 rows)
inline int heads_bwd_row_blocks(int64_t rows, int32_t hidden, int elem_bytes)
{
    const int b = colsum_row_blocks(rows, hidden, kHeadsBwdWorkgroups);
    const int64_t few = ceil_div(rows, 16);
    return elem_bytes == 4 && rows * hidden > 3200000 && b > few ? static_cast<int>(few) : b;
}

// ---- workspace of the column sums: what one call's launch writes (the entry points ask for no more), and the same for the
// largest of all calls of up to `rows` rows, which lsq_workspace_bytes tells.  The launches' numbers of partial rows follow from what
// is fastest at each size and fall here and there as the rows grow; a program that keeps one workspace of its longest
// batch's size is not to notice.
inline size_t partial_bytes(int64_t row_blocks, int32_t cols) { return static_cast<size_t>(row_blocks) * static_cast<size_t>(cols) * sizeof(float); }
inline size_t bdr_bwd_bytes(int64_t rows, int32_t hidden, int elem_bytes, bool drop)
{
    if (bdr_bwd_is_flat(rows, hidden, elem_bytes, drop)) return flat_workspace_bytes(rows, hidden);
    return partial_bytes(odd_in_packs(hidden) ? bdr_rag_row_blocks(rows, hidden) : bdr_bwd_plan(rows, hidden).row_blocks, hidden);
}
inline size_t bdr_bwd_bytes_upto(int64_t rows, int32_t hidden)
{
    if (bdr_bwd_is_flat(hidden)) return flat_workspace_bytes_upto(rows, hidden);
    if (odd_in_packs(hidden)) {                       // the flat walk of a long fp32 call included
        const int b = colsum_row_blocks_upto(rows, hidden, kBdrBwdWorkgroups);
        const size_t packs = partial_bytes(b < kBdrBwdMaxPartials ? b : kBdrBwdMaxPartials, hidden);
        const size_t flat = bdr_bwd_is_flat(rows, hidden, 4, true) || bdr_bwd_is_flat(rows, hidden, 4, false) ? flat_workspace_bytes_upto(rows, hidden) : 0;
        return packs > flat ? packs : flat;
    }
    // at most one per group of rows, and rb_max of bdr_bwd_plan
    const BdrBwdPlan one = bdr_bwd_plan(1, hidden);
    const int64_t units = ceil_div(rows, static_cast<int64_t>(kBdrBwdWaves) * (64 / one.w));
    int64_t most = kBdrBwdWorkgroups / one.col_blocks;
    if (most > kBdrBwdMaxPartials) most = kBdrBwdMaxPartials;
    if (most > units) most = units;
    return partial_bytes(most < 1 ? 1 : most, hidden);
}
inline size_t bad_bwd_bytes(int64_t rows, int32_t hidden)
{
    return bad_is_flat(hidden) ? flat_workspace_bytes(rows, hidden) : partial_bytes(bad_bwd_row_blocks(rows, hidden), hidden);
}
inline size_t bad_bwd_bytes_upto(int64_t rows, int32_t hidden)
{
    return bad_is_flat(hidden) ? flat_workspace_bytes_upto(rows, hidden) : partial_bytes(colsum_row_blocks_upto(rows, hidden, kBadBwdWorkgroups), hidden);
}
inline size_t heads_bwd_bytes(int64_t rows, int32_t cols, int elem_bytes) { return partial_bytes(heads_bwd_row_blocks(rows, cols, elem_bytes), cols); }
inline size_t heads_bwd_bytes_upto(int64_t rows, int32_t cols) { return partial_bytes(colsum_row_blocks_upto(rows, cols, kHeadsBwdWorkgroups), cols); }
inline size_t ln_bwd_bytes(int64_t rows, int32_t hidden, int sums) { return partial_bytes(static_cast<int64_t>(ln_bwd_blocks(rows, hidden)) * sums, hidden); }

// Workspace of the embedding backward:
//   order  [rows] (token position, sort key), 8 bytes each
//   second buffer of the radix sort, as many; the parts of the in-LDS sort that are too large for it (beyond 2048 tokens) lie there too
//   digit counts of the radix sort [256][workgroups]
//   beyond kEmbSortMax tokens: two fp32 rows per range
constexpr int64_t kEmbSortMax = 16384;
constexpr int kEmbRange = 64;        // entries of the sorted order that a workgroup of the accumulation owns
struct EmbBwdPlan {
    int radix_blocks;
    size_t pair_bytes, hist_bytes, part_bytes;
    size_t total() const { return 2u * pair_bytes + hist_bytes + part_bytes; }        // never falls as the rows grow
};
inline EmbBwdPlan emb_bwd_plan(int64_t rows, int32_t hidden)
{
    EmbBwdPlan p;
    p.pair_bytes = static_cast<size_t>(ceil_div(rows, kEmbRange)) * kEmbRange * 8u;        // whole ranges
    p.radix_blocks = static_cast<int>(ceil_div(rows, 2048));
    p.hist_bytes = static_cast<size_t>(256) * static_cast<size_t>(p.radix_blocks) * sizeof(int32_t);
    p.part_bytes = rows > kEmbSortMax ? 2u * static_cast<size_t>(ceil_div(rows, kEmbRange)) * static_cast<size_t>(ceil_div(hidden, kPack)) * kPack * sizeof(float) : 0;
    return p;
}

}  // namespace lsq
