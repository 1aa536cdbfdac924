// Fused bias + dropout + residual, forward and backward (Sec. IV-A of the paper,
// Transformer layers: "bias adding, dropout, and residual" in one launch).
//
// Layout for rows of whole packs (hidden % 8 == 0): W lanes of a wave (W = 32 or 16, the wider
// that divides the packs of a row, so no lane idles on a ragged last column block) own W
// consecutive packs of one row and the wave covers 64 / W rows at a time; a workgroup's column
// block is fixed, so the bias pack is loaded once into registers, every access is a 128-bit one,
// and in backward each lane accumulates the column sums of its own 8 columns with no atomics.
// The dropout mask is never stored: both directions rebuild it from the Philox
// counter of the pack.  HBM traffic: forward 3 tensors, backward 2.
//
// Backward column sums (dbias): a workgroup adds up its lanes' sums through LDS in a fixed order and
// writes one partial row of its column block to the workspace; a second small kernel sums the
// partial rows in a fixed order (bit-reproducible; no atomics).
#include "host.hpp"

namespace lsq {

constexpr bool kNT = true;    // nontemporal hint on the streamed tensors (not on gamma/beta/bias)

// A wave as 64 / W row segments of W packs: lane -> (row of the group, pack of the column block).
template <int W> struct BdrLane {
    static constexpr int SUB = 64 / W;
    int lane, sub;
    __device__ __forceinline__ BdrLane() : lane((threadIdx.x & 63) % W), sub((threadIdx.x & 63) / W) {}
};

template <typename T, bool HAS_BIAS, bool DROP, int W, bool PAIR, bool NTL>
__global__ __launch_bounds__(64 * kBdrFwdWaves) void bdr_fwd_cols(T* out, const T* x, const T* __restrict__ bias,
                                                                  const T* res, int64_t rows, int ppr, DropoutParams d)
{
    constexpr int SUB = 64 / W, U = kBdrFwdUnroll, RPI = kBdrFwdWaves * SUB * U;
    using P = LanePacks<T, PAIR ? W : 1>;
    const BdrLane<W> ln;
    const int wave = threadIdx.x >> 6;
    const int cp = blockIdx.x * W + P::pack(ln.lane);
    const bool mine = cp < ppr;
    if (!P::kPaired && !mine) return;
    // the bias stays packed and is widened where it is used: widening it here would make the
    // row loads below wait for its arrival
    RawPack<T> braw = zero_raw<T>();
    if constexpr (HAS_BIAS) braw = load_raw<T>(bias + static_cast<int64_t>(P::kPaired ? min(cp, ppr - 1) : cp) * kPack);
    for (int64_t base = static_cast<int64_t>(blockIdx.y) * RPI; base < rows; base += static_cast<int64_t>(gridDim.y) * RPI) {
        RawPack<T> xr[U], rr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = base + (u * kBdrFwdWaves + wave) * SUB + ln.sub;
            const bool ok = r < rows && (!P::kPaired || mine);
            xr[u] = P::template load<NTL>(x + (r * ppr + cp) * kPack, ok);
            rr[u] = P::template load<NTL>(res + (r * ppr + cp) * kPack, ok);
        }
        // the dropout factors need no data: they are drawn while the loads are in flight
        float k[DROP ? U : 1][8];
        if constexpr (DROP) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t r = base + (u * kBdrFwdWaves + wave) * SUB + ln.sub;
                dropout_factors8(d, static_cast<uint64_t>(r * ppr + cp), k[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = base + (u * kBdrFwdWaves + wave) * SUB + ln.sub;
            if (r < rows) {                   // (the lanes of a pair share the row)
                const int64_t pack = r * ppr + cp;
                float xf[8], rf[8], b[8];
                unpack<T>(P::settle(xr[u]), xf);
                unpack<T>(P::settle(rr[u]), rf);
                if constexpr (HAS_BIAS) opaque<T>(braw);
                unpack<T>(braw, b);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float z = xf[j] + b[j];
                    rf[j] = DROP ? fmaf(z, k[DROP ? u : 0][j], rf[j]) : rf[j] + z;
                }
                pin_f32(rf);                  // rounds like the kernel that fuses the LayerNorm behind it
                P::template store<kNT>(out + pack * kPack, rf, !P::kPaired || mine);
            }
        }
    }
}

// Backward.  partial: [gridDim.y][hidden] fp32 column sums of the workgroups' rows (nullptr:
// dbias not wanted), summed over the row blocks by colsum_finalize_kernel.
template <typename T, bool DROP, int W, bool PAIR, bool NTL>
__global__ __launch_bounds__(64 * kBdrBwdWaves) void bdr_bwd_cols(T* dx, float* __restrict__ partial, const T* dy,
                                                                  int64_t rows, int ppr, int trips, DropoutParams d)
{
    constexpr int SUB = 64 / W, NW = kBdrBwdWaves, THREADS = 64 * NW;
    __shared__ float sm[NW * 8 * 64];      // the lanes' sums
    using P = LanePacks<T, PAIR ? W : 1>;
    const BdrLane<W> ln;
    const int wave = threadIdx.x >> 6, lane = ln.sub * W + P::pack(ln.lane);      // by pack
    const int cp = blockIdx.x * W + P::pack(ln.lane);
    const bool mine = cp < ppr, active = P::kPaired || mine;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (active) {
        // A workgroup walks `trips` consecutive groups of NW * SUB rows; the pack of the next trip is
        // loaded before this trip's is used, and the dropout factors, which need no data, are
        // drawn while the loads are in flight.
        const int64_t first = static_cast<int64_t>(blockIdx.y) * trips * (NW * SUB) + wave * SUB + ln.sub;
        RawPack<T> nxt = P::template load<NTL>(dy + (first * ppr + cp) * kPack, first < rows && mine);
        for (int t = 0; t < trips; ++t) {
            const int64_t r = first + static_cast<int64_t>(t) * (NW * SUB);
            const RawPack<T> cur = nxt;
            const int64_t rn = r + NW * SUB;
            if (t + 1 < trips && rn < rows) nxt = P::template load<NTL>(dy + (rn * ppr + cp) * kPack, mine);
            if (r < rows) {
                const int64_t pack = r * ppr + cp;
                float g[8], k[8];
                if constexpr (DROP) dropout_factors8(d, static_cast<uint64_t>(pack), k);
                unpack<T>(P::settle(cur), g);
                if constexpr (DROP) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) g[j] *= k[j];
                }
                pin_f32(g);
                P::template store<kNT>(dx + pack * kPack, g, mine);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += g[j];
            }
        }
    }
    if (partial == nullptr) return;        // uniform over the grid
    // the workgroup's sums: wave by wave, row of the group by row of the group, in that order
#pragma unroll
    for (int j = 0; j < 8; ++j) sm[(wave * 8 + j) * 64 + lane] = acc[j];
    __syncthreads();
    const int hidden = ppr * kPack;
    const int c0 = blockIdx.x * W * kPack;                       // first column of the block
    const int ncols = min(W * kPack, hidden - c0);
    float* prow = partial + static_cast<int64_t>(blockIdx.y) * hidden + c0;
    for (int c = threadIdx.x; c < W * kPack; c += THREADS) {
        const int j = c / W, col = c % W;                        // consecutive threads read consecutive LDS words
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int sb = 0; sb < SUB; ++sb) t += sm[(w * 8 + j) * 64 + sb * W + col];
        if (col * kPack + j < ncols) prow[col * kPack + j] = t;
    }
}

// ---- rows that are not whole packs, walked in packs counted from the row's start (RowPackIO): a wave holds kRagLanes packs of a row, all its
// lanes stay, because a pack's dropout words come from two lanes.  Forward / backward in us, the flat walk in brackets: 8192 x 1281 bf16 with
// dropout 15.9 / 18.0 (19.2 / 25.0), 2000 x 5001 14.6 / 14.8 (19.4 / 32.2), 600 x 7001 fp16 8.9 / 11.1 (10.6 / 25.4), 500 x 259 f32 3.2 / 7.1 (8.9 / 9.1).
// (backward with 4 waves a workgroup; the waves by type and width: bdr_bwd_dispatch)
constexpr int kBdrRagWaves = 4;
template <bool DROP> constexpr int kBdrRagLanes = DROP ? kRagLanes : kWave;      // (without dropout no lane needs its neighbour)

template <typename T, bool DROP>
__global__ __launch_bounds__(64 * kBdrRagWaves) void bdr_fwd_rag(T* out, const T* x, const T* __restrict__ bias, const T* res,
                                                                 int64_t rows, RowPackIO<T, true> io, DropoutParams d)
{
    const int lane = threadIdx.x & 63, col = blockIdx.x * kBdrRagLanes<DROP> + lane, cp = min(col, io.ppr - 1);
    RawPack<T> braw = bias ? io.template ahead<false>(bias, 0, cp) : zero_raw<T>();      // uniform
    for (int64_t r = static_cast<int64_t>(blockIdx.y) * kBdrRagWaves + (threadIdx.x >> 6); r < rows; r += static_cast<int64_t>(gridDim.y) * kBdrRagWaves) {
        const RawPack<T> xr = io.template ahead<kNT>(x, r, cp), rr = io.template ahead<kNT>(res, r, cp);
        float xf[8], rf[8], b[8], k[8];
        if constexpr (DROP) dropout_factors8_row(d, static_cast<uint64_t>(io.element(r, col)), k);
        unpack<T>(io.settle(xr, cp), xf);
        unpack<T>(io.settle(rr, cp), rf);
        opaque<T>(braw);
        unpack<T>(io.settle(braw, cp), b);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float z = xf[j] + b[j];
            rf[j] = DROP ? fmaf(z, k[j], rf[j]) : rf[j] + z;
        }
        pin_f32(rf);
        if (col < io.ppr && lane < kBdrRagLanes<DROP>) io.template store<kNT>(out, r, cp, rf);
    }
}

template <typename T, bool DROP, int W>
__global__ __launch_bounds__(64 * W) void bdr_bwd_rag(T* dx, float* __restrict__ partial, const T* dy, int64_t rows,
                                                                 RowPackIO<T, true> io, DropoutParams d)
{
    __shared__ float sm[W][8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = blockIdx.x * kBdrRagLanes<DROP> + lane, cp = min(col, io.ppr - 1);
    const bool mine = col < io.ppr && lane < kBdrRagLanes<DROP>;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t stride = static_cast<int64_t>(gridDim.y) * W;
    int64_t r = static_cast<int64_t>(blockIdx.y) * W + wave;
    RawPack<T> nxt = r < rows ? io.template ahead<kNT>(dy, r, cp) : zero_raw<T>();
    for (; r < rows; r += stride) {
        const RawPack<T> cur = nxt;
        if (r + stride < rows) nxt = io.template ahead<kNT>(dy, r + stride, cp);
        float g[8], k[8];
        if constexpr (DROP) dropout_factors8_row(d, static_cast<uint64_t>(io.element(r, col)), k);
        unpack<T>(io.settle(cur, cp), g);
        if constexpr (DROP) {
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] *= k[j];
        }
        pin_f32(g);
        if (mine) io.template store<kNT>(dx, r, cp, g);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += g[j];
    }
    if (partial == nullptr) return;        // uniform over the grid
#pragma unroll
    for (int j = 0; j < 8; ++j) sm[wave][j][lane] = acc[j];
    __syncthreads();
    if (wave == 0 && mine) {
        float* dst = partial + static_cast<int64_t>(blockIdx.y) * io.hidden + cp * kPack;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float t = sm[0][j][lane];
#pragma unroll
            for (int w = 1; w < W; ++w) t += sm[w][j][lane];
            if (cp * kPack + j < io.hidden) dst[j] = t;
        }
    }
}

// ---- short rows, and long tensors of odd rows with a thin second column block (bdr_fwd_is_flat, bdr_bwd_is_flat): the operators for flat_packs_kernel
template <typename T>
struct BdrFwdFlat {
    T* out;
    const T* x;
    const T* bias;
    const T* res;
    int hidden;
    DropoutParams d;
    __device__ __forceinline__ void pack(int64_t e0, int c0, float (&g)[8]) const
    {
        const RawPack<T> xr = load_raw<T, kNT>(x + e0), rr = load_raw<T, kNT>(res + e0);
        float k[8];
        if (d.on) dropout_factors8(d, static_cast<uint64_t>(e0 >> 3), k);
        float xf[8];
        unpack<T>(xr, xf);
        unpack<T>(rr, g);
        int c = c0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float z = bias ? xf[j] + to_f32<T>(bias[c]) : xf[j];
            g[j] = d.on ? fmaf(z, k[j], g[j]) : g[j] + z;
            c = c + 1 == hidden ? 0 : c + 1;
        }
        pin_f32(g);
        store8<T, kNT>(out + e0, g);
    }
    __device__ __forceinline__ float one(int64_t e, int c) const
    {
        float z = to_f32<T>(x[e]);
        if (bias) z += to_f32<T>(bias[c]);
        const float r = to_f32<T>(res[e]);
        const float v = d.on ? fmaf(z, dropout_factor1(d, static_cast<uint64_t>(e)), r) : r + z;
        out[e] = from_f32<T>(v);
        return v;
    }
};

template <typename T>
struct BdrBwdFlat {
    T* dx;
    const T* dy;
    DropoutParams d;
    __device__ __forceinline__ void pack(int64_t e0, int, float (&g)[8]) const
    {
        const RawPack<T> cur = load_raw<T, kNT>(dy + e0);
        float k[8];
        if (d.on) dropout_factors8(d, static_cast<uint64_t>(e0 >> 3), k);
        unpack<T>(cur, g);
        if (d.on) {
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] *= k[j];
        }
        pin_f32(g);
        store8<T, kNT>(dx + e0, g);
    }
    __device__ __forceinline__ float one(int64_t e, int) const
    {
        float g = to_f32<T>(dy[e]);
        if (d.on) g *= dropout_factor1(d, static_cast<uint64_t>(e));
        dx[e] = from_f32<T>(g);
        return g;
    }
};

// fp32 in lane pairs from 2 MiB a tensor on: below, the second address and the exchange are in the way of a few waves (1 MB forward / backward
// 2.24 / 4.76 us, in pairs 2.34 / 4.80 with inputs in L2, 2.7 / 4.9 and 3.1 / 5.6 from far memory; 2 MB 4.0 / 6.0 and 3.6 / 6.3, 4 MB 5.8 / 7.1 and 5.2 / 7.2).
template <typename T>
inline bool bdr_paired(int64_t rows, int32_t hidden) { return sizeof(T) == 4 && rows * hidden >= (1 << 19); }

template <typename T>
static lsq_status bdr_fwd_dispatch(void* out, const void* x, const void* bias, const void* res, int64_t rows,
                                   int32_t hidden, const DropoutParams& d, hipStream_t s)
{
    T* o = static_cast<T*>(out);
    const T* xp = static_cast<const T*>(x);
    const T* bp = static_cast<const T*>(bias);
    const T* rp = static_cast<const T*>(res);
    const bool flat = bdr_fwd_is_flat(rows, hidden, sizeof(T), d.on != 0);
    if (!flat && !odd_in_packs(hidden)) {
        const int ppr = hidden / kPack;
        const int w = bdr_lanes_per_row(ppr);
        const int64_t rpi = static_cast<int64_t>(kBdrFwdWaves) * (64 / w) * kBdrFwdUnroll;     // rows of a workgroup's trip
        int64_t rb = ceil_div(rows, rpi);
        if (rb > 8192) rb = 8192;
        const dim3 grid(static_cast<unsigned>(ceil_div(ppr, w)), static_cast<unsigned>(rb)), block(64 * kBdrFwdWaves);
        const bool drop = d.on != 0;
        const bool pair = bdr_paired<T>(rows, hidden), cached = stays_cached(rows * hidden, sizeof(T), kCachedLeastRows) && (sizeof(T) == 2 || pair);
#define LSQ_BDR_FWD(W, PAIR, NTL)                                                                                            \
        if (w == W && pair == (PAIR) && cached != NTL) {                                                                                   \
            if (bp && drop) hipLaunchKernelGGL((bdr_fwd_cols<T, true, true, W, PAIR, NTL>), grid, block, 0, s, o, xp, bp, rp, rows, ppr, d);    \
            else if (bp) hipLaunchKernelGGL((bdr_fwd_cols<T, true, false, W, PAIR, NTL>), grid, block, 0, s, o, xp, bp, rp, rows, ppr, d);     \
            else if (drop) hipLaunchKernelGGL((bdr_fwd_cols<T, false, true, W, PAIR, NTL>), grid, block, 0, s, o, xp, bp, rp, rows, ppr, d);   \
            else hipLaunchKernelGGL((bdr_fwd_cols<T, false, false, W, PAIR, NTL>), grid, block, 0, s, o, xp, bp, rp, rows, ppr, d);            \
        }
        LSQ_BDR_FWD(32, false, true) LSQ_BDR_FWD(16, false, true)
        LSQ_BDR_FWD(32, sizeof(T) == 4, false) LSQ_BDR_FWD(16, sizeof(T) == 4, false)
        if constexpr (sizeof(T) == 4) { LSQ_BDR_FWD(32, true, true) LSQ_BDR_FWD(16, true, true) }
#undef LSQ_BDR_FWD
    } else if (!flat) {
        const RowPackIO<T, true> io(hidden);
        int64_t rb = ceil_div(rows, kBdrRagWaves);
        if (rb > 8192) rb = 8192;
        const dim3 grid(static_cast<unsigned>(ceil_div(io.ppr, d.on ? kRagLanes : kWave)), static_cast<unsigned>(rb)), block(64 * kBdrRagWaves);
        if (d.on) hipLaunchKernelGGL((bdr_fwd_rag<T, true>), grid, block, 0, s, o, xp, bp, rp, rows, io, d);
        else hipLaunchKernelGGL((bdr_fwd_rag<T, false>), grid, block, 0, s, o, xp, bp, rp, rows, io, d);
    } else {
        launch_flat_packs(BdrFwdFlat<T>{o, xp, bp, rp, hidden, d}, nullptr, nullptr, rows, hidden, s);
    }
    return launch_status();
}

template <typename T>
static lsq_status bdr_bwd_dispatch(void* dx, float* dbias, const void* dy, int64_t rows, int32_t hidden,
                                   const DropoutParams& d, void* workspace, hipStream_t s)
{
    T* o = static_cast<T*>(dx);
    const T* g = static_cast<const T*>(dy);
    const bool flat = bdr_bwd_is_flat(rows, hidden, sizeof(T), d.on != 0);
    if (!flat && !odd_in_packs(hidden)) {
        const int ppr = hidden / kPack;
        const BdrBwdPlan pl = bdr_bwd_plan(rows, hidden);
        const dim3 grid(static_cast<unsigned>(pl.col_blocks), static_cast<unsigned>(pl.row_blocks)), block(64 * kBdrBwdWaves);
        float* partial = dbias ? static_cast<float*>(workspace) : nullptr;
        const bool pair = bdr_paired<T>(rows, hidden), cached = stays_cached(rows * hidden, sizeof(T), kCachedLeastRows) && (sizeof(T) == 2 || pair);
#define LSQ_BDR_BWD(W, PAIR, NTL)                                                                                       \
        if (pl.w == W && pair == (PAIR) && cached != NTL) {                                                               \
            if (d.on) hipLaunchKernelGGL((bdr_bwd_cols<T, true, W, PAIR, NTL>), grid, block, 0, s, o, partial, g, rows, ppr, pl.trips, d);    \
            else hipLaunchKernelGGL((bdr_bwd_cols<T, false, W, PAIR, NTL>), grid, block, 0, s, o, partial, g, rows, ppr, pl.trips, d);         \
        }
        LSQ_BDR_BWD(32, false, true) LSQ_BDR_BWD(16, false, true)
        LSQ_BDR_BWD(32, sizeof(T) == 4, false) LSQ_BDR_BWD(16, sizeof(T) == 4, false)
        if constexpr (sizeof(T) == 4) { LSQ_BDR_BWD(32, true, true) LSQ_BDR_BWD(16, true, true) }
        if (dbias) launch_colsum_finalize(dbias, dbias, hidden, partial, pl.row_blocks, hidden, s);
#undef LSQ_BDR_BWD
    } else if (!flat) {
        const RowPackIO<T, true> io(hidden);
        const int rb = bdr_rag_row_blocks(rows, hidden);
        const int col_blocks = static_cast<int>(ceil_div(io.ppr, d.on ? kRagLanes : kWave));
        // 4 / 8 / 16 waves, at most 256 partial rows either way: fp16 with dropout 65536 x 257 48.3 / 32.1 / 27.3 us, 65536 x 505 67 / 50 / 52,
        // 32768 x 1001 40.7 / 33.6 / 35.6, 4096 x 1281 11.8 / 11.6 / 13.6; fp32 65536 x 257 60.5 / 38.3 / 35.1, but over several column
        // blocks 32768 x 700 52.0 / 57.7 / 58.8, 4096 x 1281 12.8 / 13.4 / 14.7, and 16 bits beyond three 16384 x 2050 0.62 / 0.65 of the flat walk
        const int waves = col_blocks <= (sizeof(T) == 2 ? 3 : 1) ? 8 : 4;
        const dim3 grid(static_cast<unsigned>(col_blocks), static_cast<unsigned>(rb)), block(64 * waves);
        float* partial = dbias ? static_cast<float*>(workspace) : nullptr;
#define LSQ_BDR_RAG(DROP)                                                                                                       \
        if (waves == 8) hipLaunchKernelGGL((bdr_bwd_rag<T, DROP, 8>), grid, block, 0, s, o, partial, g, rows, io, d);      \
        else hipLaunchKernelGGL((bdr_bwd_rag<T, DROP, 4>), grid, block, 0, s, o, partial, g, rows, io, d)
        if (d.on) { LSQ_BDR_RAG(true); } else { LSQ_BDR_RAG(false); }
#undef LSQ_BDR_RAG
        if (dbias) launch_colsum_finalize(dbias, dbias, hidden, partial, rb, hidden, s);
    } else {
        // every pack is read and written by one thread, which also hands its fp32 results to the column sums: in place is fine
        launch_flat_packs(BdrBwdFlat<T>{o, g, d}, dbias, workspace, rows, hidden, s);
    }
    return launch_status();
}

}  // namespace lsq

extern "C" lsq_status lsq_bias_dropout_residual_fwd(void* out, const void* x, const void* bias, const void* residual,
                                                    int64_t rows, int32_t hidden, float p, uint64_t seed,
                                                    uint64_t offset, lsq_dtype dt, void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p, seed, offset, &d));
    if (rows == 0) return LSQ_OK;
    LSQ_REQUIRE(out && x && residual);
    LSQ_ALIGNED(out); LSQ_ALIGNED(x); LSQ_ALIGNED(bias); LSQ_ALIGNED(residual);
    LSQ_REQUIRE(ceil_div(rows * hidden, 256) <= 0x7FFFFFFF);
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (dt) {
        case LSQ_F16: return bdr_fwd_dispatch<f16>(out, x, bias, residual, rows, hidden, d, s);
        case LSQ_BF16: return bdr_fwd_dispatch<bf16>(out, x, bias, residual, rows, hidden, d, s);
        default: return bdr_fwd_dispatch<float>(out, x, bias, residual, rows, hidden, d, s);
    }
}

extern "C" lsq_status lsq_bias_dropout_residual_bwd(void* dx, float* dbias, const void* dy, int64_t rows,
                                                    int32_t hidden, float p, uint64_t seed, uint64_t offset,
                                                    void* workspace, size_t workspace_bytes, lsq_dtype dt,
                                                    void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p, seed, offset, &d));
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (rows == 0) {
        if (dbias) return zero_fill(dbias, hidden, s);
        return LSQ_OK;
    }
    LSQ_REQUIRE(dx && dy);
    LSQ_ALIGNED(dx); LSQ_ALIGNED(dy); LSQ_ALIGNED(dbias); LSQ_ALIGNED(workspace);
    LSQ_REQUIRE(ceil_div(rows * hidden, 256) <= 0x7FFFFFFF);
    if (dbias) {
        const size_t need = bdr_bwd_bytes(rows, hidden, dt == LSQ_F32 ? 4 : 2, d.on != 0);
        if (need && (!workspace || workspace_bytes < need)) return LSQ_WORKSPACE_TOO_SMALL;
    }
    switch (dt) {
        case LSQ_F16: return bdr_bwd_dispatch<f16>(dx, dbias, dy, rows, hidden, d, workspace, s);
        case LSQ_BF16: return bdr_bwd_dispatch<bf16>(dx, dbias, dy, rows, hidden, d, workspace, s);
        default: return bdr_bwd_dispatch<float>(dx, dbias, dy, rows, hidden, d, workspace, s);
    }
}
