// LayerNorm forward and backward (Sec. IV-B of the paper, "dependent reduction
// rewriting").
//
// The paper merges the mean and variance reductions by computing E[x^2]-E[x]^2
// so that neither waits for the other.  Here a row lives in registers after one
// 128-bit load per lane and pack, so the second reduction costs no memory traffic
// at all; it is therefore taken about the mean (two passes over registers), which
// cannot cancel catastrophically.  Backward uses the xhat form of the gradient:
// its two row sums (sum g, sum g*xhat) are independent given the saved mean and
// rstd, and run side by side in the same DPP reduction steps.
//
// Layout: LPR lanes share a row (8..64 lanes of one wave, or a whole workgroup); each lane holds VPL packs of 8
// columns, strided by LPR packs so that a wave's loads are contiguous.  gamma/beta stay in
// registers while the workgroup walks down its rows.  Backward of 512..8192 columns: one pack per lane, a row over several
// waves.  dgamma/dbeta: every lane
// accumulates its own columns over its rows, the row slots of a workgroup are
// summed in a fixed order through LDS, one partial row per workgroup goes to the
// workspace and a second small kernel sums the partial rows in order.  No atomics.
#include <mutex>

#include "host.hpp"

namespace lsq {

constexpr bool kNT = true;    // nontemporal hint on the streamed tensors (not on gamma/beta/bias)

// A row's total, forward.  One width may be served by several shapes (lanes x packs per lane) depending on the number of rows
// (ln_fwd_shape), and a row must not come out with other bits because its batch is larger: all shapes add in ONE order.
// A lane sums its packs by their index modulo 256 (in LnParts accumulators), these classes add 64 apart in ascending order, then
// the two half-waves add, then 32 lanes as group_sum<32> does.  So 32 x 2 and 64 x 1, or 64 x 4 and 256 x 1, round alike.
template <int LPR, int VPL> constexpr int kLnParts = VPL < 256 / LPR ? VPL : 256 / LPR;

// the two half-waves added: lane i has lanes i % 32 and i % 32 + 32
__device__ __forceinline__ float half_waves_sum(float v)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    const unsigned lower = r.x, upper = r.y;       // (a bit cast of r.y itself reads r.x)
    return __builtin_bit_cast(float, lower) + __builtin_bit_cast(float, upper);
}

// `buf`: 256 floats where the row spans the workgroup; it may be written again only behind another barrier
template <int LPR, int VPL, bool PAIRED>
__device__ __forceinline__ float ln_row_total(const float (&part)[kLnParts<LPR, VPL>], float* buf)
{
    constexpr int N = kLnParts<LPR, VPL>;
    if constexpr (LPR <= 16) {
        return group_sum<LPR, PAIRED>(part[0]);
    } else if constexpr (LPR == 32) {
        float v = part[0], w = N > 1 ? part[1] : 0.0f;            // the classes of the lower and of the upper half-wave
#pragma unroll
        for (int k = 2; k < N; ++k) (k % 2 ? w : v) += part[k];
        return group_sum<32, PAIRED>(N > 1 ? v + w : v);
    } else {
        float v = part[0];
        if constexpr (LPR == 256) {
            buf[threadIdx.x] = v;
            __syncthreads();
            const int lane = threadIdx.x % kWave;
            v = buf[lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) v += buf[lane + w * kWave];
        } else {
#pragma unroll
            for (int k = 1; k < N; ++k) v += part[k];
        }
        v = group_sum<16, PAIRED>(half_waves_sum(v));
        const int iv = __builtin_bit_cast(int, v);
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 0)) + __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16));
    }
}

// fp32 rows in lane pairs (LanePacks; groups of 8 lanes) or with pack = lane.  Both forms add in the order of the packs, so a row's bits do not depend on the choice:
// ln_fwd_paired and ln_bwd_paired say which is faster.
//
// Raw packs of row r for this lane (zeros where the row or the pack does not exist).
// Loads only, no arithmetic: every load of the row is in flight before the first use.
// NT: past the caches; not for gamma, beta and bias, which every workgroup reads (past the caches they were fetched anew by each: forward
// 16384 x 1024 bf16 16.7 us, 14.3 from the caches, 1000 x 1024 4.0 / 3.2, 4096 x 4096 f32 36.7 / 31.0; fused 8192 x 1280 bf16 17.9 / 16.8; inputs cold).
template <typename T, int LPR, int VPL, bool NT>
__device__ __forceinline__ void ln_load_row(RawPack<T> (&raw)[VPL], const T* __restrict__ base, int64_t r, bool rv,
                                            int hidden, int nv, int sub)
{
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        const int idx = sub + k * LPR;
        if (rv && idx < nv) raw[k] = load_raw<T, NT>(base + r * hidden + idx * kPack);
        else raw[k] = zero_raw<T>();
    }
}

// The same as the lanes of P hold it: to be settled before use
template <typename P, typename T, int LPR, int VPL, bool NT>
__device__ __forceinline__ void ln_load_packs(RawPack<T> (&raw)[VPL], const T* __restrict__ base, int64_t r, bool rv, int hidden, int nv, int sub)
{
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        const int idx = sub + k * LPR;
        raw[k] = P::template load<NT>(base + r * hidden + idx * kPack, rv && idx < nv);
    }
}

// What the fused variants add around the LayerNorm (all unused, and compiled out, otherwise).
template <typename T>
struct BdrFuse {
    T* out;               // forward: h = residual + Dropout(x + bias), stored;  backward: dx of the projection
    const T* residual;    // forward only
    const T* bias;        // forward only, nullable
    DropoutParams d;
};

// FUSE: the row that is normalised is h = residual + Dropout(x + bias), built in registers from
// two loads, stored once (the next residual) and normalised from its STORED (rounded) value, so the
// result equals bias+dropout+residual followed by LayerNorm bit for bit while h is never re-read.
template <typename T, int LPR, int VPL, bool FUSE, bool DROP, bool PAIR, bool NT>
__global__ __launch_bounds__(256) void ln_fwd_kernel(T* __restrict__ y, float* __restrict__ mean,
                                                     float* __restrict__ rstd, const T* __restrict__ x,
                                                     const T* __restrict__ gamma, const T* __restrict__ beta,
                                                     int64_t rows, int hidden, float eps, BdrFuse<T> fz)
{
    static_assert(LPR <= 256, "a row is at most a workgroup");
    __shared__ float lds[2][LPR == 256 ? 256 : 1];     // in turn: sum, squares (a barrier lies between two writes of either)
    constexpr int RPB = 256 / LPR;                     // rows a workgroup handles at a time
    constexpr int NP = kLnParts<LPR, VPL>;
    using P = LanePacks<T, PAIR ? 8 : 1>;
    const int sub = P::pack(threadIdx.x % LPR);
    const int slot = threadIdx.x / LPR;
    const int nv = hidden / kPack;
    const float inv_h = 1.0f / static_cast<float>(hidden);
    const int64_t gstride = static_cast<int64_t>(gridDim.x) * RPB;

    RawPack<T> gm[VPL], bt[VPL];              // gamma/beta stay packed; widened where used
    ln_load_row<T, LPR, VPL, false>(gm, gamma, 0, true, hidden, nv, sub);
    ln_load_row<T, LPR, VPL, false>(bt, beta, 0, true, hidden, nv, sub);

    RawPack<T> bs[FUSE ? VPL : 1];
    if constexpr (FUSE) {
        if (fz.bias) ln_load_row<T, LPR, VPL, false>(bs, fz.bias, 0, true, hidden, nv, sub);
        else {
#pragma unroll
            for (int k = 0; k < VPL; ++k) bs[k] = zero_raw<T>();
        }
    }

    int64_t base = static_cast<int64_t>(blockIdx.x) * RPB;
    RawPack<T> nxt[VPL], nres[FUSE ? VPL : 1];
    ln_load_packs<P, T, LPR, VPL, NT>(nxt, x, base + slot, base + slot < rows, hidden, nv, sub);
    if constexpr (FUSE) ln_load_packs<P, T, LPR, VPL, NT>(nres, fz.residual, base + slot, base + slot < rows, hidden, nv, sub);
    for (; base < rows; base += gstride) {
        const int64_t r = base + slot;
        const bool rv = r < rows;
        RawPack<T> cur[VPL], cres[FUSE ? VPL : 1];
#pragma unroll
        for (int k = 0; k < VPL; ++k) cur[k] = P::settle(nxt[k]);
        if constexpr (FUSE) {
#pragma unroll
            for (int k = 0; k < VPL; ++k) cres[k] = P::settle(nres[k]);
        }
        if (base + gstride < rows) {          // prefetch the next row group while this one is reduced
            ln_load_packs<P, T, LPR, VPL, NT>(nxt, x, r + gstride, r + gstride < rows, hidden, nv, sub);
            if constexpr (FUSE)
                ln_load_packs<P, T, LPR, VPL, NT>(nres, fz.residual, r + gstride, r + gstride < rows, hidden, nv, sub);
        }
        if constexpr (FUSE) {
            // same expressions as the stand-alone bias+dropout+residual kernel; the pack index of
            // the dropout stream is the flat one (row * packs per row + pack)
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const int idx = sub + k * LPR;
                const bool ok = rv && idx < nv;
                if (P::kPaired ? rv && (idx & ~7) < nv : ok) {       // (whole groups of lanes; absent packs stay zeros)
                    float xf[8], rf[8], b8[8], kf[8];
                    unpack<T>(cur[k], xf);
                    unpack<T>(cres[k], rf);
                    unpack<T>(bs[k], b8);
                    if constexpr (DROP) dropout_factors8(fz.d, static_cast<uint64_t>(r) * nv + idx, kf);
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float z = xf[j] + b8[j];
                        rf[j] = DROP ? fmaf(z, kf[j], rf[j]) : rf[j] + z;
                    }
                    pin_f32(rf);              // rounds like the stand-alone bias+dropout+residual kernel
                    if (!P::kPaired || ok) cur[k] = pack_raw<T>(rf);
                    P::template store<NT>(fz.out + r * hidden + idx * kPack, cur[k], ok);
                }
            }
        }

        float xv[VPL][8];
        float part[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) part[k] = 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            unpack<T>(cur[k], xv[k]);         // absent packs are zeros: they add nothing
#pragma unroll
            for (int j = 0; j < 8; ++j) part[k % NP] += xv[k][j];
        }
        const float mu = ln_row_total<LPR, VPL, P::kPaired>(part, lds[0]) * inv_h;
#pragma unroll
        for (int k = 0; k < NP; ++k) part[k] = 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const bool ok = sub + k * LPR < nv;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float dlt = xv[k][j] - mu;
                xv[k][j] = dlt;
                part[k % NP] = ok ? fmaf(dlt, dlt, part[k % NP]) : part[k % NP];
            }
        }
        const float q = ln_row_total<LPR, VPL, P::kPaired>(part, lds[1]);
        const float rs = 1.0f / sqrtf(fmaf(q, inv_h, eps));
        if (rv && sub == 0) {
            mean[r] = mu;
            rstd[r] = rs;
        }
        T* yr = y + r * hidden;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            const bool ok = rv && idx < nv;
            if (P::kPaired ? rv && (idx & ~7) < nv : ok) {
                float o[8], g8[8], b8[8];
                unpack<T>(gm[k], g8);
                unpack<T>(bt[k], b8);
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] = fmaf(xv[k][j] * rs, g8[j], b8[j]);
                pin_f32(o);                   // the fused and the plain kernel round alike
                P::template store<NT>(yr + idx * kPack, o, ok);
            }
        }
    }
}

constexpr int kLnBwdThreads = 256;

template <int LPR>
__device__ __forceinline__ float row_sum(float v, float* lds)
{
    if constexpr (LPR >= 256) return block_allreduce<LPR / 64, OpSum>(v, lds);      // the row spans the workgroup
    else return group_sum<LPR>(v);
}

// partial: [gridDim.x][2][hidden] fp32 (dgamma row, then dbeta row).
// THREADS lanes per workgroup: THREADS/LPR rows in flight per workgroup (plus their
// prefetched successors).  Serves rows of up to 504 columns (a row within a wave, one pack per lane or two: 8000 x 256 fused 9.8 us,
// as with ln_bwd_span_kernel's shape) and those of 8193..16384.
// FUSE: the LayerNorm gradient (plus dres) is the gradient of h = residual + Dropout(x + bias): it is
// stored (the residual branch's gradient), then masked and scaled from its STORED value into
// fz.out (the projection's gradient), whose column sums (dbias) join dgamma/dbeta as a third
// partial row.  Equal to LayerNorm backward followed by bias+dropout+residual backward, one pass.
// Rows wider than 8192 columns take one 1024-thread workgroup per row, which leaves a thread 128
// registers: too few for the row, its prefetched successor and the column accumulators.  There the
// accumulators live in LDS instead, each thread reading and writing only its own columns' entries
// (131 KB for 16384 columns: no barrier, no conflict, and the LDS traffic hides behind the row
// stream).
// NT: past the caches
template <typename T, int LPR, int VPL, bool HAS_RES, int THREADS, bool FUSE, bool DROP, bool NT>
__global__ __launch_bounds__(THREADS) void ln_bwd_kernel(T* dx, float* __restrict__ partial, const T* dy,
                                                         const T* __restrict__ x, const T* __restrict__ gamma,
                                                         const float* __restrict__ mean, const float* __restrict__ rstd,
                                                         const T* dres, int64_t rows, int hidden, BdrFuse<T> fz)
{
    constexpr int NACC = FUSE ? 3 : 2;        // column accumulators: dgamma, dbeta (, dbias)
    constexpr bool kColsInLds = LPR > 256;
    extern __shared__ float colbuf[];         // [NACC][8][packs | 1]: the slots' exchange, or the accumulators themselves when LPR > 256
    __shared__ float lds[16];
    static_assert(LPR <= 64 || THREADS == LPR, "a whole-workgroup row takes the whole workgroup");
    constexpr int RPB = THREADS / LPR;
    const int sub = threadIdx.x % LPR;
    const int slot = threadIdx.x / LPR;
    const int nv = hidden / kPack;
    const float inv_h = 1.0f / static_cast<float>(hidden);
    const int64_t gstride = static_cast<int64_t>(gridDim.x) * RPB;

    RawPack<T> gm[VPL];
    ln_load_row<T, LPR, VPL, false>(gm, gamma, 0, true, hidden, nv, sub);
    float dg[VPL][8], db[VPL][8], dbi[FUSE ? VPL : 1][8];
#pragma unroll
    for (int k = 0; k < VPL; ++k)
#pragma unroll
        for (int j = 0; j < 8; ++j) { dg[k][j] = 0.0f; db[k][j] = 0.0f; }
    if constexpr (FUSE) {
#pragma unroll
        for (int k = 0; k < VPL; ++k)
#pragma unroll
            for (int j = 0; j < 8; ++j) dbi[k][j] = 0.0f;
    }

    const int cstride = nv | 1;               // odd: consecutive lanes fall in consecutive banks
    if constexpr (kColsInLds) {
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            if (idx < nv) {
#pragma unroll
                for (int j = 0; j < 16; ++j) colbuf[j * cstride + idx] = 0.0f;
            }
        }
    }

    int64_t base = static_cast<int64_t>(blockIdx.x) * RPB;
    RawPack<T> ndy[VPL], nx[VPL], nres[HAS_RES ? VPL : 1];
    float nmu = 0.0f, nrs = 0.0f;
    {
        const int64_t r = base + slot;
        const bool rv = r < rows;
        ln_load_row<T, LPR, VPL, NT>(ndy, dy, r, rv, hidden, nv, sub);
        ln_load_row<T, LPR, VPL, NT>(nx, x, r, rv, hidden, nv, sub);
        if constexpr (HAS_RES) ln_load_row<T, LPR, VPL, NT>(nres, dres, r, rv, hidden, nv, sub);
        if (rv) { nmu = mean[r]; nrs = rstd[r]; }
    }
    for (; base < rows; base += gstride) {
        const int64_t r = base + slot;
        const bool rv = r < rows;
        const int64_t ro = r * hidden;
        RawPack<T> cdy[VPL], cx[VPL], cres[HAS_RES ? VPL : 1];
#pragma unroll
        for (int k = 0; k < VPL; ++k) { cdy[k] = ndy[k]; cx[k] = nx[k]; }
        if constexpr (HAS_RES) {
#pragma unroll
            for (int k = 0; k < VPL; ++k) cres[k] = nres[k];
        }
        const float mu = nmu, rs = nrs;
        if (base + gstride < rows) {          // prefetch the next row group
            const int64_t rn = r + gstride;
            const bool rnv = rn < rows;
            ln_load_row<T, LPR, VPL, NT>(ndy, dy, rn, rnv, hidden, nv, sub);
            ln_load_row<T, LPR, VPL, NT>(nx, x, rn, rnv, hidden, nv, sub);
            if constexpr (HAS_RES) ln_load_row<T, LPR, VPL, NT>(nres, dres, rn, rnv, hidden, nv, sub);
            nmu = 0.0f; nrs = 0.0f;
            if (rnv) { nmu = mean[rn]; nrs = rstd[rn]; }
        }

        // pass 1 over registers: the two row sums and the column accumulators.  Absent packs
        // hold dy = 0, so they add nothing to any of the sums.  xhat = x*rstd - mean*rstd.
        const float nmr = -mu * rs;
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            float gy[8], xv[8], g8[8];
            unpack<T>(cdy[k], gy);
            unpack<T>(cx[k], xv);
            unpack<T>(gm[k], g8);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float xhat = fmaf(xv[j], rs, nmr);
                if constexpr (!kColsInLds) {
                    dg[k][j] = fmaf(gy[j], xhat, dg[k][j]);
                    db[k][j] += gy[j];
                } else {
                    if (sub + k * LPR < nv) {              // rows that do not exist hold dy = 0 and add nothing
                        float* a = colbuf + j * cstride + (sub + k * LPR);
                        a[0] = fmaf(gy[j], xhat, a[0]);
                        a[8 * cstride] += gy[j];
                    }
                }
                const float gg = gy[j] * g8[j];
                s1 += gg;
                s2 = fmaf(gg, xhat, s2);
            }
        }
        s1 = row_sum<LPR>(s1, lds);
        s2 = row_sum<LPR>(s2, lds);
        // dx = rstd*(g - (s1 + xhat*s2)/hidden) = g*rstd + xhat*c1 + c0
        const float c0 = -rs * s1 * inv_h, c1 = -rs * s2 * inv_h;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            if (rv && idx < nv) {
                float o[8];
                if constexpr (HAS_RES) unpack<T>(cres[k], o);
                // xhat and gamma*dy are rebuilt from the packed row (a few flops) rather than kept
                // in 16 more registers per pack across the reduction
                opaque<T>(cdy[k]);
                opaque<T>(cx[k]);
                float gy[8], xv[8], g8[8];
                unpack<T>(cdy[k], gy);
                unpack<T>(cx[k], xv);
                unpack<T>(gm[k], g8);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float v = fmaf(gy[j] * g8[j], rs, fmaf(fmaf(xv[j], rs, nmr), c1, c0));
                    o[j] = HAS_RES ? o[j] + v : v;
                }
                pin_f32(o);               // the fused and the plain kernel round alike
                if constexpr (!FUSE) {
                    store8<T, NT>(dx + ro + idx * kPack, o);
                } else {
                    const RawPack<T> hp = pack_raw<T>(o);
                    store_raw<T, NT>(dx + ro + idx * kPack, hp);
                    float gq[8];
                    unpack<T>(hp, gq);
                    if constexpr (DROP) {
                        float kf[8];
                        dropout_factors8(fz.d, static_cast<uint64_t>(r) * nv + idx, kf);
#pragma unroll
                        for (int j = 0; j < 8; ++j) gq[j] *= kf[j];
                    }
                    pin_f32(gq);
                    store8<T, NT>(fz.out + ro + idx * kPack, gq);
#pragma unroll
                    for (int j = 0; j < 8; ++j) dbi[k][j] += gq[j];
                }
            }
        }
    }

    float* prow = partial + static_cast<int64_t>(blockIdx.x) * NACC * hidden;
    if constexpr (kColsInLds) {
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            if (idx < nv) {
                float a[8], b[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) { a[j] = colbuf[j * cstride + idx]; b[j] = colbuf[(8 + j) * cstride + idx]; }
                store8<float>(prow + idx * kPack, a);
                store8<float>(prow + hidden + idx * kPack, b);
            }
        }
    } else {
        // Sum the RPB row slots in slot order through LDS.  Layout [dgamma|dbeta(|dbias)][j][pack] with
        // an odd pack stride: consecutive lanes (consecutive packs) fall in consecutive banks.  A
        // [column] layout would put the lanes of a wave 8 floats apart: a 16-way bank conflict.
        const int stride = nv | 1;
        // every slot has its own copy: all slots write at once, one barrier, then all threads
        // add the RPB copies of their columns in slot order (same sums as taking turns)
        const int per_slot = NACC * 8 * stride;
        float* mine = colbuf + slot * per_slot;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            if (idx < nv) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    mine[j * stride + idx] = dg[k][j];
                    mine[8 * stride + j * stride + idx] = db[k][j];
                    if constexpr (FUSE) mine[16 * stride + j * stride + idx] = dbi[k][j];
                }
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < NACC * hidden; c += THREADS) {
            const int which = c / hidden;
            const int cc = c - which * hidden;
            const int off = which * 8 * stride + (cc & 7) * stride + (cc >> 3);
            float t = colbuf[off];
#pragma unroll
            for (int sl = 1; sl < RPB; ++sl) t += colbuf[sl * per_slot + off];
            prow[c] = t;
        }
    }
}

// Rows of 512..8192 columns: a row spans LR lanes (a multiple of 32, several waves for all but 512 columns) and every lane
// owns ONE pack of columns, so a lane keeps 16 or 24 column accumulators instead of 16-24 per pack held and a thread needs
// 81-126 registers (RAG: 116-158).  With a whole row per wave (up to 264 registers, one wave per
// SIMD) nothing overlapped a row's chain of loads, two reductions, dropout draw and stores.  A workgroup, one per compute unit, holds
// `slots` rows at a time; the waves of a row meet in LDS once per row: every 32 lanes leave their two sums, a barrier, then
// every 32 lanes read all of them (at most 32) back with one access and add them by DPP.  Two buffers make the one
// barrier enough: a buffer is written again only behind the next row's barrier.  The next row is loaded ahead, the dropout
// words are drawn between the reductions and the barrier, where they fill the wait for the slowest wave.  No lane shares its
// columns with another lane of its row, so the epilogue only adds the slots (a tree over LDS, fixed order).
// Fused with dropout and residual gradient, bf16 8192 x 1280: 27.8 -> 23.1 us, 3000 x 3072: 38 -> 21; plain 2600 x 2048: 14.0 -> 10.8;
// f32 fused 4000 x 1280: 27.5 -> 23.9 (second stage not counted).  The copy of the bytes takes 17 us at 8192 x 1280.  Counters there / at
// 8192 x 1024 fp16 / 2100 x 512 f32: 2.5 / 2 / 0.75 waves per SIMD, which wait for memory, LDS or the barrier in 61 / 55 / 65 % of their life
// and for issue in 13 / 15 / 5 %; vector ALU busy 32 / 23 / 5 %, memory units stalled 0.4 / 0.2 / 0.2 %.  So it is still a row's chain, with
// too few rows beside it, most of all in short calls.
// LRC = 64: 512 columns, a row per wave, no exchange, never in pairs (300 rows f32 6.3 us, in pairs 6.6).  Partial rows as ln_bwd_kernel's.
// RAG: rows that are not whole packs, in packs counted from the row's start (RowPackIO; not fused).
template <typename T, int LRC, bool HAS_RES, int MAXT, bool FUSE, bool DROP, bool RAG, bool PAIR, bool NT>
__global__ __launch_bounds__(MAXT) void ln_bwd_span_kernel(T* dx, float* __restrict__ partial, const T* dy,
                                                           const T* __restrict__ x, const T* __restrict__ gamma,
                                                           const float* __restrict__ mean, const float* __restrict__ rstd,
                                                           const T* dres, int64_t rows, int hidden, int lanes, BdrFuse<T> fz)
{
    static_assert(!RAG || !FUSE, "the fused boundary is for rows of whole packs");
    constexpr int NACC = FUSE ? 3 : 2;        // column accumulators: dgamma, dbeta (, dbias)
    extern __shared__ float span_lds[];       // the rows' exchange [2][32-lane groups][2], later the slots' [slots / 2][NACC * 8][lanes]
    const int LR = LRC ? LRC : lanes;
    const int slots = blockDim.x / LR;
    static_assert(!PAIR || (sizeof(T) == 4 && !RAG && LRC == 0), "lane pairs are for fp32 rows of whole packs that span several waves");
    using P = LanePacks<T, PAIR ? 32 : 1>;
    const int slot = threadIdx.x / LR, sub = P::pack(threadIdx.x - slot * LR);
    const RowPackIO<T, RAG> io(hidden);
    const int nv = io.ppr;
    const bool on = sub < nv;
    const float inv_h = 1.0f / static_cast<float>(hidden);
    const int64_t gstride = static_cast<int64_t>(gridDim.x) * slots;

    float g8[8];
    unpack<T>(on ? io.template load<false>(gamma, 0, sub) : zero_raw<T>(), g8);
    float acc[NACC][8];
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[a][j] = 0.0f;

    RawPack<T> ndy, nx, nres;
    float nmu, nrs;
    auto fetch = [&](int64_t r) {             // zeros where the row or the pack does not exist
        ndy = zero_raw<T>(); nx = zero_raw<T>();
        if constexpr (HAS_RES) nres = zero_raw<T>();
        nmu = 0.0f; nrs = 0.0f;
        if (r < rows) {
            if constexpr (P::kPaired) {
                ndy = P::template load<NT>(dy + io.element(r, sub), on);
                nx = P::template load<NT>(x + io.element(r, sub), on);
                if constexpr (HAS_RES) nres = P::template load<NT>(dres + io.element(r, sub), on);
            } else if (on) {
                ndy = io.template ahead<NT>(dy, r, sub);
                nx = io.template ahead<NT>(x, r, sub);
                if constexpr (HAS_RES) nres = io.template ahead<NT>(dres, r, sub);
            }
            nmu = mean[r]; nrs = rstd[r];
        }
    };
    auto settle = [&](const RawPack<T>& v) {
        if constexpr (P::kPaired) return P::settle(v);
        else return io.settle(v, sub);
    };
    int64_t base = static_cast<int64_t>(blockIdx.x) * slots;
    fetch(base + slot);
    float* sums = span_lds;                   // of this row; the other buffer next
    float* other = span_lds + blockDim.x / 16;
    // Packs at any alignment with a residual gradient take 144 registers (fp32 158) with the next row loaded ahead; a 1024-thread workgroup
    // has 128 and spilt 17 (46) of them: 700 x 6145 f32 54 us against 34 on the generic path.  Loaded behind the row, 4 (15) are spilt:
    // 32.8 us, 700 x 7001 fp16 25.0 (before 37.1, generic 38.2).
    constexpr bool AHEAD = !(RAG && HAS_RES && MAXT > kLnSpanThreads);
    for (; base < rows; base += gstride) {    // the same trips for every thread
        const int64_t r = base + slot;
        const RawPack<T> cdy = ndy, cx = nx, cres = nres;
        const float mu = nmu, rs = nrs;
        if (AHEAD && base + gstride < rows) fetch(r + gstride);

        // the two row sums and the column sums; absent packs and rows hold dy = 0
        const float nmr = -mu * rs;
        float gy[8], xh[8], s1 = 0.0f, s2 = 0.0f;
        unpack<T>(settle(cdy), gy);
        unpack<T>(settle(cx), xh);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            xh[j] = fmaf(xh[j], rs, nmr);
            acc[0][j] = fmaf(gy[j], xh[j], acc[0][j]);
            acc[1][j] += gy[j];
            gy[j] *= g8[j];
            s1 += gy[j];
            s2 = fmaf(gy[j], xh[j], s2);
        }
        uint32_t w[4];
        if constexpr (LRC == 64) {
            s1 = group_sum<64>(s1);
            s2 = group_sum<64>(s2);
        } else {
            s1 = PAIR ? paired_half_wave_sum(s1) : group_sum<32>(s1);
            s2 = PAIR ? paired_half_wave_sum(s2) : group_sum<32>(s2);
            if ((threadIdx.x & 31) == 0) {
                sums[threadIdx.x / 16] = s1;
                sums[threadIdx.x / 16 + 1] = s2;
            }
        }
        if constexpr (FUSE && DROP) {
            const uint64_t g = static_cast<uint64_t>(r) * nv + sub;
            philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), fz.d.ctr2, fz.d.ctr3, fz.d.key0, fz.d.key1, w);
#pragma unroll
            for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(w[j]));      // drawn here, not behind the barrier
        }
        if constexpr (LRC != 64) {
            __syncthreads();
            const int l = threadIdx.x & 31, groups = LR / 32, at = 2 * (slot * groups + (l < groups ? l : 0));
            s1 = group_sum<32>(l < groups ? sums[at] : 0.0f);
            s2 = group_sum<32>(l < groups ? sums[at + 1] : 0.0f);
            float* t = sums; sums = other; other = t;
        }
        // dx = rstd*(g - (s1 + xhat*s2)/hidden) = g*rstd + xhat*c1 + c0
        const float c0 = -rs * s1 * inv_h, c1 = -rs * s2 * inv_h;
        if (r < rows && (P::kPaired || on)) {
            float o[8];
            if constexpr (HAS_RES) unpack<T>(settle(cres), o);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float v = fmaf(gy[j], rs, fmaf(xh[j], c1, c0));
                o[j] = HAS_RES ? o[j] + v : v;
            }
            pin_f32(o);                       // the fused and the plain kernel round alike
            const RawPack<T> hp = pack_raw<T>(o);
            if constexpr (P::kPaired) P::template store<NT>(dx + io.element(r, sub), o, on);
            else io.template put<NT>(dx, r, sub, hp);
            if constexpr (FUSE) {
                float gq[8];
                unpack<T>(hp, gq);
                if constexpr (DROP) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        gq[2 * j] *= (w[j] & 0xFFFFu) >= fz.d.t16 ? fz.d.scale : 0.0f;
                        gq[2 * j + 1] *= (w[j] >> 16) >= fz.d.t16 ? fz.d.scale : 0.0f;
                    }
                }
                pin_f32(gq);
                if constexpr (P::kPaired) P::template store<NT>(fz.out + io.element(r, sub), gq, on);
                else store8<T, NT>(fz.out + io.element(r, sub), gq);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[2][j] += gq[j];
            }
        }
        if (!AHEAD && base + gstride < rows) fetch(r + gstride);
    }

    for (int left = slots; left > 1;) {       // slot k takes slot k + half, until one is left
        const int half = (left + 1) / 2;
        __syncthreads();                      // the exchange, or the step before, has been read
        if (slot >= half && slot < left) {
            float* m = span_lds + (slot - half) * NACC * 8 * LR + sub;
#pragma unroll
            for (int a = 0; a < NACC * 8; ++a) m[a * LR] = acc[a / 8][a % 8];
        }
        __syncthreads();
        if (slot + half < left) {
            const float* m = span_lds + slot * NACC * 8 * LR + sub;
#pragma unroll
            for (int a = 0; a < NACC * 8; ++a) acc[a / 8][a % 8] += m[a * LR];
        }
        left = half;
    }
    if (slot == 0 && on) {
        float* prow = partial + static_cast<int64_t>(blockIdx.x) * NACC * hidden + sub * kPack;
#pragma unroll
        for (int a = 0; a < NACC; ++a) {
            if constexpr (RAG) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (sub * kPack + j < hidden) prow[a * hidden + j] = acc[a][j];
            } else {
                store8<float>(prow + a * hidden, acc[a]);
            }
        }
    }
}

// Forward of rows that are not whole packs: a row over LR lanes, one pack per lane, as in ln_bwd_span_kernel; mean and variance are
// two exchanges through LDS (their buffers alternate, so a barrier each is enough).  Forward / backward with residual gradient in us, one wave or
// workgroup per row with element accesses in brackets: 8192 x 1281 bf16 13.2 / 27.7 (23.5 / 54.9), 3000 x 1999 f32 10.8 / 28.2 (32.6 / 50.9),
// 600 x 7001 fp16 11.2 / 39.8 (21.0 / 44.6), 6000 x 300 5.8 / 11.4 (6.2 / 25.9), 500 x 259 f32 3.3 / 7.8 (3.5 / 12.2).
template <typename T, int MAXT>
__global__ __launch_bounds__(MAXT) void ln_fwd_rag_kernel(T* __restrict__ y, float* __restrict__ mean, float* __restrict__ rstd,
                                                          const T* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
                                                          int64_t rows, int hidden, float eps, int LR)
{
    __shared__ float sums[2][MAXT / 32];
    const RowPackIO<T, true> io(hidden);
    const int slots = blockDim.x / LR, slot = threadIdx.x / LR, sub = threadIdx.x - slot * LR;
    const bool on = sub < io.ppr;
    const int left = on ? hidden - sub * kPack : 0;                // columns of this pack, 8 or more but for the last
    const float inv_h = 1.0f / static_cast<float>(hidden);
    const int64_t gstride = static_cast<int64_t>(gridDim.x) * slots;
    auto total = [&](float v, float* buf) {
        v = group_sum<32>(v);
        if (LR == 32) return v;                                    // a row within a wave: the same additions without LDS and barrier
        if (LR == 64) return half_waves_sum(v);
        if ((threadIdx.x & 31) == 0) buf[threadIdx.x / 32] = v;
        __syncthreads();
        const int l = threadIdx.x & 31, groups = LR / 32;
        return group_sum<32>(l < groups ? buf[slot * groups + l] : 0.0f);
    };
    const RawPack<T> gm = on ? io.template ahead<false>(gamma, 0, sub) : zero_raw<T>(), bt = on ? io.template ahead<false>(beta, 0, sub) : zero_raw<T>();
    int64_t base = static_cast<int64_t>(blockIdx.x) * slots;
    RawPack<T> nxt = base + slot < rows && on ? io.template ahead<kNT>(x, base + slot, sub) : zero_raw<T>();
    for (; base < rows; base += gstride) {                         // the same trips for every thread
        const int64_t r = base + slot;
        const RawPack<T> cur = nxt;
        if (r + gstride < rows && on) nxt = io.template ahead<kNT>(x, r + gstride, sub);
        float v[8], s = 0.0f, q = 0.0f;
        unpack<T>(io.settle(cur, sub), v);                         // absent columns are zeros: they add nothing to the sum
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
        const float mu = total(s, sums[0]) * inv_h;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            v[j] -= mu;
            q = j < left ? fmaf(v[j], v[j], q) : q;
        }
        const float rs = 1.0f / sqrtf(fmaf(total(q, sums[1]), inv_h, eps));
        if (r < rows && on) {
            if (sub == 0) { mean[r] = mu; rstd[r] = rs; }
            float o[8], g8[8], b8[8];
            unpack<T>(io.settle(gm, sub), g8);
            unpack<T>(io.settle(bt, sub), b8);
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = fmaf(v[j] * rs, g8[j], b8[j]);
            io.template store<kNT>(y, r, sub, o);
        }
    }
}

// ---- generic path: any hidden; TH = 64 (one wave per row) or 256 lanes (one workgroup per row: rows beyond the
// register buckets), rows re-read from cache
// PACKS: the row is a whole number of packs (rows beyond 16384 columns), walked in 128-bit accesses.
template <typename T, int TH, bool PACKS>
__global__ __launch_bounds__(256) void ln_fwd_generic(T* __restrict__ y, float* __restrict__ mean,
                                                      float* __restrict__ rstd, const T* __restrict__ x,
                                                      const T* __restrict__ gamma, const T* __restrict__ beta,
                                                      int64_t rows, int hidden, float eps)
{
    __shared__ float lds[4];
    constexpr int W = PACKS ? kPack : 1;       // elements per access
    const int lane = threadIdx.x % TH;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * (256 / TH) + threadIdx.x / TH;
    if (r >= rows) return;                     // whole waves (TH = 64) or the whole workgroup (TH = 256) leave together
    auto row_total = [&](float v) {
        if constexpr (TH == 64) return group_sum<64>(v);
        else return block_allreduce<4, OpSum>(v, lds);
    };
    auto get = [&](const T* p, float (&f)[W]) {
        if constexpr (PACKS) load8<T>(p, f);
        else f[0] = to_f32<T>(p[0]);
    };
    const T* xr = x + r * hidden;
    const float inv_h = 1.0f / static_cast<float>(hidden);
    float s = 0.0f;
    for (int i = lane * W; i < hidden; i += TH * W) {
        float v[W];
        get(xr + i, v);
#pragma unroll
        for (int j = 0; j < W; ++j) s += v[j];
    }
    const float mu = row_total(s) * inv_h;
    float q = 0.0f;
    for (int i = lane * W; i < hidden; i += TH * W) {
        float v[W];
        get(xr + i, v);
#pragma unroll
        for (int j = 0; j < W; ++j) { const float d = v[j] - mu; q = fmaf(d, d, q); }
    }
    const float rs = 1.0f / sqrtf(fmaf(row_total(q), inv_h, eps));
    if (lane == 0) { mean[r] = mu; rstd[r] = rs; }
    T* yr = y + r * hidden;
    for (int i = lane * W; i < hidden; i += TH * W) {
        float v[W], gm[W], bt[W];
        get(xr + i, v);
        get(gamma + i, gm);
        get(beta + i, bt);
#pragma unroll
        for (int j = 0; j < W; ++j) v[j] = fmaf((v[j] - mu) * rs, gm[j], bt[j]);
        if constexpr (PACKS) store8<T>(yr + i, v);
        else yr[i] = from_f32<T>(v[0]);
    }
}

template <typename T, int TH, bool PACKS>
__global__ __launch_bounds__(256) void ln_bwd_generic(T* dx, const T* dy, const T* __restrict__ x,
                                                      const T* __restrict__ gamma, const float* __restrict__ mean,
                                                      const float* __restrict__ rstd, const T* dres,
                                                      int64_t rows, int hidden)
{
    __shared__ float lds[4];
    constexpr int W = PACKS ? kPack : 1;
    const int lane = threadIdx.x % TH;
    const int64_t r = static_cast<int64_t>(blockIdx.x) * (256 / TH) + threadIdx.x / TH;
    if (r >= rows) return;
    auto row_total = [&](float v) {
        if constexpr (TH == 64) return group_sum<64>(v);
        else return block_allreduce<4, OpSum>(v, lds);
    };
    auto get = [&](const T* p, float (&f)[W]) {
        if constexpr (PACKS) load8<T>(p, f);
        else f[0] = to_f32<T>(p[0]);
    };
    const int64_t ro = r * hidden;
    const float mu = mean[r], rs = rstd[r];
    const float inv_h = 1.0f / static_cast<float>(hidden);
    float s1 = 0.0f, s2 = 0.0f;
    for (int i = lane * W; i < hidden; i += TH * W) {
        float gy[W], xv[W], gm[W];
        get(dy + ro + i, gy);
        get(x + ro + i, xv);
        get(gamma + i, gm);
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const float gg = gy[j] * gm[j];
            s1 += gg;
            s2 = fmaf(gg, (xv[j] - mu) * rs, s2);
        }
    }
    const float a = row_total(s1) * inv_h, b = row_total(s2) * inv_h;
    for (int i = lane * W; i < hidden; i += TH * W) {
        float gy[W], xv[W], gm[W], rv[W];
        get(dy + ro + i, gy);
        get(x + ro + i, xv);
        get(gamma + i, gm);
        if (dres) get(dres + ro + i, rv);
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const float gg = gy[j] * gm[j];
            const float xhat = (xv[j] - mu) * rs;
            float v = rs * (gg - fmaf(xhat, b, a));
            if (dres) v += rv[j];
            gy[j] = v;
        }
        if constexpr (PACKS) store8<T>(dx + ro + i, gy);
        else dx[ro + i] = from_f32<T>(gy[0]);
    }
}

// dgamma/dbeta for the generic path, first stage: one thread per column, gridDim.y row
// blocks that each walk every gridDim.y-th row (four rows in flight); partial[y] =
// [dgamma | dbeta] of block y, summed by colsum_finalize_kernel like the fast path's.
// Runs BEFORE ln_bwd_generic so that dx may alias dy.
template <typename T>
__global__ __launch_bounds__(256) void ln_dparams_generic(float* __restrict__ partial,
                                                          const T* __restrict__ dy, const T* __restrict__ x,
                                                          const float* __restrict__ mean, const float* __restrict__ rstd,
                                                          int64_t rows, int hidden)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= hidden) return;
    float sg = 0.0f, sb = 0.0f;
    const int64_t stride = gridDim.y;
    for (int64_t r0 = blockIdx.y; r0 < rows; r0 += 4 * stride) {
        float gy[4], xv[4], mu[4], rs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t r = r0 + u * stride;
            const bool ok = r < rows;
            gy[u] = ok ? to_f32<T>(dy[r * hidden + c]) : 0.0f;
            xv[u] = ok ? to_f32<T>(x[r * hidden + c]) : 0.0f;
            mu[u] = ok ? mean[r] : 0.0f;
            rs[u] = ok ? rstd[r] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            sg = fmaf(gy[u], (xv[u] - mu[u]) * rs[u], sg);
            sb += gy[u];
        }
    }
    float* prow = partial + static_cast<int64_t>(blockIdx.y) * 2 * hidden;
    prow[c] = sg;
    prow[hidden + c] = sb;
}

// The same first stage for rows of whole packs: one thread per PACK of 8 columns (128-bit
// loads), four rows in flight.  Serves the rows that are too wide for the column
// accumulators to stay in registers next to the row itself.
template <typename T>
__global__ __launch_bounds__(256) void ln_dparams_packed(float* __restrict__ partial,
                                                         const T* __restrict__ dy, const T* __restrict__ x,
                                                         const float* __restrict__ mean, const float* __restrict__ rstd,
                                                         int64_t rows, int hidden)
{
    const int idx = blockIdx.x * 256 + threadIdx.x;       // pack of the row
    if (idx >= hidden / kPack) return;
    float sg[8] = {0, 0, 0, 0, 0, 0, 0, 0}, sb[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t stride = gridDim.y;
    for (int64_t r0 = blockIdx.y; r0 < rows; r0 += 4 * stride) {
        RawPack<T> gy[4], xv[4];
        float mu[4], rs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t r = r0 + u * stride;
            const bool ok = r < rows;
            gy[u] = ok ? load_raw<T, false>(dy + r * hidden + idx * kPack) : zero_raw<T>();
            xv[u] = ok ? load_raw<T, false>(x + r * hidden + idx * kPack) : zero_raw<T>();
            mu[u] = ok ? mean[r] : 0.0f;
            rs[u] = ok ? rstd[r] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float g8[8], x8[8];
            unpack<T>(gy[u], g8);
            unpack<T>(xv[u], x8);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                sg[j] = fmaf(g8[j], (x8[j] - mu[u]) * rs[u], sg[j]);
                sb[j] += g8[j];
            }
        }
    }
    float* prow = partial + static_cast<int64_t>(blockIdx.y) * 2 * hidden;
    store8<float>(prow + idx * kPack, sg);
    store8<float>(prow + hidden + idx * kPack, sb);
}

constexpr int kLnWideLpr = 1024, kLnWideVpl = 2;      // the bucket of rows with 1025..2048 packs

// ------------------------------------------------------------------ dispatch
// Shape buckets: lanes per row and packs per lane for a row of nv packs.
struct LnShape { int lpr, vpl; };

inline LnShape ln_shape(int hidden)
{
    if (hidden % kPack != 0) return {0, 0};
    const int nv = hidden / kPack;
    // rows of up to 384 packs: lanes of one wave, the shape with the fewest idle lane slots; among
    // equals 32 lanes (two rows per wave) before 64.  256..1536 columns in steps of 256 fit 32 x 1..6
    // exactly, 2560 and 3072 fit 64 x 5 and 64 x 6.  Measured forward at 8192 rows, 32 x 4 against
    // 64 x 2 at 1024 columns: 8.3 against 9.1 us (fused with bias+dropout+residual 13.9 against 15.7);
    // 32 x 2 against 64 x 1 at 512: 5.6 against 6.2; 32 x 6 against 64 x 3 at 1536: 11.6 against 12.3.
    // (32 x 8 at 2048 helps the plain forward, 14.3 against 16.8 us, but costs the fused one 2 us: not built.)
    static const LnShape wave_shapes[] = {{32, 1}, {32, 2}, {32, 3}, {32, 4}, {32, 5}, {32, 6}, {64, 1}, {64, 2}, {64, 3},
                                          {64, 4}, {64, 5}, {64, 6}, {16, 1}, {8, 1}};
    if (nv <= 384) {
        LnShape best{0, 0};
        for (const LnShape& c : wave_shapes)
            if (c.lpr * c.vpl >= nv && (best.lpr == 0 || c.lpr * c.vpl < best.lpr * best.vpl)) best = c;
        return best;
    }
    if (nv <= 512) return {256, 2};
    if (nv <= 768) return {256, 3};       // 5120 columns: 640 of 768 pack slots in use (of 1024 as 256 x 4); 6144 fit exactly
    if (nv <= 1024) return {256, 4};
    if (nv <= 2048) return {kLnWideLpr, kLnWideVpl};     // hidden up to 16384: one large workgroup per row
    return {0, 0};
}

// Forward: the shape above, but more lanes per row (a shorter chain per row) where the calls are short or the shape leaves a lane
// four packs or more.  Measured, fused / plain: 512 x 512 f32 64 x 1 3.9 / 3.1 us, 32 x 2 4.7 / 3.2; 3000 x 1024 64 x 2 7.4 / 4.7, 32 x 4
// 7.7 / 5.1 (4096 rows 9.0 / 5.8 against 8.3 / 5.4: the line is between).  600 x 3072 256 x 2 6.0 / 4.3, 64 x 6 7.0 / 4.6; 600 x 2048 256 x 1
// 5.1 / 3.9, 64 x 4 5.6 / 4.1.  8192 x 2048 256 x 1 27.8 / 15.8, 64 x 4 29.6 / 17.4; 8192 x 2560 256 x 2 34.3 / 18.6, 64 x 5 35.8 / 19.0; rows that fill
// three quarters of such lanes or less stay (4096 x 3072 256 x 2 21.2 / 12.2, 64 x 6 22.2 / 11.2; 8192 x 1536 21.1 / 11.9 against 22.9 / 10.2),
// and so do those of 225..320 packs in 16 bits between 3073 and 5120 rows, where their one-row workgroups just overflow the compute
// units (4096 x 2560 256 x 2 20.7 / 13.1, 64 x 5 18.8 / 11.4; 3584 x 2048 256 x 1 15.3, 64 x 4 14.2).
// The shape changes with the number of rows: ln_row_total keeps a row's bits out of it.
inline LnShape ln_fwd_shape(int64_t rows, int hidden, int elem_bytes)
{
    const LnShape s = ln_shape(hidden);
    const int nv = hidden / kPack;
    if (s.lpr == 0 || s.lpr >= 256) return s;
    const bool overflow = elem_bytes == 2 && rows > 3072 && rows <= 5120;
    if (nv > 128 && nv <= 256 && ((nv > 224 && !overflow) || rows <= 1024)) return {256, 1};
    if (nv > 256 && ((nv <= 320 && !overflow) || rows <= 1024)) return {256, 2};
    if (s.lpr == 32 && s.vpl % 2 == 0 && rows <= 3072) return {64, s.vpl / 2};
    return s;
}

// fp32 forward in lane pairs: not the calls of a few waves, whose time is latency, which the exchange adds to, and of rows that end
// inside a 128-byte line, where two pieces meet, only those of up to 2048 columns that are neither small nor long (long ones fetch each line once through the caches).
// us, inputs cold: pack = lane past the caches / pairs everywhere / this rule: 8192 x 2048 33.4 / 25.5 / 25.5, fused with dropout 61.5 / 48.7 / 48.8; 300 x 1024 3.4 / 3.8 / 3.4,
// 4.7 / 4.9 / 4.5; 300 x 2304 4.5 / 5.0 / 4.7, 6.1 / 7.0 / 6.5; 8192 x 2040 35.7 / 37.3 / 29.9, 66.7 / 74.1 / 56.4; 3000 x 1304 11.6 / 10.0 / 9.7, 20.2 / 16.3 / 17.6.
// The fused shapes of four packs per lane and more take 256 registers and more in pairs, one wave per SIMD, and gain all the same (8192 x 4096 110 / 94 us) but
// where that leaves a short last round (600 x 8192 with dropout 21 / 23).  256 lanes x 8 packs would spill.
inline bool ln_fwd_paired(int64_t rows, int hidden)
{
    const int64_t n = rows * hidden;
    if (n < (hidden <= 2048 ? 3ll << 18 : 1ll << 20)) return false;
    return hidden % 32 == 0 || (hidden < 2048 && n < 7ll << 19);
}

// fp32 backward where a row spans several waves, in lane pairs (groups of 32) beyond half a Mi elements: below, the exchange is in a chain that nothing covers. us,
// pack = lane past the caches / pairs / pack = lane through the caches, inputs not in L2: 300 x 1000 7.9 / 8.1 / 7.9, fused with dropout and residual gradient 9.3 / 9.8 / 9.4, 512 x
// 1024 7.8 / 8.0 / 8.0, 9.1 / 9.5 / 9.6; 1000 x 1024 9.0 / 8.7 / 9.2, 11.0 / 10.6 / 11.8, 8192 x 1280 30.4 / 28.5 / 28.8, 47.1 / 44.1 / 45.4, 1000 x 8192 36.5 / 29.3 / 29.5, 58.9 / 46.0 /
// 47.9; rows that end inside a line the same: 8192 x 1304 32.0 / 29.5 / 29.6, 50.2 / 45.0 / 46.1, 5000 x 2040 32.6 / 29.4 / 28.9, 50.0 / 47.0 / 45.3.
template <typename T>
inline bool ln_bwd_paired(int64_t rows, int hidden) { return sizeof(T) == 4 && rows * hidden > (1 << 19); }

// fp32 with pack = lane goes through the caches, or half lines move, but only from 3 Mi elements on: below, as of a call whose inputs are not in L2, that is slower (300 x
// 512 2.4 / 2.8 us). us, past the caches / through them, inputs just written / in far memory / in the Infinity Cache: forward 419 x 5000 9.3 / 10.6, 6.1 / 7.1, 5.7 / 6.2; 1258 x 5000 23.2 /
// 20.6, 15.0 / 15.3, 14.1 / 10.9; 8388 x 1000 28.7 / 26.3, 21.1 / 20.3, 17.8 / 14.4; backward, fused with dropout and residual gradient, 8192 x 256 17.3 / 18.6, 14.4 / 15.4, 13.2 / 12.4;
// 16384 x 512 49.5 / 46.5, 40.3 / 39.1, 37.8 / 29.1; 65536 x 128 49.6 / 47.0, 38.1 / 39.2, 38.6 / 29.3.  256 lanes x 8 packs only if fused (1000 x 16384 68.2 / 55.9, plain 29.7 / 31.0), backward of
// more than 8192 columns always (30 x 16384 54.8 / 46.0, 57.5 / 47.1, 56.6 / 39.6).
// The fused forward of up to 4096 columns from 1.5 Mi on: 612 x 2568 14.5 / 13.7, 9.4 / 9.4, 8.7 / 7.1; 1063 x 2800 22.9 / 21.5, 16.5 / 15.8, 15.7 / 12.7; wider ones 500 x 4104 16.0 / 16.4, 9.4 / 11.1, 8.5 / 8.8.
template <typename T>
inline bool ln_cached(int64_t rows, int hidden, bool fused_fwd = false)
{
    return sizeof(T) == 4 && rows * hidden >= (fused_fwd && hidden <= 4096 ? 3ll << 19 : 3ll << 20);
}

// Row groups per workgroup: two, the second loaded ahead (8192 x 1280: one 11.1, two 9.2, four 10.4 us), but one where all groups find
// a compute unit of their own: up to 256 always (one against two, all shapes: 0.66-0.90), up to 768 where the kernel is small enough for
// three on a unit.  Time of one over two for 257..512 / 513..768 groups: 16 bits up to 5 packs per lane 0.87-1.02 / 0.90-1.05, more and
// 256 x 4 0.97-1.29 / 0.98-1.14; fp32 1 pack 0.90-1.03 / 0.97-1.01, more 1.02-1.24 (300 x 5120 fused 10.3 us as two, 13.5 as one; 300 x 2304 plain
// is the exception, 4.9 against 4.5) / 0.89-1.04.  Beyond 768: 0.95-1.31, above 1 nearly everywhere.
inline int ln_fwd_blocks(int64_t rows, LnShape sh, int elem_bytes)
{
    const int64_t groups = ceil_div(rows, static_cast<int64_t>(256 / sh.lpr));
    const bool small = elem_bytes == 2 ? sh.vpl <= (sh.lpr < 256 ? 5 : 3) : sh.vpl == 1 || groups > 512;
    int64_t b = groups <= 256 || (groups <= 768 && small) ? groups : ceil_div(groups, 2);
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    return static_cast<int>(b);
}

// (64 x 5: 16 bits only, see ln_fwd_shape)
#define LSQ_LN_FWD_CASES(X) X(8, 1) X(16, 1) X(32, 1) X(64, 1) X(64, 2) X(64, 3) X(64, 4) X(64, 6) X(256, 2) X(256, 3) X(256, 4) \
    X(32, 2) X(32, 3) X(32, 4) X(32, 5) X(32, 6) X(256, 6) X(256, 8) X(256, 1)

// fuse != nullptr: x is the projection output and *fuse carries h / residual / bias / dropout
template <typename T>
static lsq_status ln_fwd_dispatch(void* y, float* mean, float* rstd, const void* x, const void* gamma, const void* beta,
                                  int64_t rows, int32_t hidden, float eps, hipStream_t s,
                                  const BdrFuse<T>* fuse = nullptr)
{
    T* yp = static_cast<T*>(y);
    const T* xp = static_cast<const T*>(x);
    const T* gp = static_cast<const T*>(gamma);
    const T* bp = static_cast<const T*>(beta);
    LnShape sh = ln_fwd_shape(rows, hidden, sizeof(T));
    // rows of 8193..16384 columns: the forward has the registers for 6 or 8 packs per lane of a 256-thread
    // workgroup (0.70 of peak at 12288 columns against 0.53 with the backward's 1024 lanes x 2 packs).  The fused
    // boundary follows (it would be 10 % faster on 1024 lanes, but then no longer bit-identical to the two calls).
    if (sh.lpr > 256) sh = hidden / kPack <= 1536 ? LnShape{256, 6} : LnShape{256, 8};
    if (ln_rag_spans(hidden)) {
        const int quarter = 256 / ln_span_lanes(hidden);           // rows at a time: 256 threads, or one row
        const int lanes = quarter < 2 ? static_cast<int>(ceil_div(ln_span_lanes(hidden), 64)) * 64 : ln_span_lanes(hidden), slots = quarter < 2 ? 1 : quarter / 2 * 2;
        const int64_t groups = ceil_div(rows, slots);
        const dim3 g(static_cast<unsigned>(groups <= 768 ? groups : groups <= 16384 ? ceil_div(groups, 2) : 8192)), b(static_cast<unsigned>(slots * lanes));
        if (b.x <= 512) hipLaunchKernelGGL((ln_fwd_rag_kernel<T, 512>), g, b, 0, s, yp, mean, rstd, xp, gp, bp, rows, hidden, eps, lanes);
        else hipLaunchKernelGGL((ln_fwd_rag_kernel<T, 1024>), g, b, 0, s, yp, mean, rstd, xp, gp, bp, rows, hidden, eps, lanes);
        return launch_status();
    }
    if (sh.lpr == 0) {
        // rows too long for the register buckets come in small numbers: a whole workgroup per row
        if (hidden % kPack == 0)
            hipLaunchKernelGGL((ln_fwd_generic<T, 256, true>), dim3(static_cast<unsigned>(rows)), dim3(256), 0, s,
                               yp, mean, rstd, xp, gp, bp, rows, hidden, eps);
        else if (hidden > 2048)
            hipLaunchKernelGGL((ln_fwd_generic<T, 256, false>), dim3(static_cast<unsigned>(rows)), dim3(256), 0, s,
                               yp, mean, rstd, xp, gp, bp, rows, hidden, eps);
        else
            hipLaunchKernelGGL((ln_fwd_generic<T, 64, false>), dim3(static_cast<unsigned>(ceil_div(rows, 4))), dim3(256), 0, s,
                               yp, mean, rstd, xp, gp, bp, rows, hidden, eps);
        return launch_status();
    }
    bool launched = false;
    const dim3 grid(ln_fwd_blocks(rows, sh, sizeof(T))), block(256);
    const BdrFuse<T> none{};
    const bool pair = sizeof(T) == 4 && ln_fwd_paired(rows, hidden), cached = ln_cached<T>(rows, hidden, fuse != nullptr);
#define X(L, V)                                                                                              \
    if (sh.lpr == L && sh.vpl == V) {                                                                        \
        launched = true;                                                                                     \
        constexpr bool kPair = sizeof(T) == 4 && V < 8;                                                      \
        if (pair && kPair) { F(L, V, kPair, true) }                                                          \
        else if (cached && (V < 8 || fuse)) { F(L, V, false, sizeof(T) == 2) }                               \
        else { F(L, V, false, true) }                                                                        \
    }
#define F(L, V, PAIR, NT)                                                                                    \
        if (!fuse) hipLaunchKernelGGL((ln_fwd_kernel<T, L, V, false, false, PAIR, NT>), grid, block, 0, s, yp, mean, rstd, xp, gp, bp, rows, hidden, eps, none); \
        else if (fuse->d.on) hipLaunchKernelGGL((ln_fwd_kernel<T, L, V, true, true, PAIR, NT>), grid, block, 0, s, yp, mean, rstd, xp, gp, bp, rows, hidden, eps, *fuse); \
        else hipLaunchKernelGGL((ln_fwd_kernel<T, L, V, true, false, PAIR, NT>), grid, block, 0, s, yp, mean, rstd, xp, gp, bp, rows, hidden, eps, *fuse);
    LSQ_LN_FWD_CASES(X)
    if constexpr (sizeof(T) == 2) { X(64, 5) }
#undef X
#undef F
    return launched ? launch_status() : LSQ_LAUNCH_FAILED;      // a shape without its kernel
}

// Backward of rows with 1025..2048 packs: the column accumulators are thread-private LDS entries
// (up to 131 KB, above the 64 KiB a kernel gets by default: the limit is raised once per device).
template <typename T, int L, int V>
static lsq_status ln_bwd_wide(T* dxp, float* partial, const T* dyp, const T* xp, const T* gp, const float* mean,
                              const float* rstd, const T* rp, int64_t rows, int32_t hidden, int P, hipStream_t s)
{
    constexpr int TH = L >= 256 ? L : 256;
    const BdrFuse<T> nofuse{};
    const size_t shmem = sizeof(float) * 16 * ((hidden / kPack) | 1);
    auto* kres = &ln_bwd_kernel<T, L, V, true, TH, false, false, sizeof(T) == 2>;
    auto* kplain = &ln_bwd_kernel<T, L, V, false, TH, false, false, sizeof(T) == 2>;
    // once per residual variant and device (a host-side note, guarded for concurrent host threads)
    static std::mutex mu;
    static bool ready[2][64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return LSQ_LAUNCH_FAILED;
    const bool known = dev >= 0 && dev < 64;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!known || !ready[rp ? 1 : 0][dev]) {
            if (hipFuncSetAttribute(rp ? reinterpret_cast<const void*>(kres) : reinterpret_cast<const void*>(kplain),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) != hipSuccess)
                return LSQ_LAUNCH_FAILED;
            if (known) ready[rp ? 1 : 0][dev] = true;
        }
    }
    if (rp) hipLaunchKernelGGL(kres, dim3(P), dim3(TH), shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, nofuse);
    else hipLaunchKernelGGL(kplain, dim3(P), dim3(TH), shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, nofuse);
    return launch_status();
}

template <typename T>
static lsq_status ln_bwd_dispatch(void* dx, float* dgamma, float* dbeta, const void* dy, const void* x,
                                  const void* gamma, const float* mean, const float* rstd, const void* dres,
                                  void* workspace, int64_t rows, int32_t hidden, hipStream_t s,
                                  const BdrFuse<T>* fuse = nullptr, float* dbias = nullptr)
{
    T* dxp = static_cast<T*>(dx);
    const T* dyp = static_cast<const T*>(dy);
    const T* xp = static_cast<const T*>(x);
    const T* gp = static_cast<const T*>(gamma);
    const T* rp = static_cast<const T*>(dres);
    const LnShape sh = ln_shape(hidden);
    if (sh.lpr == 0 && !ln_rag_spans(hidden)) {
        const int Pg = ln_bwd_blocks(rows, hidden);
        float* gpartial = static_cast<float*>(workspace);
        if (hidden % kPack == 0)
            hipLaunchKernelGGL((ln_dparams_packed<T>), dim3(static_cast<unsigned>(ceil_div(hidden / kPack, 256)), static_cast<unsigned>(Pg)),
                               dim3(256), 0, s, gpartial, dyp, xp, mean, rstd, rows, hidden);
        else
            hipLaunchKernelGGL((ln_dparams_generic<T>), dim3(static_cast<unsigned>(ceil_div(hidden, 256)), static_cast<unsigned>(Pg)),
                               dim3(256), 0, s, gpartial, dyp, xp, mean, rstd, rows, hidden);
        launch_colsum_finalize(dgamma, dbeta, hidden, gpartial, Pg, 2 * hidden, s);
        if (hidden % kPack == 0)
            hipLaunchKernelGGL((ln_bwd_generic<T, 256, true>), dim3(static_cast<unsigned>(rows)), dim3(256), 0, s,
                               dxp, dyp, xp, gp, mean, rstd, rp, rows, hidden);
        else if (hidden > 2048)
            hipLaunchKernelGGL((ln_bwd_generic<T, 256, false>), dim3(static_cast<unsigned>(rows)), dim3(256), 0, s,
                               dxp, dyp, xp, gp, mean, rstd, rp, rows, hidden);
        else
            hipLaunchKernelGGL((ln_bwd_generic<T, 64, false>), dim3(static_cast<unsigned>(ceil_div(rows, 4))), dim3(256), 0, s,
                               dxp, dyp, xp, gp, mean, rstd, rp, rows, hidden);
        return launch_status();
    }
    const int P = ln_bwd_blocks(rows, hidden);
    float* partial = static_cast<float*>(workspace);
    if (sh.lpr > 256) {       // 8193..16384 columns (never fused: the entry point splits such rows into its two operators)
        lsq_status st;
        // (256 lanes x 6 or 8 packs with the same LDS accumulators: 200 us against 122 us at 8192 x 12288)
        st = ln_bwd_wide<T, kLnWideLpr, kLnWideVpl>(dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, P, s);
        if (st != LSQ_OK) return st;
        launch_colsum_finalize(dgamma, dbeta, hidden, partial, P, 2 * hidden, s);
        return launch_status();
    }
    const BdrFuse<T> none{};
    bool launched = ln_bwd_spans(hidden);
    if (launched) {
        const LnBwdPlan pl = ln_bwd_span_plan(rows, hidden);
        const dim3 grid(P), block(pl.slots * pl.lanes);
        const size_t exchange = sizeof(float) * (block.x / 8), tree = sizeof(float) * (pl.slots / 2) * (fuse ? 3 : 2) * 8 * pl.lanes;
        const size_t shmem = exchange > tree ? exchange : tree;
#define X(C, M, PAIR, NT)                                                                                    \
    if (!fuse) {                                                                                             \
        if (rp) hipLaunchKernelGGL((ln_bwd_span_kernel<T, C, true, M, false, false, false, PAIR, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, none); \
        else hipLaunchKernelGGL((ln_bwd_span_kernel<T, C, false, M, false, false, false, PAIR, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, none);   \
    } else if (fuse->d.on) {                                                                                 \
        if (rp) hipLaunchKernelGGL((ln_bwd_span_kernel<T, C, true, M, true, true, false, PAIR, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, *fuse);  \
        else hipLaunchKernelGGL((ln_bwd_span_kernel<T, C, false, M, true, true, false, PAIR, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, *fuse);    \
    } else {                                                                                                 \
        if (rp) hipLaunchKernelGGL((ln_bwd_span_kernel<T, C, true, M, true, false, false, PAIR, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, *fuse); \
        else hipLaunchKernelGGL((ln_bwd_span_kernel<T, C, false, M, true, false, false, PAIR, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, *fuse);   \
    }
        if (ln_rag_spans(hidden)) {
#define R(H, M) hipLaunchKernelGGL((ln_bwd_span_kernel<T, 0, H, M, false, false, true, false, true>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, pl.lanes, none)
            if (rp) { if (block.x <= kLnSpanThreads) R(true, kLnSpanThreads); else R(true, 1024); }
            else { if (block.x <= kLnSpanThreads) R(false, kLnSpanThreads); else R(false, 1024); }
#undef R
        } else if (pl.lanes == 64) {
            if (ln_cached<T>(rows, hidden)) { X(64, kLnSpanThreads, false, sizeof(T) == 2) }
            else { X(64, kLnSpanThreads, false, true) }
        }
        else if (block.x <= kLnSpanThreads && ln_bwd_paired<T>(rows, hidden)) { X(0, kLnSpanThreads, sizeof(T) == 4, true) }
        else if (block.x <= kLnSpanThreads) { X(0, kLnSpanThreads, false, true) }
        else if (ln_bwd_paired<T>(rows, hidden)) { X(0, 1024, sizeof(T) == 4, true) }
        else { X(0, 1024, false, true) }
#undef X
    }
    // shorter rows: lanes of one wave, one pack each, or two of 32 lanes
    const int nacc = fuse ? 3 : 2;
    const bool cached = ln_cached<T>(rows, hidden);
    const size_t one_copy = sizeof(float) * 8 * nacc * ((hidden / kPack) | 1);
#define X(L, V, NT)                                                                                          \
    if (!ln_bwd_spans(hidden) && sh.lpr == L && sh.vpl == V && cached != (NT)) {                                                        \
        launched = true;                                                                                     \
        constexpr int TH = kLnBwdThreads;                                                                    \
        const size_t shmem = one_copy * (TH / L);                                                            \
        const dim3 grid(P), block(TH);                                                                       \
        if (!fuse) {                                                                                         \
            if (rp) hipLaunchKernelGGL((ln_bwd_kernel<T, L, V, true, TH, false, false, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, none); \
            else hipLaunchKernelGGL((ln_bwd_kernel<T, L, V, false, TH, false, false, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, none);   \
        } else if (fuse->d.on) {                                                                            \
            if (rp) hipLaunchKernelGGL((ln_bwd_kernel<T, L, V, true, TH, true, true, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, *fuse); \
            else hipLaunchKernelGGL((ln_bwd_kernel<T, L, V, false, TH, true, true, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, *fuse);   \
        } else {                                                                                             \
            if (rp) hipLaunchKernelGGL((ln_bwd_kernel<T, L, V, true, TH, true, false, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, *fuse); \
            else hipLaunchKernelGGL((ln_bwd_kernel<T, L, V, false, TH, true, false, NT>), grid, block, shmem, s, dxp, partial, dyp, xp, gp, mean, rstd, rp, rows, hidden, *fuse);   \
        }                                                                                                    \
    }
    X(8, 1, true) X(16, 1, true) X(32, 1, true) X(32, 2, true)       // what ln_shape gives up to 63 packs
    if constexpr (sizeof(T) == 4) { X(8, 1, false) X(16, 1, false) X(32, 1, false) X(32, 2, false) }
#undef X
    if (!launched) return LSQ_LAUNCH_FAILED;                    // a shape without its kernel
    if (fuse) launch_colsum_finalize(dgamma, dbeta, hidden, partial, P, 3 * hidden, s, dbias, 2 * hidden);
    else launch_colsum_finalize(dgamma, dbeta, hidden, partial, P, 2 * hidden, s);
    return launch_status();
}

}  // namespace lsq

extern "C" lsq_status lsq_layernorm_fwd(void* y, float* mean, float* rstd, const void* x, const void* gamma,
                                        const void* beta, int64_t rows, int32_t hidden, float eps, lsq_dtype dt,
                                        void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0 && eps >= 0.0f);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    if (rows == 0) return LSQ_OK;
    LSQ_REQUIRE(y && mean && rstd && x && gamma && beta);
    LSQ_ALIGNED(y); LSQ_ALIGNED(x); LSQ_ALIGNED(gamma); LSQ_ALIGNED(beta);
    LSQ_REQUIRE(rows <= 0x7FFFFFFF);
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (dt) {
        case LSQ_F16: return ln_fwd_dispatch<f16>(y, mean, rstd, x, gamma, beta, rows, hidden, eps, s);
        case LSQ_BF16: return ln_fwd_dispatch<bf16>(y, mean, rstd, x, gamma, beta, rows, hidden, eps, s);
        default: return ln_fwd_dispatch<float>(y, mean, rstd, x, gamma, beta, rows, hidden, eps, s);
    }
}

extern "C" lsq_status lsq_layernorm_bwd(void* dx, float* dgamma, float* dbeta, const void* dy, const void* x,
                                        const void* gamma, const float* mean, const float* rstd, const void* dres_in,
                                        void* workspace, size_t workspace_bytes, int64_t rows, int32_t hidden,
                                        lsq_dtype dt, void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    LSQ_REQUIRE(dgamma && dbeta);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (rows == 0) {
        lsq_status st = zero_fill(dgamma, hidden, s);
        return st != LSQ_OK ? st : zero_fill(dbeta, hidden, s);
    }
    LSQ_REQUIRE(dx && dy && x && gamma && mean && rstd);
    LSQ_ALIGNED(dx); LSQ_ALIGNED(dy); LSQ_ALIGNED(x); LSQ_ALIGNED(gamma); LSQ_ALIGNED(dres_in); LSQ_ALIGNED(workspace);
    LSQ_REQUIRE(rows <= 0x7FFFFFFF);
    const size_t need = lsq_workspace_bytes(LSQ_OP_LAYERNORM_BWD, rows, hidden);
    if (need && (!workspace || workspace_bytes < need)) return LSQ_WORKSPACE_TOO_SMALL;
    switch (dt) {
        case LSQ_F16: return ln_bwd_dispatch<f16>(dx, dgamma, dbeta, dy, x, gamma, mean, rstd, dres_in, workspace, rows, hidden, s);
        case LSQ_BF16: return ln_bwd_dispatch<bf16>(dx, dgamma, dbeta, dy, x, gamma, mean, rstd, dres_in, workspace, rows, hidden, s);
        default: return ln_bwd_dispatch<float>(dx, dgamma, dbeta, dy, x, gamma, mean, rstd, dres_in, workspace, rows, hidden, s);
    }
}

// ---- LayerNorm backward for callers that may not allocate: the partial rows of the column sums go to
// device memory the library itself holds, one copy per GPU, for as long as the process lives.
namespace lsq {
constexpr size_t kLnScratchBytes = 8u << 20;
static __device__ __align__(256) unsigned char scratch[kLnScratchBytes];

// The array's address on the current device.  `scratch` itself is only a host-side handle: the
// address is asked for once per device (each GPU holds its own copy at its own address) and kept.
static void* ln_scratch_on_current_device()
{
    static std::mutex mu;
    static void* ptr[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        ptr[dev] = p;
    }
    return ptr[dev];
}
}  // namespace lsq

extern "C" lsq_status lsq_layernorm_bwd_noalloc(void* dx, float* dgamma, float* dbeta, const void* dy, const void* x,
                                                const void* gamma, const float* mean, const float* rstd,
                                                const void* dres_in, int64_t rows, int32_t hidden, lsq_dtype dt,
                                                void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0);
    if (lsq_workspace_bytes(LSQ_OP_LAYERNORM_BWD, rows, hidden) > kLnScratchBytes) return LSQ_WORKSPACE_TOO_SMALL;
    void* ws = nullptr;
    if (rows > 0) {
        ws = ln_scratch_on_current_device();
        if (!ws) return LSQ_LAUNCH_FAILED;
    }
    return lsq_layernorm_bwd(dx, dgamma, dbeta, dy, x, gamma, mean, rstd, dres_in, ws, kLnScratchBytes, rows, hidden, dt,
                             stream);
}

// ---- fused sub-layer boundary of a pre-LN Transformer
namespace lsq {
template <typename T>
static lsq_status bdr_ln_fwd_typed(void* h, void* y, float* mean, float* rstd, const void* x, const void* bias,
                                   const void* residual, const void* gamma, const void* beta, int64_t rows,
                                   int32_t hidden, float eps, const DropoutParams& d, hipStream_t s)
{
    const BdrFuse<T> fz{static_cast<T*>(h), static_cast<const T*>(residual), static_cast<const T*>(bias), d};
    return ln_fwd_dispatch<T>(y, mean, rstd, x, gamma, beta, rows, hidden, eps, s, &fz);
}

template <typename T>
static lsq_status bdr_ln_bwd_typed(void* dh, void* dx, float* dgamma, float* dbeta, float* dbias, const void* dy,
                                   const void* h, const void* gamma, const float* mean, const float* rstd,
                                   const void* dres_in, void* workspace, int64_t rows, int32_t hidden,
                                   const DropoutParams& d, hipStream_t s)
{
    const BdrFuse<T> fz{static_cast<T*>(dx), nullptr, nullptr, d};
    return ln_bwd_dispatch<T>(dh, dgamma, dbeta, dy, h, gamma, mean, rstd, dres_in, workspace, rows, hidden, s, &fz, dbias);
}
}  // namespace lsq

extern "C" lsq_status lsq_bdr_layernorm_fwd(void* h, void* y, float* mean, float* rstd, const void* x, const void* bias,
                                            const void* residual, const void* gamma, const void* beta, int64_t rows,
                                            int32_t hidden, float p, uint64_t seed, uint64_t offset, float eps,
                                            lsq_dtype dt, void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0 && eps >= 0.0f);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p, seed, offset, &d));
    if (rows == 0) return LSQ_OK;
    LSQ_REQUIRE(h && y && mean && rstd && x && residual && gamma && beta);
    LSQ_ALIGNED(h); LSQ_ALIGNED(y); LSQ_ALIGNED(x); LSQ_ALIGNED(bias); LSQ_ALIGNED(residual); LSQ_ALIGNED(gamma); LSQ_ALIGNED(beta);
    LSQ_REQUIRE(ceil_div(rows * hidden, 256) <= 0x7FFFFFFF);
    if (ln_shape(hidden).lpr == 0) {      // no register bucket for this row length: the two operators back to back
        const lsq_status st = lsq_bias_dropout_residual_fwd(h, x, bias, residual, rows, hidden, p, seed, offset, dt, stream);
        return st != LSQ_OK ? st : lsq_layernorm_fwd(y, mean, rstd, h, gamma, beta, rows, hidden, eps, dt, stream);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (dt) {
        case LSQ_F16: return bdr_ln_fwd_typed<f16>(h, y, mean, rstd, x, bias, residual, gamma, beta, rows, hidden, eps, d, s);
        case LSQ_BF16: return bdr_ln_fwd_typed<bf16>(h, y, mean, rstd, x, bias, residual, gamma, beta, rows, hidden, eps, d, s);
        default: return bdr_ln_fwd_typed<float>(h, y, mean, rstd, x, bias, residual, gamma, beta, rows, hidden, eps, d, s);
    }
}

extern "C" lsq_status lsq_bdr_layernorm_bwd(void* dh, void* dx, float* dgamma, float* dbeta, float* dbias, const void* dy,
                                            const void* h, const void* gamma, const float* mean, const float* rstd,
                                            const void* dres_in, void* workspace, size_t workspace_bytes, int64_t rows,
                                            int32_t hidden, float p, uint64_t seed, uint64_t offset, lsq_dtype dt,
                                            void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(rows >= 0 && hidden > 0);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p, seed, offset, &d));
    LSQ_REQUIRE(dgamma && dbeta && dbias);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (rows == 0) {
        lsq_status st = zero_fill(dgamma, hidden, s);
        if (st == LSQ_OK) st = zero_fill(dbeta, hidden, s);
        return st != LSQ_OK ? st : zero_fill(dbias, hidden, s);
    }
    LSQ_REQUIRE(dh && dx && dy && h && gamma && mean && rstd);
    LSQ_ALIGNED(dh); LSQ_ALIGNED(dx); LSQ_ALIGNED(dy); LSQ_ALIGNED(h); LSQ_ALIGNED(gamma); LSQ_ALIGNED(dres_in);
    LSQ_ALIGNED(workspace);
    LSQ_REQUIRE(ceil_div(rows * hidden, 256) <= 0x7FFFFFFF);
    const size_t fused = ln_bwd_bytes(rows, hidden, 3), apart = bdr_bwd_bytes(rows, hidden, dt == LSQ_F32 ? 4 : 2, d.on != 0), need = fused > apart ? fused : apart;
    if (need && (!workspace || workspace_bytes < need)) return LSQ_WORKSPACE_TOO_SMALL;
    if (ln_shape(hidden).lpr == 0 || ln_shape(hidden).lpr > 256) {      // no fused bucket: the two operators back to back
        const lsq_status st = lsq_layernorm_bwd(dh, dgamma, dbeta, dy, h, gamma, mean, rstd, dres_in, workspace,
                                                workspace_bytes, rows, hidden, dt, stream);
        return st != LSQ_OK ? st : lsq_bias_dropout_residual_bwd(dx, dbias, dh, rows, hidden, p, seed, offset, workspace,
                                                                workspace_bytes, dt, stream);
    }
    switch (dt) {
        case LSQ_F16: return bdr_ln_bwd_typed<f16>(dh, dx, dgamma, dbeta, dbias, dy, h, gamma, mean, rstd, dres_in, workspace, rows, hidden, d, s);
        case LSQ_BF16: return bdr_ln_bwd_typed<bf16>(dh, dx, dgamma, dbeta, dbias, dy, h, gamma, mean, rstd, dres_in, workspace, rows, hidden, d, s);
        default: return bdr_ln_bwd_typed<float>(dh, dx, dgamma, dbeta, dbias, dy, h, gamma, mean, rstd, dres_in, workspace, rows, hidden, d, s);
    }
}
