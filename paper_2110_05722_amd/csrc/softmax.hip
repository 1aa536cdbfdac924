// Masked, variable-length attention softmax, forward and backward (Sec. IV-B of
// the paper, Softmax: maximum, partition function, normalisation; backward is
// the softmax Jacobian of Sec. IV-A contracted with the upstream gradient).
//
// The paper copes with the spread of shapes ("a few to thousands" of columns,
// "thousands to millions" of rows) by tuning templates at run time.  Here the
// shape picks a compile-time bucket instead: LPR lanes share a row (1..64 lanes
// of a wave64), each lane keeps VPL packs of 8 scores in registers, so a row is
// read from HBM once, and both reductions run on DPP inside the wave.  Short rows put many rows in one wave (k_len 32 -> 16 rows per
// wave) so lanes are never idle.  Rows of 257..2048 packs take one workgroup
// each (the reductions cross its four waves through LDS).  Both exist in a form for rows
// of whole packs and in one for any other length (RAG), the common case of a batch
// that is padded to its longest sentence; longer rows fall to a three-pass kernel that
// re-reads the row from cache.
//
// The RAG form walks the aligned packs of the flat tensor that a row touches.  Many of the shorter such rows are faster through LDS,
// where every lane is busy whatever the alignment (sm_lds_shape).  With everything through LDS up to 2048 keys (2-byte LDS accesses and
// three barriers bound it) and 2-byte global accesses beyond, forward + backward took, fp16 unless stated, then -> now in us:
// 113 keys padded with dropout 64 x 16 x 113 47 -> 37, 201 keys 73 -> 52, 301 keys 97 -> 61, 751 keys causal 277 -> 97,
// 2001 keys bf16 415 -> 228, 3001 keys 624 -> 162, 7001 keys 78 -> 25.  All in registers lost at 27..63 keys fp16 (29 keys forward
// of 4 M scores 6.6 -> 8.9) and at 10..90 keys fp32 (29 keys with dropout 9.7 -> 20).
//
// Results are not materialised in fp32 before they are narrowed (as LayerNorm's are): in 109 of 202 fp16 kernels the compiler folds a last product into the conversion, one rounding
// where the others have two, so two of them may differ by an ulp in a few results of 100000.
//
// Masks restrict the SET the softmax runs over: packs that lie wholly beyond the
// row's limit (key padding, or the causal diagonal) are not even loaded, and
// their outputs are written as exact zeros.  Attention-probability dropout is
// fused (Philox per pack, mask regenerated in backward).
#include <atomic>
#include <mutex>

#include "host.hpp"

namespace lsq {
// Threads per workgroup of the packed kernels (lanes per row <= 64: the waves of a workgroup share nothing).  The
// backward is 2-3 % faster as one-wave workgroups (106 against 109 us at 8 x 20 x 1024 x 1024 causal, 62.6 against 64 us
// with key padding at 512 keys, 16.8 against 17.1 us at 256 keys), the forward 3-4 % slower at 256 keys and equal elsewhere.
constexpr int kSmWgFwd = 256, kSmWgBwd = 64;

constexpr float kLog2e = 1.4426950408889634f;

struct SoftmaxGeom {
    int64_t nrows;        // batch * heads * q_len (below 2^31)
    int rows_per_batch;   // heads * q_len
    FastDiv by_rows_per_batch, by_q_len;
    int q_len, k_len;
    int causal;           // 0 / 1
    int shift;            // k_len - q_len (end-aligned causal mask)
    float scale;
};

// key and query lengths of the batch (either may be absent)
struct SoftmaxLens {
    const int32_t* __restrict__ key;
    const int32_t* __restrict__ query;
};

// number of allowed keys (a prefix of the row) for query row `row`; 0 for a padded query
__device__ __forceinline__ int row_limit(const SoftmaxGeom& g, const SoftmaxLens& len, int64_t row)
{
    int limit = g.k_len;
    const uint32_t r32 = static_cast<uint32_t>(row);
    const int i = static_cast<int>(r32 - fastdiv(r32, g.by_q_len) * static_cast<uint32_t>(g.q_len));
    if (len.key || len.query) {
        // the rows of a wave almost always belong to one sentence: its lengths come through
        // the scalar path (one cached load per wave), the vector path serves a straddling wave
        const int b = static_cast<int>(fastdiv(r32, g.by_rows_per_batch));
        const int b0 = __builtin_amdgcn_readfirstlane(b);
        if (len.key) {
            int kl = len.key[b0];
            if (b != b0) kl = len.key[b];
            limit = min(max(kl, 0), g.k_len);
        }
        if (len.query) {
            int ql = len.query[b0];
            if (b != b0) ql = len.query[b];
            if (i >= ql) limit = 0;
        }
    }
    if (g.causal) limit = min(limit, max(i + 1 + g.shift, 0));
    return limit;
}

// Whether the pack that starts at position j0 of a row holds an allowed key.  The first pack of a ragged row starts before the row
// (j0 < 0), below the limit even of an empty or absent one.
template <bool RAG>
__device__ __forceinline__ bool pack_needed(int j0, int limit) { return j0 < limit && (!RAG || limit > 0); }

// With query lengths the rows of padded queries, often half of the tensor, need no load at all.  Then a row's limit is waited for before anything
// is loaded (`sm_late_*`; otherwise the first 128 bytes go out before it is known), and a wave whose rows are all empty writes its zeros and
// leaves (`sm_leaves_fwd`).  Where which is faster, time of the late loads over the early ones (lengths full ... half):
//  - rows of up to 128 bytes are loaded whole before the limit.  16 bits, whole packs: forward 1.10-1.23 (64 x 16 x 64 x 64 fp16 with dropout
//    6.9 -> 8.9 us), backward of 4 M elements 1.05-1.22, of 16 M 1.03 ... 0.84; more queries than keys under a causal mask leave most rows
//    empty: 1.1 ... 0.68.  Any other length and fp32: 1.0-1.06 ... 0.63-1.0, fp32 forward with dropout 0.82-0.88 ... 0.76;
//  - forward, whole packs, below 1024 bytes 0.76-1.0; longer ones with half of their rows empty lose (1000 keys fp16 with dropout
//    1.12, fp32 1.27, 512 keys fp32 1.18), full ones gain 1-4 %; only 16 bits without dropout keep 0.89-1.0 at any length;
//  - forward, any other length 0.77-1.0 and with the leaving waves up to 0.10 less, but 16 bits beyond 1536 keys 1.0-1.18 (2001 keys),
//    and with dropout beyond 640 leaving costs 0-0.13 again (1025 keys, half 0.99 -> 1.05, 2001 1.18 -> 1.23);
//  - backward 0.72-1.0, but fp32 whole packs beyond 1024 keys 1.01-1.07 at half;
//  - a causal mask keeps the rows' ends apart: beyond 128 bytes 0.84-1.02 in both directions at every length, leaving included
//    (409 x 1537 bf16 with dropout 19.0 -> 17.1 us); only 16 bits with dropout, whole packs of 1024 bytes on, lose it again on tensors beyond
//    the Infinity Cache (1000 x 1000 keys: 15 M scores 0.93, 128 M 1.08).
template <typename T, bool RAG>
__device__ __forceinline__ bool sm_late_short(const SoftmaxGeom& g)       // rows of up to 128 bytes
{
    return sizeof(T) == 4 || RAG || (g.causal && g.shift < 0);
}
template <typename T, bool DROP, bool RAG>
__device__ __forceinline__ bool sm_late_fwd(const SoftmaxGeom& g)
{
    const int bytes = g.k_len * static_cast<int>(sizeof(T));
    if (bytes <= 128) return sm_late_short<T, RAG>(g);
    if (g.causal) return RAG || sizeof(T) == 4 || !DROP || bytes < 1024 || g.nrows * g.k_len <= (int64_t{64} << 20);
    return RAG ? sizeof(T) == 4 || g.k_len <= 1536 : bytes < 1024 || (sizeof(T) == 2 && !DROP);
}
template <typename T, bool DROP>
__device__ __forceinline__ bool sm_leaves_fwd(const SoftmaxGeom& g) { return g.causal || !(sizeof(T) == 2 && DROP && g.k_len > 640); }
template <typename T, bool RAG>
__device__ __forceinline__ bool sm_late_bwd(const SoftmaxGeom& g)
{
    if (g.k_len * static_cast<int>(sizeof(T)) <= 128) return sm_late_short<T, RAG>(g) || g.nrows * g.k_len >= (int64_t{8} << 20);
    return sizeof(T) == 2 || RAG || g.causal || g.k_len <= 1024;
}

// ---- where the packs of a row lie.  RAG = false: rows are whole packs (k_len % 8 == 0), pack idx of a row starts at
// its element 8 * idx.  RAG = true: any k_len.  The packs are those of the FLAT tensor (aligned 128-bit accesses, and the
// groups the dropout contract counts): a row that starts s elements into a pack touches (s + k_len + 7) / 8 of them, pack
// idx starts at row position 8 * idx - s, and the first and the last may be shared with the neighbouring rows.  Loading a
// neighbour's elements is harmless (they are masked in registers), storing is done element by element for the
// part that belongs to the row.
//
// Positions are kept relative to the workgroup's first pack: what is 64 bits wide (the row index times k_len, the tensor's
// size) is computed once in scalar registers, and a lane's addresses are a scalar base plus a 32-bit offset.
template <bool RAG>
struct RowPacks {
    int first;            // the row's first pack, counted from the workgroup's first pack
    int s, n;             // elements of that pack in front of the row; packs the row touches
};

// The rows of a workgroup: `row0` on, `rows` of them exist (capped at 2^30, which no workgroup reaches).
template <bool RAG>
struct BlockRows {
    int64_t row0, pack0;  // first row; first pack of the flat tensor that it touches
    int s, rows, elems;   // elements of that pack in front of the first row; existing rows; elements of the tensor from pack0 on (capped)
    __device__ __forceinline__ BlockRows(const SoftmaxGeom& g, int64_t first_row)
    {
        constexpr int64_t kCap = 1 << 30;
        row0 = first_row;
        const int64_t e0 = first_row * g.k_len, total = g.nrows * g.k_len;
        pack0 = static_cast<int64_t>(static_cast<uint64_t>(e0) / kPack);
        s = RAG ? static_cast<int>(e0 & (kPack - 1)) : 0;
        rows = static_cast<int>(min(g.nrows - first_row, kCap));
        elems = static_cast<int>(min(total - pack0 * kPack, kCap));
    }
    __device__ __forceinline__ RowPacks<RAG> row(const SoftmaxGeom& g, int i) const
    {
        const unsigned e = static_cast<unsigned>(s + i * g.k_len);
        RowPacks<RAG> p;
        p.first = static_cast<int>(e / kPack);
        p.s = RAG ? static_cast<int>(e % kPack) : 0;
        p.n = (RAG ? p.s + g.k_len + kPack - 1 : g.k_len) / kPack;
        return p;
    }
};

// Nontemporal hints of the ragged form.  Rows that do not start on a 128-byte line share lines between a lane's packs and
// with their neighbours, and a line that is fetched or written in two pieces should stay in L2 in between: the loads go
// without the hint up to a wave per row (113 keys, dropout and padding: 21.3 / 20.5 us forward / backward against 28.3 / 21.8),
// the stores where a store instruction covers 128 bytes of a row or a row takes three (19.3 / 17.6 us; 751 keys causal 43.0 / 53.7
// against 43.9 / 61.9).  Longer pieces keep it (2001 keys: 101 against 129 us backward; 201: 27.0 against 31.3 us forward).
// fp32 rows are twice as many lines, and their stores keep the hint with one pack per lane only (201 keys with dropout, 48 M scores:
// 164 -> 129 us forward; 1001 keys 149 -> 111).
template <int LPR, int VPL, bool RAG> constexpr bool sm_load_nt() { return !RAG || LPR > kWave; }
template <typename T, int LPR, int VPL, bool RAG> constexpr bool sm_store_nt()
{
    return !RAG || VPL == 1 || LPR > kWave || (sizeof(T) == 2 && (LPR == kWave || (LPR > 8 && VPL == 2)));
}

// Packs in lane pairs (LanePacks), fp32 rows of 8 lanes and more: sm_paired below.  Both forms add in the order of the packs, so a row of whole packs has the same
// bits whatever the size of the call.  A pack that is loaded before the row's limit is known lies in
// the first group of 8, and there in the first half: in the first piece of every lane of the group.
template <typename T, bool PAIR> using SmPacks = LanePacks<T, PAIR ? 8 : 1>;

// pack `idx` of a row (`base`: the workgroup's first pack); the last pack of the tensor may be cut short
template <typename T, int LPR, int VPL, bool RAG>
__device__ __forceinline__ RawPack<T> load_row_pack(const T* base, const RowPacks<RAG>& p, int idx, int elems)
{
    const unsigned e = static_cast<unsigned>(p.first + idx) * kPack;
    if constexpr (RAG) {
        const int left = elems - static_cast<int>(e);
        if (left < kPack) {
            RawPack<T> r = zero_raw<T>();
            T f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = j < left ? base[e + j] : from_f32<T>(0.0f);
            __builtin_memcpy(&r, f, sizeof(r));
            return r;
        }
    }
    return load_raw<T, sm_load_nt<LPR, VPL, RAG>()>(base + e);
}

// A pack as registers: 4 for fp16/bf16, 8 for fp32.
template <typename T> struct PackWords { uint32_t w[sizeof(T) * 2]; };

// elements [a, 8) (TAIL = false) or [0, b) (TAIL = true) of the pack at `at`, in at most three naturally aligned
// stores of 4, 2 and 1 elements (one store per element cost 20 cycles of a compute unit each, 8 per pack)
template <typename T, bool TAIL>
__device__ __forceinline__ void store_part(T* at, const RawPack<T>& r, int edge)
{
    const PackWords<T> p = __builtin_bit_cast(PackWords<T>, r);
    const int n = TAIL ? edge : kPack - edge;                         // elements stored (1..7)
    const int o2 = TAIL ? (edge & 4) : (edge + (edge & 1));           // where the pieces of two and of one start
    const int o1 = TAIL ? edge - 1 : edge;
    if constexpr (sizeof(T) == 2) {
        if (n & 4) *reinterpret_cast<uvec2*>(at + (TAIL ? 0 : 4)) = TAIL ? uvec2{p.w[0], p.w[1]} : uvec2{p.w[2], p.w[3]};
        if (n & 2) {
            const uint32_t v = o2 < 4 ? (o2 < 2 ? p.w[0] : p.w[1]) : (o2 < 6 ? p.w[2] : p.w[3]);
            *reinterpret_cast<uint32_t*>(at + o2) = v;
        }
        if (n & 1) {
            const uint32_t v = o1 < 4 ? (o1 < 2 ? p.w[0] : p.w[1]) : (o1 < 6 ? p.w[2] : p.w[3]);
            *reinterpret_cast<uint16_t*>(at + o1) = static_cast<uint16_t>(v >> (16 * (o1 & 1)));
        }
    } else {
        if (n & 4) *reinterpret_cast<uvec4*>(at + (TAIL ? 0 : 4)) = TAIL ? uvec4{p.w[0], p.w[1], p.w[2], p.w[3]} : uvec4{p.w[4], p.w[5], p.w[6], p.w[7]};
        if (n & 2) {
            const uvec2 v = o2 < 4 ? (o2 < 2 ? uvec2{p.w[0], p.w[1]} : uvec2{p.w[2], p.w[3]})
                                   : (o2 < 6 ? uvec2{p.w[4], p.w[5]} : uvec2{p.w[6], p.w[7]});
            *reinterpret_cast<uvec2*>(at + o2) = v;
        }
        if (n & 1) {
            uint32_t v = p.w[0];
#pragma unroll
            for (int j = 1; j < 8; ++j) v = o1 == j ? p.w[j] : v;
            *reinterpret_cast<uint32_t*>(at + o1) = v;
        }
    }
}

// Zeros from position `lim` of the row on and (DROP) where the element was dropped: for the rare rows where an infinity or a
// NaN would reach those positions (0 * NaN).  It works on the finished packs, so that ordinary rows pay a branch and no
// registers; `flat` is the row's first pack in the tensor.
template <typename T, int LPR, bool DROP, int VPL>
__device__ __forceinline__ void mask_packs(RawPack<T> (&pk)[VPL], int sub, int s, int lim, DropoutParams d = {}, int64_t flat = 0)
{
    // keys of its own, or the twenty round keys of the ordinary draw stay in scalar registers for this one
    if constexpr (DROP) asm volatile("" : "+s"(d.key0), "+s"(d.key1));
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        int allowed = lim - ((sub + k * LPR) * kPack - s);                // of this pack's 8 elements
        // What the ordinary rows must not pay for: the masks of the first pass kept for this one, and packs that cross the branch
        // as single halves instead of words (8-12 % of the forward with dropout each).
        asm volatile("" : "+v"(allowed));
        opaque(pk[k]);
        float f[8];
        unpack<T>(pk[k], f);
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = j < allowed ? f[j] : 0.0f;
        if constexpr (DROP) dropout_keep8(d, static_cast<uint64_t>(flat + sub + k * LPR), f);
        pk[k] = pack_raw<T>(f);
        opaque(pk[k]);
    }
}

// Stores one result row, VPL packs per lane.  A pack that two rows of one wave share is stored once, whole: the lane
// that holds the end of a row fetches the start of the next row's first pack from that row's lane 0.  What is left
// in parts is the first pack of the wave's first row and the last pack of its last.  All lanes of the wave call it
// (`rv`: the row exists); LPR = 256 means the row spans the workgroup.  Rows of at most a pack may share one with
// several others and are stored element by element.
template <typename T, int LPR, int VPL, bool RAG, bool PAIR>
__device__ __forceinline__ void store_row(T* base, const RowPacks<RAG>& p, int sub, bool rv, bool next_rv, int k_len,
                                          const RawPack<T> (&pk)[VPL])
{
    T* at = base + static_cast<unsigned>(p.first + sub) * kPack;      // of pack k: at + k * LPR * kPack
    if constexpr (!RAG) {
#pragma unroll
        for (int k = 0; k < VPL; ++k)
            SmPacks<T, PAIR>::template store<sm_store_nt<T, LPR, VPL, RAG>()>(at + k * LPR * kPack, pk[k], rv && sub + k * LPR < p.n);
    } else {
        if (k_len <= kPack) {                                         // uniform
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                float f[8];
                unpack<T>(pk[k], f);
                const int p0 = (sub + k * LPR) * kPack - p.s;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (rv && static_cast<unsigned>(p0 + j) < static_cast<unsigned>(k_len)) at[k * LPR * kPack + j] = from_f32<T>(f[j]);
            }
            return;
        }
        const int cut = (p.s + k_len) % kPack;                        // elements of the last pack that are this row's (0: all)
        RawPack<T> tail = pk[0];
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            const bool head = k == 0 && sub == 0 && p.s > 0;
            const bool last = idx == p.n - 1 && cut > 0;
            if (last) tail = pk[k];
            if (rv && idx < p.n && !head && !last) store_raw<T, sm_store_nt<T, LPR, VPL, RAG>()>(at + k * LPR * kPack, pk[k]);
        }
        const int kt = (p.n - 1) / LPR;                               // the last pack is pack kt of lane (n - 1) % LPR
        const bool mine = rv && cut > 0 && sub + kt * LPR == p.n - 1;
        T* tail_at = at + kt * LPR * kPack;
        bool whole = false;
        if constexpr (LPR < kWave) {
            const int lane = threadIdx.x % kWave;
            const int from = (lane / LPR + 1) * LPR;                  // lane 0 of the next row
            PackWords<T> t = __builtin_bit_cast(PackWords<T>, tail);
            const PackWords<T> h = __builtin_bit_cast(PackWords<T>, pk[0]);
            whole = mine && from < kWave && next_rv;
#pragma unroll
            for (int i = 0; i < static_cast<int>(sizeof(T)) * 2; ++i) {
                const uint32_t o = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from * 4, static_cast<int>(h.w[i])));
                if constexpr (sizeof(T) == 2)       // which of the word's two elements are this row's
                    t.w[i] = cut >= 2 * i + 2 ? t.w[i] : cut == 2 * i + 1 ? (t.w[i] & 0xFFFFu) | (o & 0xFFFF0000u) : o;
                else
                    t.w[i] = cut > i ? t.w[i] : o;
            }
            if (whole) store_raw<T, sm_store_nt<T, LPR, VPL, RAG>()>(tail_at, __builtin_bit_cast(RawPack<T>, t));
            if (rv && p.s > 0 && lane == 0) store_part<T, false>(at, pk[0], p.s);
        } else {
            if (rv && p.s > 0 && sub == 0) store_part<T, false>(at, pk[0], p.s);
        }
        if (mine && !whole) store_part<T, true>(tail_at, tail, cut);
    }
}

// The rows [first, first + count) of the workgroup, all of them empty (padded queries, empty sentences): their elements are one range
// of the tensor, written as zeros in whole packs by the wave.  Half of the waves of a padded batch hold nothing else; the row by
// row way, with its reductions and the pieces at every row's ends, cost as much issue time there as in a row of a few keys
// (64 x 16 x 113 x 113 fp16 with padding and dropout, forward and backward: 39.8 -> 37.5 us).
template <typename T, bool NT, bool RAG>
__device__ __forceinline__ void zero_rows(T* base, const BlockRows<RAG>& blk, int first, int count, int k_len)
{
    const int lane = threadIdx.x % kWave;
    const int end = min(first + count, blk.rows);
    if (first >= end) return;
    const int a = blk.s + first * k_len, b = blk.s + end * k_len;
    const int a8 = (a + kPack - 1) / kPack * kPack, b8 = b / kPack * kPack;
    constexpr int V = 16 / sizeof(T);
    for (int e = a8 + lane * V; e < b8; e += kWave * V) st_f4<NT>(reinterpret_cast<float*>(base + e), fvec4{0, 0, 0, 0});
    if constexpr (RAG) {                                              // what is shared with the rows beside them
        if (a + lane < min(a8, b)) base[a + lane] = from_f32<T>(0.0f);
        if (b8 >= a8 && b8 + lane < b) base[b8 + lane] = from_f32<T>(0.0f);
    }
}

// RPT rows per lane group: the loads of all RPT rows are issued before the first
// reduction, so a wave has RPT*VPL packs per lane in flight and the two dependent
// round trips (lengths, then scores) are paid once per RPT rows.
template <typename T, int LPR, int VPL, int RPT, bool DROP, bool RAG, bool PAIR>
__global__ __launch_bounds__(kSmWgFwd) void softmax_fwd_kernel(T* y, T* __restrict__ yd, const T* x,
                                                          SoftmaxLens len, SoftmaxGeom g, DropoutParams d)
{
    constexpr int RPB = kSmWgFwd / LPR;
    using P = SmPacks<T, PAIR>;
    const int sub = P::pack(threadIdx.x % LPR);
    const BlockRows<RAG> blk(g, static_cast<int64_t>(blockIdx.x) * (RPT * RPB));
    x += blk.pack0 * kPack;
    y += blk.pack0 * kPack;
    if constexpr (DROP) yd += blk.pack0 * kPack;
    int row[RPT];             // counted from the workgroup's first
    RowPacks<RAG> rp[RPT];
    int limit[RPT];
    // Loads first, arithmetic after.  The packs of a row's first 128 bytes are loaded before the
    // row's limit is known (unless the row is empty that line is needed whatever the limit, and
    // what lies beyond the limit is masked in registers): with a key-padding mask the limit comes
    // from memory, and waiting for it first would put two dependent round trips in front of
    // every row.  The other packs are loaded only if they reach into the allowed prefix.
    // (a limit that is computed from the row index alone, causal or none, waits for nothing).  With query lengths see sm_late_fwd.
    const bool late = len.query && sm_late_fwd<T, DROP, RAG>(g);
    const int kEarly = late ? -kPack : (len.key || len.query) ? 128 / static_cast<int>(sizeof(T)) : 0;
    RawPack<T> raw[RPT][VPL];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        row[r] = r * RPB + threadIdx.x / LPR;
        rp[r] = blk.row(g, row[r]);
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR, j0 = idx * kPack - rp[r].s;
            if constexpr (P::kPaired) {
                raw[r][k] = P::template load<true>(x + static_cast<unsigned>(rp[r].first + idx) * kPack, k == 0 && j0 < kEarly && row[r] < blk.rows && j0 < g.k_len);
            } else if (j0 < kEarly) {
                if (row[r] < blk.rows && j0 < g.k_len) raw[r][k] = load_row_pack<T, LPR, VPL, RAG>(x, rp[r], idx, blk.elems);
                else raw[r][k] = zero_raw<T>();
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) limit[r] = row[r] < blk.rows ? row_limit(g, len, blk.row0 + row[r]) : 0;
    if (late && sm_leaves_fwd<T, DROP>(g)) {                    // uniform
        bool empty = true;
#pragma unroll
        for (int r = 0; r < RPT; ++r) empty = empty && limit[r] <= 0;
        if (__ballot(!empty) == 0) {
            constexpr bool nt = sm_store_nt<T, LPR, VPL, RAG>();
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const int first = r * RPB + static_cast<int>(threadIdx.x / kWave) * (kWave / LPR);
                zero_rows<T, nt, RAG>(y, blk, first, kWave / LPR, g.k_len);
                if constexpr (DROP) zero_rows<T, nt, RAG>(yd, blk, first, kWave / LPR, g.k_len);
            }
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR, j0 = idx * kPack - rp[r].s;
            const bool need = pack_needed<RAG>(j0, limit[r]);         // implies a valid row and pack
            if constexpr (P::kPaired) {
                P::template load_into<true>(raw[r][k], x + static_cast<unsigned>(rp[r].first + idx) * kPack, j0 >= kEarly && need);
            } else if (j0 >= kEarly) {
                if (need) raw[r][k] = load_row_pack<T, LPR, VPL, RAG>(x, rp[r], idx, blk.elems);
                else raw[r][k] = zero_raw<T>();
            }
        }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int lim = limit[r];
        float v[VPL][8];
        bool live[VPL];       // wave-uniform: does any lane of the wave hold an allowed element of pack k?
        float mx = -INFINITY;
        // A positive scale (every attention scale is) commutes with the maximum and folds into the exponent's fma: one
        // multiplication per element less in a kernel that is bound by vector-ALU issue slots.  Any other scale is
        // multiplied in first (a uniform branch).
        const bool fold = g.scale > 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int j0 = (sub + k * LPR) * kPack - rp[r].s;
            live[k] = __ballot(pack_needed<RAG>(j0, lim)) != 0;
            if (live[k]) {    // a pack that is masked for the whole wave costs no arithmetic
                unpack<T>(P::settle(raw[r][k]), v[k]);
                if (!fold) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[k][j] *= g.scale;
                }
                const int allowed = lim - j0;             // of this pack's 8 elements (<= 0: none, >= 8: all)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    bool in = j < allowed;
                    if constexpr (RAG) { if (k == 0) in = in && j + j0 >= 0; }      // only pack 0 can start before the row
                    v[k][j] = in ? v[k][j] : -INFINITY;
                    mx = fmaxf(mx, v[k][j]);
                }
            }
        }
        mx = group_max<LPR>(mx);
        const float c = fold ? g.scale * kLog2e : kLog2e;
        const float mxs = (lim > 0 ? mx : 0.0f) * c;
        float z = 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            if (live[k]) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float e = __builtin_amdgcn_exp2f(fmaf(v[k][j], c, -mxs));   // exp2(-inf) = 0 on masked lanes
                    v[k][j] = e;
                    z += e;
                }
            }
        }
        z = group_sum<LPR, P::kPaired>(z);
        const float inv = lim > 0 ? 1.0f / z : 0.0f;
        // a NaN row (a NaN or +inf among its scores, or nothing but -inf) stays NaN inside the mask only
        const bool nan_row = __ballot(z != z) != 0;            // wave-uniform
        const bool rv = row[r] < blk.rows, next_rv = row[r] + 1 < blk.rows;
        RawPack<T> pk[VPL];
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            pk[k] = zero_raw<T>();
            if (live[k]) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[k][j] *= inv;
                pk[k] = pack_raw<T>(v[k]);
            }
        }
        if (nan_row) mask_packs<T, LPR, false>(pk, sub, rp[r].s, lim);
        store_row<T, LPR, VPL, RAG, PAIR>(y, rp[r], sub, rv, next_rv, g.k_len, pk);
        if constexpr (DROP) {
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const int idx = sub + k * LPR;
                if (live[k] && idx * kPack - rp[r].s < lim) {    // packs beyond the mask are zeros whatever the draw
                    float kf[8];
                    dropout_factors8(d, static_cast<uint64_t>(blk.pack0 + (rp[r].first + idx)), kf);
#pragma unroll
                    for (int j = 0; j < 8; ++j) kf[j] *= v[k][j];
                    pk[k] = pack_raw<T>(kf);
                }
            }
            if (nan_row) mask_packs<T, LPR, true>(pk, sub, rp[r].s, lim, d, blk.pack0 + rp[r].first);
            store_row<T, LPR, VPL, RAG, PAIR>(yd, rp[r], sub, rv, next_rv, g.k_len, pk);
        }
    }
}

template <typename T, int LPR, int VPL, int RPT, bool DROP, bool RAG, bool PAIR>
__global__ __launch_bounds__(kSmWgBwd) void softmax_bwd_kernel(T* dx, const T* dy, const T* __restrict__ y,
                                                          SoftmaxLens len, SoftmaxGeom g, DropoutParams d)
{
    constexpr int RPB = kSmWgBwd / LPR;
    using P = SmPacks<T, PAIR>;
    const int sub = P::pack(threadIdx.x % LPR);
    const BlockRows<RAG> blk(g, static_cast<int64_t>(blockIdx.x) * (RPT * RPB));
    y += blk.pack0 * kPack;
    dy += blk.pack0 * kPack;
    dx += blk.pack0 * kPack;
    int row[RPT];             // counted from the workgroup's first
    RowPacks<RAG> rp[RPT];
    int limit[RPT];
    // as in forward: the first 128 bytes of a row are loaded before its limit is known, unless sm_late_bwd says otherwise
    const bool late = len.query && sm_late_bwd<T, RAG>(g);
    const int kEarly = late ? -kPack : (len.key || len.query) ? 128 / static_cast<int>(sizeof(T)) : 0;
    RawPack<T> ry[RPT][VPL], rg[RPT][VPL];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        row[r] = r * RPB + threadIdx.x / LPR;
        rp[r] = blk.row(g, row[r]);
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR, j0 = idx * kPack - rp[r].s;
            if constexpr (P::kPaired) {
                const unsigned e = static_cast<unsigned>(rp[r].first + idx) * kPack;
                const bool ok = k == 0 && j0 < kEarly && row[r] < blk.rows && j0 < g.k_len;
                ry[r][k] = P::template load<true>(y + e, ok);
                rg[r][k] = P::template load<true>(dy + e, ok);
            } else if (j0 < kEarly) {
                if (row[r] < blk.rows && j0 < g.k_len) {
                    ry[r][k] = load_row_pack<T, LPR, VPL, RAG>(y, rp[r], idx, blk.elems);
                    rg[r][k] = load_row_pack<T, LPR, VPL, RAG>(dy, rp[r], idx, blk.elems);
                } else {
                    ry[r][k] = zero_raw<T>();
                    rg[r][k] = zero_raw<T>();
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) limit[r] = row[r] < blk.rows ? row_limit(g, len, blk.row0 + row[r]) : 0;
    if (late) {                                                       // uniform
        bool empty = true;
#pragma unroll
        for (int r = 0; r < RPT; ++r) empty = empty && limit[r] <= 0;
        if (__ballot(!empty) == 0) {
            constexpr bool nt = sm_store_nt<T, LPR, VPL, RAG>();
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const int first = r * RPB + static_cast<int>(threadIdx.x / kWave) * (kWave / LPR);
                zero_rows<T, nt, RAG>(dx, blk, first, kWave / LPR, g.k_len);
            }
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR, j0 = idx * kPack - rp[r].s;
            const bool need = pack_needed<RAG>(j0, limit[r]);
            if constexpr (P::kPaired) {
                const unsigned e = static_cast<unsigned>(rp[r].first + idx) * kPack;
                const bool ok = j0 >= kEarly && need;
                P::template load_into<true>(ry[r][k], y + e, ok);
                P::template load_into<true>(rg[r][k], dy + e, ok);
            } else if (j0 >= kEarly) {
                if (need) {
                    ry[r][k] = load_row_pack<T, LPR, VPL, RAG>(y, rp[r], idx, blk.elems);
                    rg[r][k] = load_row_pack<T, LPR, VPL, RAG>(dy, rp[r], idx, blk.elems);
                } else {
                    ry[r][k] = zero_raw<T>();
                    rg[r][k] = zero_raw<T>();
                }
            }
        }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int lim = limit[r];
        float yv[VPL][8], gv[VPL][8];
        float dot = 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * LPR;
            const int j0 = idx * kPack - rp[r].s;
            unpack<T>(P::settle(ry[r][k]), yv[k]);
            unpack<T>(P::settle(rg[r][k]), gv[k]);
            if constexpr (DROP) {
                // RAG: a dropped infinity is 0.  For whole packs the factors, which are ready before the data, are 5 % faster at 16 keys;
                // a dropped infinity spoils the row's sum there.
                if (j0 < lim) {
                    const uint64_t pack = static_cast<uint64_t>(blk.pack0 + (rp[r].first + idx));
                    if constexpr (RAG) {
                        dropout_keep8(d, pack, gv[k]);
#pragma unroll
                        for (int j = 0; j < 8; ++j) gv[k][j] *= d.scale;
                    } else {
                        float kf[8];
                        dropout_factors8(d, pack, kf);
#pragma unroll
                        for (int j = 0; j < 8; ++j) gv[k][j] *= kf[j];
                    }
                }
            }
            const int allowed = lim - j0;                 // of this pack's 8 elements (<= 0: none, >= 8: all)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                bool out = j >= allowed;
                if constexpr (RAG) { if (k == 0) out = out || j + j0 < 0; }
                if (out) { yv[k][j] = 0.0f; gv[k][j] = 0.0f; }       // whatever sits beyond the mask never counts
                dot = fmaf(gv[k][j], yv[k][j], dot);
            }
        }
        dot = group_sum<LPR, P::kPaired>(dot);
        const bool spoilt = __ballot(!__builtin_isfinite(dot)) != 0;      // wave-uniform: an infinity or a NaN reached a row's sum
        RawPack<T> pk[VPL];
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            float o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)      // outside the allowed set y and dy are zero here: the sum with +0 turns the product's -0 into +0
                o[j] = g.scale * yv[k][j] * (gv[k][j] - dot) + 0.0f;
            pk[k] = pack_raw<T>(o);
        }
        if (spoilt) mask_packs<T, LPR, false>(pk, sub, rp[r].s, lim);           // 0 * (0 - dot) is NaN there
        store_row<T, LPR, VPL, RAG, PAIR>(dx, rp[r], sub, row[r] < blk.rows, row[r] + 1 < blk.rows, g.k_len, pk);
    }
}

// ---- the same rows through LDS (k_len % 8 != 0, up to 512 keys), where the register form is the slower one (sm_lds_shape below has
// the lines).  A workgroup's rows are one contiguous element range [e0, e1) of the tensor: the aligned packs that cover
// it are copied to LDS, LPR lanes per row work on LDS with element accesses, every lane EPL elements that lie LPR apart, and the
// results leave in packs again.  The first and the last pack may be shared with the neighbouring workgroups: reading
// them is harmless, writing is done element by element for the part that belongs here.  Element i of LDS = element
// (e0 & ~7) + i of the tensor.  One Philox call per pack, its keep decisions as bits in LDS.  What bounds it is LDS issue (two accesses
// per element) and three barriers; every lane is busy whatever the row's alignment, where the register form
// idles the lanes between the packs that a row touches and the next shape.
template <int LPR, int EPL> constexpr int lds_rows_elems() { return 256 * EPL + 16; }     // of a staged tensor: 256 / LPR rows of LPR * EPL, and their cut packs

// the keep bits of the packs [p0, p1) (bit j = element j survives)
template <int NBYTES>
__device__ __forceinline__ void lds_keep_bits(uint8_t (&keep)[NBYTES], const DropoutParams& d, int64_t p0, int64_t p1)
{
    for (int64_t pk = p0 + threadIdx.x; pk < p1; pk += 256) {
        uint32_t w[4], bits = 0;
        philox4x32_10(static_cast<uint32_t>(pk), static_cast<uint32_t>(static_cast<uint64_t>(pk) >> 32), d.ctr2, d.ctr3, d.key0, d.key1, w);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bits |= ((w[j] & 0xFFFFu) >= d.t16 ? 1u : 0u) << (2 * j);
            bits |= ((w[j] >> 16) >= d.t16 ? 1u : 0u) << (2 * j + 1);
        }
        keep[pk - p0] = static_cast<uint8_t>(bits);
    }
}

template <typename T>
__device__ __forceinline__ void lds_rows_in(T* buf, const T* src, int64_t e0, int64_t e1, int64_t total)
{
    const int64_t p0 = e0 >> 3, p1 = (e1 + 7) >> 3;
    for (int64_t pk = p0 + threadIdx.x; pk < p1; pk += 256) {
        T* dst = buf + (pk - p0) * kPack;
        const int64_t base = pk * kPack;
        if (base + kPack <= total) {
            *reinterpret_cast<RawPack<T>*>(dst) = load_raw<T, true>(src + base);
        } else {
            for (int j = 0; j < kPack; ++j)
                if (base + j < total) dst[j] = src[base + j];
        }
    }
}

template <typename T>
__device__ __forceinline__ void lds_rows_out(T* dst, const T* buf, int64_t e0, int64_t e1)
{
    const int64_t p0 = e0 >> 3, p1 = (e1 + 7) >> 3;
    for (int64_t pk = p0 + threadIdx.x; pk < p1; pk += 256) {
        const T* from = buf + (pk - p0) * kPack;
        const int64_t base = pk * kPack;
        if (base >= e0 && base + kPack <= e1) {
            store_raw<T, true>(dst + base, *reinterpret_cast<const RawPack<T>*>(from));
        } else {
            for (int j = 0; j < kPack; ++j)
                if (base + j >= e0 && base + j < e1) dst[base + j] = from[j];
        }
    }
}

template <typename T, int LPR, int EPL, bool DROP>
__global__ __launch_bounds__(256) void softmax_fwd_lds(T* y, T* __restrict__ yd, const T* x, SoftmaxLens len, SoftmaxGeom g, DropoutParams d)
{
    constexpr int RPB = 256 / LPR, NBUF = lds_rows_elems<LPR, EPL>();
    __shared__ uint8_t keep[DROP ? NBUF / kPack : 1];
    __shared__ __align__(16) T xs[NBUF];
    __shared__ __align__(16) T ys[NBUF];
    __shared__ __align__(16) T yds[DROP ? NBUF : 8];
    const int sub = threadIdx.x % LPR;
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * RPB;
    const int64_t row = row0 + threadIdx.x / LPR;
    const bool rv = row < g.nrows;
    const int limit = rv ? row_limit(g, len, row) : 0;
    const int64_t ro = row * g.k_len;
    const int64_t e0 = row0 * g.k_len, e1 = min(row0 + RPB, g.nrows) * g.k_len;
    const int lo = static_cast<int>(ro - (e0 & ~static_cast<int64_t>(7)));     // this row's first element in LDS
    lds_rows_in<T>(xs, x, e0, e1, g.nrows * g.k_len);
    if constexpr (DROP) lds_keep_bits(keep, d, e0 >> 3, (e1 + 7) >> 3);
    __syncthreads();
    float v[EPL];
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        const int j = sub + m * LPR;
        v[m] = j < limit ? to_f32<T>(xs[lo + j]) * g.scale : -INFINITY;
    }
    float mx = v[0];
#pragma unroll
    for (int m = 1; m < EPL; ++m) mx = fmaxf(mx, v[m]);
    mx = group_max<LPR>(mx);
    const float mxs = (limit > 0 ? mx : 0.0f) * kLog2e;
    float z = 0.0f;
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        v[m] = __builtin_amdgcn_exp2f(fmaf(v[m], kLog2e, -mxs));
        z += v[m];
    }
    z = group_sum<LPR>(z);
    const float inv = limit > 0 ? 1.0f / z : 0.0f;
#pragma unroll
    for (int m = 0; m < EPL; ++m) v[m] *= inv;       // 0 beyond the limit (exp2(-inf)), and on empty rows
    if (__ballot(z != z) != 0) {                     // a NaN row stays NaN inside the mask only
#pragma unroll
        for (int m = 0; m < EPL; ++m) v[m] = sub + m * LPR < limit ? v[m] : 0.0f;
    }
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        const int j = sub + m * LPR;
        if (rv && j < g.k_len) {
            ys[lo + j] = from_f32<T>(v[m]);
            if constexpr (DROP) {
                const bool kept = (keep[(lo + j) >> 3] >> ((lo + j) & 7)) & 1;
                yds[lo + j] = from_f32<T>(kept ? v[m] * d.scale : 0.0f);
            }
        }
    }
    __syncthreads();
    lds_rows_out<T>(y, ys, e0, e1);
    if constexpr (DROP) lds_rows_out<T>(yd, yds, e0, e1);
}

template <typename T, int LPR, int EPL, bool DROP>
__global__ __launch_bounds__(256) void softmax_bwd_lds(T* dx, const T* dy, const T* __restrict__ y, SoftmaxLens len, SoftmaxGeom g, DropoutParams d)
{
    constexpr int RPB = 256 / LPR, NBUF = lds_rows_elems<LPR, EPL>();
    __shared__ uint8_t keep[DROP ? NBUF / kPack : 1];
    __shared__ __align__(16) T ysh[NBUF];
    __shared__ __align__(16) T gsh[NBUF];        // dy in, dx out
    const int sub = threadIdx.x % LPR;
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * RPB;
    const int64_t row = row0 + threadIdx.x / LPR;
    const bool rv = row < g.nrows;
    const int limit = rv ? row_limit(g, len, row) : 0;
    const int64_t ro = row * g.k_len;
    const int64_t e0 = row0 * g.k_len, e1 = min(row0 + RPB, g.nrows) * g.k_len;
    const int lo = static_cast<int>(ro - (e0 & ~static_cast<int64_t>(7)));
    lds_rows_in<T>(ysh, y, e0, e1, g.nrows * g.k_len);
    lds_rows_in<T>(gsh, dy, e0, e1, g.nrows * g.k_len);
    if constexpr (DROP) lds_keep_bits(keep, d, e0 >> 3, (e1 + 7) >> 3);
    __syncthreads();
    float yv[EPL], gv[EPL];
    float dot = 0.0f;
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        const int j = sub + m * LPR;
        yv[m] = j < limit ? to_f32<T>(ysh[lo + j]) : 0.0f;
        gv[m] = j < limit ? to_f32<T>(gsh[lo + j]) : 0.0f;
        if constexpr (DROP) {
            if (j < limit) {
                const bool kept = (keep[(lo + j) >> 3] >> ((lo + j) & 7)) & 1;
                gv[m] = kept ? gv[m] * d.scale : 0.0f;
            }
        }
        dot = fmaf(gv[m], yv[m], dot);
    }
    dot = group_sum<LPR>(dot);
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        const int j = sub + m * LPR;
        // every element is read and written by one lane only
        if (rv && j < g.k_len) gsh[lo + j] = from_f32<T>(j < limit ? g.scale * yv[m] * (gv[m] - dot) : 0.0f);
    }
    __syncthreads();
    lds_rows_out<T>(dx, gsh, e0, e1);
}

// ---- long rows (257..2048 packs: about 2048 < k_len <= 16384): one workgroup per row, VPL packs per thread in
// registers, the two reductions cross the four waves through LDS.  Still one read of the row.
template <typename T, int VPL, bool DROP, bool RAG, bool PAIR>
__global__ __launch_bounds__(256) void softmax_fwd_wide(T* y, T* __restrict__ yd, const T* x,
                                                        SoftmaxLens len, SoftmaxGeom g, DropoutParams d)
{
    __shared__ float red[4];
    using P = SmPacks<T, PAIR>;
    const int sub = P::pack(threadIdx.x);
    const int64_t row = blockIdx.x;
    const BlockRows<RAG> blk(g, row);
    const RowPacks<RAG> rp = blk.row(g, 0);
    x += blk.pack0 * kPack;
    y += blk.pack0 * kPack;
    if constexpr (DROP) yd += blk.pack0 * kPack;
    const int limit = row_limit(g, len, row);
    RawPack<T> raw[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        const int idx = sub + k * 256;
        if constexpr (P::kPaired) raw[k] = P::template load<true>(x + static_cast<unsigned>(rp.first + idx) * kPack, idx * kPack < limit);
        else if (idx * kPack - rp.s < limit) raw[k] = load_row_pack<T, 256, VPL, RAG>(x, rp, idx, blk.elems);
        else raw[k] = zero_raw<T>();
    }
    float v[VPL][8];
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        const int j0 = (sub + k * 256) * kPack - rp.s;
        unpack<T>(P::settle(raw[k]), v[k]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            bool in = j0 + j < limit;
            if constexpr (RAG) { if (k == 0) in = in && j0 + j >= 0; }
            v[k][j] = in ? v[k][j] * g.scale : -INFINITY;
            mx = fmaxf(mx, v[k][j]);
        }
    }
    mx = block_allreduce<4, OpMax>(mx, red);
    const float mxs = (limit > 0 ? mx : 0.0f) * kLog2e;
    float z = 0.0f;
#pragma unroll
    for (int k = 0; k < VPL; ++k)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float e = __builtin_amdgcn_exp2f(fmaf(v[k][j], kLog2e, -mxs));
            v[k][j] = e;
            z += e;
        }
    z = block_allreduce<4, OpSum, P::kPaired>(z, red);
    const float inv = limit > 0 ? 1.0f / z : 0.0f;
    RawPack<T> pk[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[k][j] *= inv;
        pk[k] = pack_raw<T>(v[k]);
    }
    const bool nan_row = z != z;                                          // uniform: a NaN row stays NaN inside the mask only
    if (nan_row) mask_packs<T, 256, false>(pk, sub, rp.s, limit);
    store_row<T, 256, VPL, RAG, PAIR>(y, rp, sub, true, false, g.k_len, pk);
    if constexpr (DROP) {
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = sub + k * 256;
            if (idx * kPack - rp.s < limit) {
                float kf[8];
                dropout_factors8(d, static_cast<uint64_t>(blk.pack0 + (rp.first + idx)), kf);
#pragma unroll
                for (int j = 0; j < 8; ++j) kf[j] *= v[k][j];
                pk[k] = pack_raw<T>(kf);
            }
        }
        if (nan_row) mask_packs<T, 256, true>(pk, sub, rp.s, limit, d, blk.pack0 + rp.first);
        store_row<T, 256, VPL, RAG, PAIR>(yd, rp, sub, true, false, g.k_len, pk);
    }
}

template <typename T, int VPL, bool DROP, bool RAG, bool PAIR>
__global__ __launch_bounds__(256) void softmax_bwd_wide(T* dx, const T* dy, const T* __restrict__ y,
                                                        SoftmaxLens len, SoftmaxGeom g, DropoutParams d)
{
    __shared__ float red[4];
    using P = SmPacks<T, PAIR>;
    const int sub = P::pack(threadIdx.x);
    const int64_t row = blockIdx.x;
    const BlockRows<RAG> blk(g, row);
    const RowPacks<RAG> rp = blk.row(g, 0);
    y += blk.pack0 * kPack;
    dy += blk.pack0 * kPack;
    dx += blk.pack0 * kPack;
    const int limit = row_limit(g, len, row);
    RawPack<T> ry[VPL], rg[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        const int idx = sub + k * 256;
        if constexpr (P::kPaired) {
            const unsigned e = static_cast<unsigned>(rp.first + idx) * kPack;
            ry[k] = P::template load<true>(y + e, idx * kPack < limit);
            rg[k] = P::template load<true>(dy + e, idx * kPack < limit);
        } else if (idx * kPack - rp.s < limit) {
            ry[k] = load_row_pack<T, 256, VPL, RAG>(y, rp, idx, blk.elems);
            rg[k] = load_row_pack<T, 256, VPL, RAG>(dy, rp, idx, blk.elems);
        } else {
            ry[k] = zero_raw<T>();
            rg[k] = zero_raw<T>();
        }
    }
    float yv[VPL][8], gv[VPL][8];
    float dot = 0.0f;
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        const int idx = sub + k * 256;
        const int j0 = idx * kPack - rp.s;
        unpack<T>(P::settle(ry[k]), yv[k]);
        unpack<T>(P::settle(rg[k]), gv[k]);
        if constexpr (DROP) {
            if (j0 < limit) {
                float kf[8];
                dropout_factors8(d, static_cast<uint64_t>(blk.pack0 + (rp.first + idx)), kf);
#pragma unroll
                for (int j = 0; j < 8; ++j) gv[k][j] *= kf[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            bool out = j0 + j >= limit;
            if constexpr (RAG) { if (k == 0) out = out || j0 + j < 0; }
            if (out) { yv[k][j] = 0.0f; gv[k][j] = 0.0f; }       // a neighbour's or a masked element never counts, NaN or not
            dot = fmaf(gv[k][j], yv[k][j], dot);
        }
    }
    dot = block_allreduce<4, OpSum, P::kPaired>(dot, red);
    RawPack<T> pk[VPL];
#pragma unroll
    for (int k = 0; k < VPL; ++k) {
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            o[j] = ((sub + k * 256) * kPack - rp.s + j < limit) ? g.scale * yv[k][j] * (gv[k][j] - dot) : 0.0f;
        pk[k] = pack_raw<T>(o);
    }
    store_row<T, 256, VPL, RAG, PAIR>(dx, rp, sub, true, false, g.k_len, pk);
}

// ---- rows of more than 2048 packs (beyond about 16384 keys): one workgroup per row, element-strided, the row is
// re-read from cache
template <typename T>
__global__ __launch_bounds__(256) void softmax_fwd_generic(T* y, T* __restrict__ yd, const T* x,
                                                           SoftmaxLens key_len, SoftmaxGeom g,
                                                           DropoutParams d)
{
    __shared__ float lds[4];
    constexpr int TH = 256;
    const int lane = threadIdx.x;
    const int64_t row = blockIdx.x;
    const int limit = row_limit(g, key_len, row);
    const int64_t ro = row * g.k_len;
    float mx = -INFINITY;
    for (int j = lane; j < limit; j += TH) mx = fmaxf(mx, to_f32<T>(x[ro + j]) * g.scale);
    mx = block_allreduce<4, OpMax>(mx, lds);
    const float mxs = (limit > 0 ? mx : 0.0f) * kLog2e;
    float z = 0.0f;
    for (int j = lane; j < limit; j += TH) z += __builtin_amdgcn_exp2f(fmaf(to_f32<T>(x[ro + j]) * g.scale, kLog2e, -mxs));
    z = block_allreduce<4, OpSum>(z, lds);
    const float inv = limit > 0 ? 1.0f / z : 0.0f;
    for (int j = lane; j < g.k_len; j += TH) {
        float o = 0.0f;
        if (j < limit) o = __builtin_amdgcn_exp2f(fmaf(to_f32<T>(x[ro + j]) * g.scale, kLog2e, -mxs)) * inv;
        y[ro + j] = from_f32<T>(o);
        if (yd) {
            const float f = dropout_factor1(d, static_cast<uint64_t>(ro + j));
            yd[ro + j] = from_f32<T>(f != 0.0f ? o * f : 0.0f);
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void softmax_bwd_generic(T* dx, const T* dy, const T* __restrict__ y,
                                                           SoftmaxLens key_len, SoftmaxGeom g,
                                                           DropoutParams d)
{
    __shared__ float lds[4];
    constexpr int TH = 256;
    const int lane = threadIdx.x;
    const int64_t row = blockIdx.x;
    const int limit = row_limit(g, key_len, row);
    const int64_t ro = row * g.k_len;
    float dot = 0.0f;
    for (int j = lane; j < limit; j += TH) {
        float gg = to_f32<T>(dy[ro + j]);
        if (d.on) {
            const float f = dropout_factor1(d, static_cast<uint64_t>(ro + j));
            gg = f != 0.0f ? gg * f : 0.0f;
        }
        dot = fmaf(gg, to_f32<T>(y[ro + j]), dot);
    }
    dot = block_allreduce<4, OpSum>(dot, lds);
    for (int j = lane; j < g.k_len; j += TH) {
        float o = 0.0f;
        if (j < limit) {
            float gg = to_f32<T>(dy[ro + j]);
            if (d.on) {
                const float f = dropout_factor1(d, static_cast<uint64_t>(ro + j));
                gg = f != 0.0f ? gg * f : 0.0f;
            }
            o = g.scale * to_f32<T>(y[ro + j]) * (gg - dot);
        }
        dx[ro + j] = from_f32<T>(o);
    }
}

// ------------------------------------------------------------------ dispatch
// packs per thread of the one-workgroup-per-row kernels for rows of np packs; 0: too long
inline int softmax_wide_vpl(int np) { return np <= 512 ? 2 : np <= 1024 ? 4 : np <= 2048 ? 8 : 0; }

// ---- launch shapes of the register path for rows of up to 2048 keys, and their choice at run time.
// The paper copes with the spread of softmax shapes by keeping several templates and searching for
// the best parameters before training starts (Sec. IV-B, Softmax, last paragraph).  Here a template
// is (lanes per row, packs per lane, rows per lane group); every row length has a short list of
// candidates, the first of which is the default, and lsq_softmax_tune times them on the caller's
// own buffers and records the winner per (row-length bucket, mask kind, dropout, storage width,
// direction), which the dispatch then uses.
struct SmCand { int lpr, vpl, rpt; };
constexpr int kSmBuckets = 10, kSmMaxCand = 4;
struct SmBucket { int max_packs, n; SmCand c[kSmMaxCand]; };
// Defaults measured on MI355X at the shapes of the five configurations (fp16): rows of 128 keys under a
// key-padding mask take 18.3 / 16.3 us (forward with attention dropout / backward) as 8 lanes x 2 packs
// against 20.6 / 18.2 us as 16 lanes x 1 pack, two rows per group: each of a lane's two loads then covers
// whole 128-byte lines of 8 rows, the first of which is issued before the sentence length has arrived.
static const SmBucket kSmTable[kSmBuckets] = {
    {1, 2, {{1, 1, 2}, {1, 1, 1}}},
    {2, 2, {{2, 1, 2}, {2, 1, 1}}},
    {4, 2, {{4, 1, 2}, {4, 1, 1}}},
    {8, 3, {{8, 1, 2}, {8, 1, 1}, {4, 2, 1}}},
    {16, 4, {{8, 2, 1}, {16, 1, 2}, {16, 1, 1}, {8, 2, 2}}},
    {32, 4, {{16, 2, 1}, {32, 1, 2}, {32, 1, 1}, {8, 4, 1}}},      // 256 keys, key padding: 32.0 / 26.7 us against 38.5 / 34.6 us as 32 x 1, two rows
    {64, 3, {{32, 2, 1}, {64, 1, 2}, {64, 1, 1}}},      // 512 keys, no mask: 44.5 / 63.9 us against 45.5 / 66.6 us as 64 x 1, two rows
    {128, 2, {{64, 2, 1}, {32, 4, 1}}},
    {192, 1, {{64, 3, 1}}},
    {256, 1, {{64, 4, 1}}},
};
#define LSQ_SM_CASES(X)                                                                                      \
    X(1, 1, 1) X(1, 1, 2) X(2, 1, 1) X(2, 1, 2) X(4, 1, 1) X(4, 1, 2) X(8, 1, 1) X(8, 1, 2) X(4, 2, 1)       \
    X(8, 2, 1) X(8, 2, 2) X(16, 1, 1) X(16, 1, 2) X(32, 1, 1) X(32, 1, 2) X(16, 2, 1) X(8, 4, 1)             \
    X(64, 1, 1) X(64, 1, 2) X(32, 2, 1) X(64, 2, 1) X(32, 4, 1) X(64, 3, 1) X(64, 4, 1)

inline int sm_bucket(int k_len)
{
    const int nv = k_len / kPack;
    for (int b = 0; b < kSmBuckets; ++b)
        if (nv <= kSmTable[b].max_packs) return b;
    return -1;
}

// what lsq_softmax_tune has recorded: [bucket][mask kind][dropout][storage width][direction], -1 = default
static std::atomic<signed char> sm_tuned[kSmBuckets][4][2][2][2];
static std::atomic<bool> sm_tuned_init{false};
static std::mutex sm_tuned_mutex;

inline void sm_tuned_prepare()
{
    if (sm_tuned_init.load(std::memory_order_acquire)) return;
    std::lock_guard<std::mutex> lock(sm_tuned_mutex);
    if (sm_tuned_init.load(std::memory_order_relaxed)) return;
    for (auto& a : sm_tuned) for (auto& b : a) for (auto& c : b) for (auto& e : c) for (auto& f : e) f.store(-1, std::memory_order_relaxed);
    sm_tuned_init.store(true, std::memory_order_release);
}

inline std::atomic<signed char>& sm_slot(int bucket, const SoftmaxLens& len, const SoftmaxGeom& g, bool drop, size_t elem, int dir)
{
    sm_tuned_prepare();
    const int mask = ((len.key || len.query) ? 1 : 0) + (g.causal ? 2 : 0);
    return sm_tuned[bucket][mask][drop ? 1 : 0][elem == 2 ? 0 : 1][dir];
}

// `forced` >= 0 picks that candidate of the row length's list; -1 the recorded one, else the default.
// A candidate with several rows per lane group falls back to one row when the grid would
// otherwise drop under kSmMinBlocks workgroups.
constexpr int64_t kSmMinBlocks = 1024;
inline SmCand sm_choose(const SoftmaxLens& len, const SoftmaxGeom& g, bool drop, size_t elem, int dir, int forced)
{
    const int b = sm_bucket(g.k_len);
    int pick = forced;
    if (pick < 0) pick = sm_slot(b, len, g, drop, elem, dir).load(std::memory_order_relaxed);
    if (pick < 0 || pick >= kSmTable[b].n) pick = 0;
    SmCand c = kSmTable[b].c[pick];
    if (c.rpt > 1 && ceil_div(g.nrows, 256 / c.lpr) < kSmMinBlocks * c.rpt) c.rpt = 1;
    return c;
}

// ---- rows that are not whole packs (k_len % 8 != 0): the packs a row can touch at most, and the shape for them.  A row
// starts at any multiple of gcd(k_len, 8) inside a pack.
inline int sm_ragged_packs(int k_len)
{
    int step = 1;
    while (step < kPack && k_len % (2 * step) == 0) step *= 2;
    return (kPack - step + k_len + kPack - 1) / kPack;
}
// Shapes by packs touched (lanes per row, packs per lane), one row per lane group (two cost 2-8 % here).  Three packs
// per lane fill the gaps between the powers of two, because a row needs a pack or two more than its elements fill.  The
// backward of short rows has fewer lanes with two or three packs each: 4 x 2 against 8 x 1 at 45 keys 11.5 against 14.4 us
// (dropout) and 10.3 against 12.5; the forward of those rows is faster the other way, 10.2 against 12.2 us.
struct SmRagged { int lpr, vpl; };
static const SmRagged kSmRaggedFwd[] = {{2, 1}, {4, 1}, {8, 1}, {4, 3}, {8, 2}, {8, 3}, {16, 2}, {16, 3}, {32, 2}, {32, 3}, {64, 2}, {64, 3}, {64, 4}};
static const SmRagged kSmRaggedBwd[] = {{2, 1}, {2, 2}, {4, 2}, {4, 3}, {8, 2}, {8, 3}, {16, 2}, {16, 3}, {32, 2}, {32, 3}, {64, 2}, {64, 3}, {64, 4}};
#define LSQ_SM_RAGGED_CASES(X)                                                                               \
    X(4, 3, 1) X(8, 2, 1) X(8, 3, 1) X(16, 2, 1) X(16, 3, 1) X(32, 2, 1) X(32, 3, 1) X(64, 2, 1) X(64, 3, 1) X(64, 4, 1)
#define LSQ_SM_RAGGED_FWD(X) X(2, 1, 1) X(4, 1, 1) X(8, 1, 1) LSQ_SM_RAGGED_CASES(X)
#define LSQ_SM_RAGGED_BWD(X) X(2, 1, 1) X(2, 2, 1) X(4, 2, 1) LSQ_SM_RAGGED_CASES(X)
template <int N>
inline SmCand sm_ragged_choose(const SmRagged (&table)[N], int np)
{
    for (const SmRagged& c : table)
        if (c.lpr * c.vpl >= np) return {c.lpr, c.vpl, 1};
    return {0, 0, 0};                       // not reached: the tables end at 256 packs
}

// ---- which rows that are not whole packs go through LDS instead (lpr = 0: none).  Both forms were measured at every such length up
// to 135 and some up to 2047 (fp16 and fp32; 1, 6, 20 and 48 M scores; no mask, key padding, causal; with and without dropout); the lines
// below are where the LDS form was the faster one.  Four things decide:
//  - how well the packs that a row touches fill the register shape: 5 to 8 packs in 8 lanes (29 keys fp16 forward 6.6 us against 8.9,
//    with dropout 9.5 against 13.7), and one pack more than a power of two, "brim" (127 keys with dropout 12.1 against 14.6);
//  - fp32 packs are two accesses and eight registers: short fp32 rows lose from about 12 keys on (29 keys with dropout 9.7 against 20 us);
//  - tensors beyond the 256 MB last-level cache ("far"), where a line that is written in pieces goes out twice (63 keys fp16 backward
//    of 48 M scores 52 us against 73); and calls of under 2 M scores ("small"), where the registers' longer code shows;
//  - a mask: the register form skips what lies beyond it, the LDS form reads it (`lens`: lengths given; `open`: no mask at all).
struct SmLds { int lpr, epl; };
inline SmLds sm_lds_shape(int dir, size_t elem, int k, bool drop, bool lens, bool causal, int64_t total)
{
    const bool open = !lens && !causal;
    const int64_t bytes = total * static_cast<int64_t>(elem) * (dir == 0 && !drop ? 2 : 3);
    const bool far = bytes > (static_cast<int64_t>(256) << 20), small = total < (1 << 21), mid = total >= (1 << 22);
    const int np = sm_ragged_packs(k);
    const bool brim8 = np == 9 && k < 64, brim16 = np == 17 && k < 128, brim32 = np == 33 && k < 256, brim64 = np == 65 && k < 512;
    bool lds = false;
    if (elem == 2 && dir == 0) {
        lds = (np >= 5 && np <= 8) || (brim8 && (drop || !lens)) || (np == 3 && k < 16 && (small || (drop && !lens))) ||
              (drop && ((brim16 && !lens) || (brim32 && (!lens || small)) || (brim64 && open))) ||
              (drop && k > 64 && ((k < 128 && !lens && far) || (k <= 112 && small) || (k > 128 && k < 190 && small)));
    } else if (elem == 2) {
        lds = (far && !drop && ((open && k >= 36 && k < 128) || (!lens && ((k >= 36 && k < 64) || (k > 102 && k < 128))))) ||
              (far && (brim8 || brim16) && (!drop || open)) || (mid && !drop && !lens && brim8) || (mid && !drop && open && brim32);
    } else if (dir == 0) {
        const bool filled = k == 52 || k == 60 || (k == 44 && !lens);    // whole half-packs, 6 to 8 of them: the register shape is full
        lds = (drop && k <= 58 && (k >= 12 || (k >= 10 && !small)) && !filled) ||
              (!drop && k <= 58 && (lens ? (k == 12 && mid) || k == 19 || k >= 21 : k >= 12) && !filled) ||
              (k >= 5 && k <= 7 && (small ? drop || k > 5 : drop && !lens && k > 5)) || (brim8 && (small || (open && !drop))) ||
              (k > 64 && k < 88 && (open || far || small)) || (far && drop && !causal && k >= 88 && k <= 108) || (far && open && k >= 88 && k <= 96) ||
              (drop && small && k > 96 && k < 190) || (open && far && k > 128 && k <= 175);
    } else {
        lds = (far && k >= (lens ? 20 : drop ? 14 : 10) && k <= (open ? 128 : 88)) || (far && open && k > 128 && k <= 195) ||
              (k >= 18 && k <= 28 && k != 27 && (!lens || k >= 21) && !(drop && k < 20)) || (!lens && !drop && k == 12) ||
              (small && !drop && !lens && (k == 7 || (k >= 13 && k <= 17))) ||
              (open && !drop && ((mid && k > 28 && k < 48) || (k > 64 && k < 88)));
    }
    if (!lds) return {0, 0};
    return k <= 8 ? SmLds{8, 1} : k <= 16 ? SmLds{8, 2} : k <= 32 ? SmLds{8, 4} : k <= 64 ? SmLds{8, 8} : k <= 128 ? SmLds{16, 8} : k <= 256 ? SmLds{32, 8} : SmLds{64, 8};
}
#define LSQ_SM_LDS_CASES(X) X(8, 1) X(8, 2) X(8, 4) X(8, 8) X(16, 8) X(32, 8) X(64, 8)

// fp32 rows in lane pairs (SmPacks): with a lane's pack as two 16-byte accesses 32 bytes apart each line is read and written in halves.  Time with consecutive
// packs and in pairs, forward with dropout / backward, us, inputs cold: 4 x 16 x 1024 x 1024 160 -> 134 / 151 -> 129, with padding 183 -> 128 / 105 -> 91;
// 8 x 16 x 512 x 512 80 -> 67 / 75 -> 65; 32 x 16 x 128 x 128 23.4 -> 19.0 / 20.6 -> 18.6; 64 x 16 x 64 x 64 14.7 -> 9.6 / 11.8 -> 11.0; 2 x 4 x 4096 x 4096
// causal 428 -> 237 / 202 -> 178.  Not where rows are not whole 128-byte lines (their pieces meet in the middle of a line: 1000 keys 55 -> 74 / 52 -> 57, 200 keys 32.5 -> 37.0
// forward), and not below 2 Mi scores, where the second address and the exchange are in the way of a few waves (16 x 8 x 1 x 512 3.4 -> 4.0 / 2.7 -> 3.5;
// 8 x 20 x 96 x 96 with padding 6.1 -> 6.4 / 5.1 -> 5.6).
inline bool sm_paired(size_t storage, const SoftmaxGeom& g) { return storage == 4 && g.k_len % 32 == 0 && g.nrows * g.k_len >= (1 << 21); }

// The paths by row length, with `np` the packs a row touches (base pointers are 16-byte aligned, checked at the entry):
// up to 256 packs the lanes of a wave, up to 2048 a workgroup per row, beyond that the element-strided kernels; each in a
// form for rows of whole packs and one for any other length.
template <typename T>
static lsq_status softmax_fwd_dispatch(void* y, void* yd, const void* x, SoftmaxLens key_len, const SoftmaxGeom& g,
                                       const DropoutParams& d, hipStream_t s, int forced = -1)
{
    T* yp = static_cast<T*>(y);
    T* ydp = static_cast<T*>(yd);
    const T* xp = static_cast<const T*>(x);
    const bool rag = g.k_len % kPack != 0;
    const int np = rag ? sm_ragged_packs(g.k_len) : g.k_len / kPack;
    const bool drop = d.on != 0, pair = sm_paired(sizeof(T), g);
    if (np > 256) {
        const dim3 grid(static_cast<unsigned>(g.nrows)), block(256);
        const int vpl = softmax_wide_vpl(np);
        if (vpl == 0) hipLaunchKernelGGL((softmax_fwd_generic<T>), grid, block, 0, s, yp, ydp, xp, key_len, g, d);
        constexpr bool kPair = sizeof(T) == 4;
#define W2(V, RAG, PAIR)                                                                                     \
            {                                                                                                \
                if (drop) hipLaunchKernelGGL((softmax_fwd_wide<T, V, true, RAG, PAIR>), grid, block, 0, s, yp, ydp, xp, key_len, g, d);   \
                else hipLaunchKernelGGL((softmax_fwd_wide<T, V, false, RAG, PAIR>), grid, block, 0, s, yp, ydp, xp, key_len, g, d);       \
            }
#define W(V)                                                                                                 \
        if (vpl == V) {                                                                                      \
            if (rag) W2(V, true, false)                                                                      \
            else if (pair) W2(V, false, kPair)                                                               \
            else W2(V, false, false)                                                                         \
        }
        W(2) W(4) W(8)
#undef W
#undef W2
        return launch_status();
    }
    if (rag) {
        const SmLds l = sm_lds_shape(0, sizeof(T), g.k_len, drop, key_len.key || key_len.query, g.causal != 0, g.nrows * g.k_len);
        if (l.lpr != 0) {
            const dim3 grid(static_cast<unsigned>(ceil_div(g.nrows, 256 / l.lpr)));
#define X(L, E)                                                                                              \
            if (l.lpr == L && l.epl == E) {                                                                  \
                if (drop) hipLaunchKernelGGL((softmax_fwd_lds<T, L, E, true>), grid, dim3(256), 0, s, yp, ydp, xp, key_len, g, d); \
                else hipLaunchKernelGGL((softmax_fwd_lds<T, L, E, false>), grid, dim3(256), 0, s, yp, ydp, xp, key_len, g, d);    \
            }
            LSQ_SM_LDS_CASES(X)
#undef X
            return launch_status();
        }
    }
    const SmCand c = rag ? sm_ragged_choose(kSmRaggedFwd, np) : sm_choose(key_len, g, drop, sizeof(T), 0, forced);
    const dim3 grid(static_cast<unsigned>(ceil_div(ceil_div(g.nrows, kSmWgFwd / c.lpr), c.rpt)));
#define XP(L, V, R, RAG, PAIR)                                                                               \
    {                                                                                                        \
        if (drop) hipLaunchKernelGGL((softmax_fwd_kernel<T, L, V, R, true, RAG, PAIR>), grid, dim3(kSmWgFwd), 0, s, yp, ydp, xp, key_len, g, d); \
        else hipLaunchKernelGGL((softmax_fwd_kernel<T, L, V, R, false, RAG, PAIR>), grid, dim3(kSmWgFwd), 0, s, yp, ydp, xp, key_len, g, d);    \
    }
#define XR(L, V, R, RAG)                                                                                     \
    if (rag == RAG && c.lpr == L && c.vpl == V && c.rpt == R) {                                              \
        constexpr bool kPair = sizeof(T) == 4 && !RAG && L >= 8;                                             \
        if (pair) XP(L, V, R, RAG, kPair)                                                                    \
        else XP(L, V, R, RAG, false)                                                                         \
    }
#define X(L, V, R) XR(L, V, R, false)
    LSQ_SM_CASES(X)
#undef X
#define X(L, V, R) XR(L, V, R, true)
    LSQ_SM_RAGGED_FWD(X)
#undef X
#undef XR
#undef XP
    return launch_status();
}

template <typename T>
static lsq_status softmax_bwd_dispatch(void* dx, const void* dy, const void* y, SoftmaxLens key_len,
                                       const SoftmaxGeom& g, const DropoutParams& d, hipStream_t s, int forced = -1)
{
    T* dxp = static_cast<T*>(dx);
    const T* dyp = static_cast<const T*>(dy);
    const T* yp = static_cast<const T*>(y);
    const bool rag = g.k_len % kPack != 0;
    const int np = rag ? sm_ragged_packs(g.k_len) : g.k_len / kPack;
    const bool drop = d.on != 0, pair = sm_paired(sizeof(T), g);
    if (np > 256) {
        const dim3 grid(static_cast<unsigned>(g.nrows)), block(256);
        const int vpl = softmax_wide_vpl(np);
        if (vpl == 0) hipLaunchKernelGGL((softmax_bwd_generic<T>), grid, block, 0, s, dxp, dyp, yp, key_len, g, d);
        constexpr bool kPair = sizeof(T) == 4;
#define W2(V, RAG, PAIR)                                                                                     \
            {                                                                                                \
                if (drop) hipLaunchKernelGGL((softmax_bwd_wide<T, V, true, RAG, PAIR>), grid, block, 0, s, dxp, dyp, yp, key_len, g, d);   \
                else hipLaunchKernelGGL((softmax_bwd_wide<T, V, false, RAG, PAIR>), grid, block, 0, s, dxp, dyp, yp, key_len, g, d);       \
            }
#define W(V)                                                                                                 \
        if (vpl == V) {                                                                                      \
            if (rag) W2(V, true, false)                                                                      \
            else if (pair) W2(V, false, kPair)                                                               \
            else W2(V, false, false)                                                                         \
        }
        W(2) W(4) W(8)
#undef W
#undef W2
        return launch_status();
    }
    if (rag) {
        const SmLds l = sm_lds_shape(1, sizeof(T), g.k_len, drop, key_len.key || key_len.query, g.causal != 0, g.nrows * g.k_len);
        if (l.lpr != 0) {
            const dim3 grid(static_cast<unsigned>(ceil_div(g.nrows, 256 / l.lpr)));
#define X(L, E)                                                                                              \
            if (l.lpr == L && l.epl == E) {                                                                  \
                if (drop) hipLaunchKernelGGL((softmax_bwd_lds<T, L, E, true>), grid, dim3(256), 0, s, dxp, dyp, yp, key_len, g, d); \
                else hipLaunchKernelGGL((softmax_bwd_lds<T, L, E, false>), grid, dim3(256), 0, s, dxp, dyp, yp, key_len, g, d);    \
            }
            LSQ_SM_LDS_CASES(X)
#undef X
            return launch_status();
        }
    }
    const SmCand c = rag ? sm_ragged_choose(kSmRaggedBwd, np) : sm_choose(key_len, g, drop, sizeof(T), 1, forced);
    const dim3 grid(static_cast<unsigned>(ceil_div(ceil_div(g.nrows, kSmWgBwd / c.lpr), c.rpt)));
#define XP(L, V, R, RAG, PAIR)                                                                               \
    {                                                                                                        \
        if (drop) hipLaunchKernelGGL((softmax_bwd_kernel<T, L, V, R, true, RAG, PAIR>), grid, dim3(kSmWgBwd), 0, s, dxp, dyp, yp, key_len, g, d); \
        else hipLaunchKernelGGL((softmax_bwd_kernel<T, L, V, R, false, RAG, PAIR>), grid, dim3(kSmWgBwd), 0, s, dxp, dyp, yp, key_len, g, d);    \
    }
#define XR(L, V, R, RAG)                                                                                     \
    if (rag == RAG && c.lpr == L && c.vpl == V && c.rpt == R) {                                              \
        constexpr bool kPair = sizeof(T) == 4 && !RAG && L >= 8;                                             \
        if (pair) XP(L, V, R, RAG, kPair)                                                                    \
        else XP(L, V, R, RAG, false)                                                                         \
    }
#define X(L, V, R) XR(L, V, R, false)
    LSQ_SM_CASES(X)
#undef X
#define X(L, V, R) XR(L, V, R, true)
    LSQ_SM_RAGGED_BWD(X)
#undef X
#undef XR
#undef XP
    return launch_status();
}

static lsq_status softmax_check(const void* a, const void* b, int32_t batch, int32_t heads, int32_t q_len,
                                int32_t k_len, float scale, int dt, SoftmaxGeom* g)
{
    (void)a; (void)b;
    if (batch < 0 || heads < 0 || q_len < 0 || k_len < 0) return LSQ_INVALID_ARG;
    if (!(scale == scale) || isinf(scale)) return LSQ_INVALID_ARG;
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    const int64_t rpb = static_cast<int64_t>(heads) * q_len;
    if (rpb > 0x7FFFFFFF) return LSQ_INVALID_ARG;
    g->nrows = static_cast<int64_t>(batch) * rpb;
    g->rows_per_batch = static_cast<int>(rpb);
    g->by_rows_per_batch = make_fastdiv(static_cast<uint32_t>(rpb));
    g->by_q_len = make_fastdiv(static_cast<uint32_t>(q_len));
    g->q_len = q_len;
    g->k_len = k_len;
    g->shift = k_len - q_len;
    g->scale = scale;
    if (g->nrows > 0x7FFFFFFF) return LSQ_INVALID_ARG;
    return LSQ_OK;
}

}  // namespace lsq

extern "C" lsq_status lsq_softmax_varlen_fwd(void* y, void* y_drop, const void* x, const int32_t* key_len,
                                             const int32_t* query_len, int32_t batch, int32_t heads, int32_t q_len,
                                             int32_t k_len, int32_t causal, float scale, float p_attn, uint64_t seed,
                                             uint64_t offset, lsq_dtype dt, void* stream)
{
    using namespace lsq;
    const SoftmaxLens len{key_len, query_len};
    SoftmaxGeom g;
    lsq_status st = softmax_check(y, x, batch, heads, q_len, k_len, scale, dt, &g);
    if (st != LSQ_OK) return st;
    g.causal = causal != 0;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p_attn, seed, offset, &d));
    LSQ_REQUIRE((d.on != 0) == (y_drop != nullptr));
    if (g.nrows == 0 || k_len == 0) return LSQ_OK;
    LSQ_REQUIRE(y && x);
    LSQ_ALIGNED(y); LSQ_ALIGNED(y_drop); LSQ_ALIGNED(x);
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (dt) {
        case LSQ_F16: return softmax_fwd_dispatch<f16>(y, y_drop, x, len, g, d, s);
        case LSQ_BF16: return softmax_fwd_dispatch<bf16>(y, y_drop, x, len, g, d, s);
        default: return softmax_fwd_dispatch<float>(y, y_drop, x, len, g, d, s);
    }
}

extern "C" lsq_status lsq_softmax_fwd(void* y, void* y_drop, const void* x, const int32_t* key_len, int32_t batch,
                                      int32_t heads, int32_t q_len, int32_t k_len, int32_t causal, float scale,
                                      float p_attn, uint64_t seed, uint64_t offset, lsq_dtype dt, void* stream)
{
    return lsq_softmax_varlen_fwd(y, y_drop, x, key_len, nullptr, batch, heads, q_len, k_len, causal, scale, p_attn,
                                  seed, offset, dt, stream);
}

extern "C" lsq_status lsq_softmax_varlen_bwd(void* dx, const void* dy, const void* y, const int32_t* key_len,
                                             const int32_t* query_len, int32_t batch, int32_t heads, int32_t q_len,
                                             int32_t k_len, int32_t causal, float scale, float p_attn, uint64_t seed,
                                             uint64_t offset, lsq_dtype dt, void* stream)
{
    using namespace lsq;
    const SoftmaxLens len{key_len, query_len};
    SoftmaxGeom g;
    lsq_status st = softmax_check(dx, dy, batch, heads, q_len, k_len, scale, dt, &g);
    if (st != LSQ_OK) return st;
    g.causal = causal != 0;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p_attn, seed, offset, &d));
    if (g.nrows == 0 || k_len == 0) return LSQ_OK;
    LSQ_REQUIRE(dx && dy && y);
    LSQ_ALIGNED(dx); LSQ_ALIGNED(dy); LSQ_ALIGNED(y);
    hipStream_t s = static_cast<hipStream_t>(stream);
    switch (dt) {
        case LSQ_F16: return softmax_bwd_dispatch<f16>(dx, dy, y, len, g, d, s);
        case LSQ_BF16: return softmax_bwd_dispatch<bf16>(dx, dy, y, len, g, d, s);
        default: return softmax_bwd_dispatch<float>(dx, dy, y, len, g, d, s);
    }
}

extern "C" lsq_status lsq_softmax_bwd(void* dx, const void* dy, const void* y, const int32_t* key_len, int32_t batch,
                                      int32_t heads, int32_t q_len, int32_t k_len, int32_t causal, float scale,
                                      float p_attn, uint64_t seed, uint64_t offset, lsq_dtype dt, void* stream)
{
    return lsq_softmax_varlen_bwd(dx, dy, y, key_len, nullptr, batch, heads, q_len, k_len, causal, scale, p_attn, seed,
                                  offset, dt, stream);
}

// ---- run-time choice of the launch shape (Sec. IV-B, Softmax: templates + parameter search before training)
extern "C" int32_t lsq_softmax_candidates(int32_t k_len)
{
    using namespace lsq;
    if (k_len <= 0 || k_len % kPack != 0) return 1;
    const int b = sm_bucket(k_len);
    return b < 0 ? 1 : kSmTable[b].n;
}

extern "C" lsq_status lsq_softmax_tune(int32_t* best_fwd, int32_t* best_bwd, float* us, void* y, void* y_drop, void* dx,
                                       const void* x, const void* dy, const int32_t* key_len, const int32_t* query_len,
                                       int32_t batch, int32_t heads, int32_t q_len, int32_t k_len, int32_t causal,
                                       float scale, float p_attn, uint64_t seed, uint64_t offset, lsq_dtype dt,
                                       int32_t force, int32_t reps, void* stream)
{
    using namespace lsq;
    const SoftmaxLens len{key_len, query_len};
    SoftmaxGeom g;
    lsq_status st = softmax_check(y, x, batch, heads, q_len, k_len, scale, dt, &g);
    if (st != LSQ_OK) return st;
    g.causal = causal != 0;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p_attn, seed, offset, &d));
    LSQ_REQUIRE(force >= -2 && reps >= 1 && reps <= 10000);
    if (best_fwd) *best_fwd = 0;
    if (best_bwd) *best_bwd = 0;
    if (us)
        for (int i = 0; i < 2 * kSmMaxCand; ++i) us[i] = -1.0f;
    const int ncand = lsq_softmax_candidates(k_len);
    const size_t elem = dt == LSQ_F32 ? 4 : 2;
    const bool drop = d.on != 0;
    const int b = sm_bucket(k_len);
    if (force != -1) {                       // set (>= 0) or forget (-2): nothing is launched
        LSQ_REQUIRE(force < ncand);
        if (ncand > 1) {
            sm_slot(b, len, g, drop, elem, 0).store(static_cast<signed char>(force < 0 ? -1 : force));
            sm_slot(b, len, g, drop, elem, 1).store(static_cast<signed char>(force < 0 ? -1 : force));
        }
        if (best_fwd) *best_fwd = force < 0 ? 0 : force;
        if (best_bwd) *best_bwd = force < 0 ? 0 : force;
        return LSQ_OK;
    }
    if (g.nrows == 0 || k_len == 0 || ncand <= 1) return LSQ_OK;
    LSQ_REQUIRE(y && x && dx && dy);
    LSQ_REQUIRE(drop == (y_drop != nullptr));
    LSQ_ALIGNED(y); LSQ_ALIGNED(y_drop); LSQ_ALIGNED(x); LSQ_ALIGNED(dx); LSQ_ALIGNED(dy);
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return LSQ_LAUNCH_FAILED;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return LSQ_LAUNCH_FAILED; }
    auto launch = [&](int dir, int cand) -> lsq_status {
        if (dir == 0) {
            switch (dt) {
                case LSQ_F16: return softmax_fwd_dispatch<f16>(y, y_drop, x, len, g, d, s, cand);
                case LSQ_BF16: return softmax_fwd_dispatch<bf16>(y, y_drop, x, len, g, d, s, cand);
                default: return softmax_fwd_dispatch<float>(y, y_drop, x, len, g, d, s, cand);
            }
        }
        switch (dt) {
            case LSQ_F16: return softmax_bwd_dispatch<f16>(dx, dy, y, len, g, d, s, cand);
            case LSQ_BF16: return softmax_bwd_dispatch<bf16>(dx, dy, y, len, g, d, s, cand);
            default: return softmax_bwd_dispatch<float>(dx, dy, y, len, g, d, s, cand);
        }
    };
    st = LSQ_OK;
    for (int dir = 0; dir < 2 && st == LSQ_OK; ++dir) {
        int best = 0;
        float best_ms = 0.0f;
        for (int c = 0; c < ncand && st == LSQ_OK; ++c) {
            for (int i = 0; i < 2 && st == LSQ_OK; ++i) st = launch(dir, c);          // warm-up
            if (st != LSQ_OK) break;
            float ms = 0.0f;
            bool ok = hipEventRecord(e0, s) == hipSuccess;
            for (int i = 0; i < reps && st == LSQ_OK; ++i) st = launch(dir, c);
            ok = ok && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                 hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
            if (!ok) st = LSQ_LAUNCH_FAILED;
            if (st != LSQ_OK) break;
            if (us) us[dir * kSmMaxCand + c] = ms * 1000.0f / static_cast<float>(reps);
            if (c == 0 || ms < best_ms) { best = c; best_ms = ms; }
        }
        if (st == LSQ_OK) {
            sm_slot(b, len, g, drop, elem, dir).store(static_cast<signed char>(best));
            if (dir == 0 && best_fwd) *best_fwd = best;
            if (dir == 1 && best_bwd) *best_bwd = best;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return st;
}
