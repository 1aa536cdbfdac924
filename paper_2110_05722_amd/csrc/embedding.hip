// Embedding layer, forward and backward (Sec. IV-A of the paper, embedding layer):
//   forward   y[t,:] = Dropout_p(scale * E[w_t,:] + P[l_t,:])
//   backward  dE[w,:] += scale * sum_{t: w_t = w} m_t (.) dy[t,:]      dP[l,:] += sum_b m (.) dy[b,l,:]
//
// The paper sums the gradient rows of a repeated token with atomicAdd.  Floating-point
// atomics make the result depend on the arrival order; here the sum has a fixed order
// instead, with no atomics at all:
//   1. order: the tokens of a call, equal ids together in ascending position.  Up to 16384 tokens a few
//      workgroups sort them, each the ids of one residue class, in LDS (stable radix sort), while the other workgroups
//      of the launch stream dy for dP; beyond that the sort runs over many workgroups, two launches per digit;
//   2. accumulate: workgroups take 64 entries of the sorted order and 16 packs of the columns and sum m (.) dy of equal
//      neighbours in ascending position in fp32; an id that goes on beyond its 64 entries has workgroups of its own
//      that share its columns, or beyond 16384 tokens leaves an fp32 row per 64 entries, which a last launch adds.
//      One rounding of dE per call either way.
// Tokens equal to pad_idx (or outside the vocabulary) produce zero rows and no gradient.
#include <limits.h>

#include "host.hpp"

namespace lsq {

constexpr bool kNT = true;
constexpr int kEmbWaves = 4;

__device__ __forceinline__ bool emb_is_pad(int w, int vocab, int pad_idx) { return w == pad_idx || w < 0 || w >= vocab; }

template <typename T, bool DROP, bool RAG>
__global__ __launch_bounds__(256) void emb_fwd_cols(T* __restrict__ out, const int32_t* __restrict__ tokens,
                                                    const T* __restrict__ emb, const T* __restrict__ pos, int64_t rows,
                                                    int len, RowPackIO<T, RAG> io, int vocab, int pad_idx, float scale,
                                                    DropoutParams d, FastDiv by_len)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cp = blockIdx.x * 64 + lane;
    if (cp >= io.ppr) return;
    const int64_t stride = static_cast<int64_t>(gridDim.y) * kEmbWaves;
    for (int64_t t = static_cast<int64_t>(blockIdx.y) * kEmbWaves + wave; t < rows; t += stride) {
        const int w = tokens[t];
        const int t31 = static_cast<int>(t);                         // tokens of a call are below 2^31 (checked at the entry): one 32 x 32 product
        float o[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (!emb_is_pad(w, vocab, pad_idx)) {
            const uint32_t t32 = static_cast<uint32_t>(t31);
            const int l = static_cast<int>(t32 - fastdiv(t32, by_len) * static_cast<uint32_t>(len));
            float e[8], pp[8];
            const RawPack<T> re = io.template ahead<false>(emb, w, cp), rp = io.template ahead<false>(pos, l, cp);
            unpack<T>(io.settle(re, cp), e);
            unpack<T>(io.settle(rp, cp), pp);
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = fmaf(scale, e[j], pp[j]);
            if constexpr (DROP) {
                float k[8];
                io.factors(d, t31, cp, k);
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] *= k[j];
            }
        }
        io.template store<kNT>(out, t31, cp, o);
    }
}

// Rows that are not whole packs, one element per thread: faster than a wave per row while the rows are narrow (few lanes have a pack) or
// the call small (two groups are drawn per pack).  32 x 1024 tokens, dropout, fp16, in us: 9 columns 3.7 against 17.9, 100 13.4 against 17.9,
// 161 20.1 against 18.6; 8 x 64 tokens, fp32: 257 3.2 against 3.6, 1001 4.4 against 3.9.
constexpr int kEmbFlatColumns = 145;
constexpr int64_t kEmbFlatElements = 400000;
template <typename T>
__global__ __launch_bounds__(256) void emb_fwd_flat(T* __restrict__ out, const int32_t* __restrict__ tokens,
                                                    const T* __restrict__ emb, const T* __restrict__ pos, int64_t rows,
                                                    int len, int hidden, int vocab, int pad_idx, float scale, DropoutParams d)
{
    const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (e >= rows * hidden) return;
    const int64_t t = e / hidden;
    const int i = static_cast<int>(e - t * hidden);
    const int w = tokens[t];
    float v = 0.0f;
    if (!emb_is_pad(w, vocab, pad_idx)) {
        v = fmaf(scale, to_f32<T>(emb[static_cast<int64_t>(w) * hidden + i]), to_f32<T>(pos[(t % len) * hidden + i]));
        if (d.on) v *= dropout_factor1(d, static_cast<uint64_t>(e));
    }
    out[e] = from_f32<T>(v);
}

// sort key of a token: its id, with padding last; kNoKey stands for "beyond the data"
constexpr unsigned kPadKey = 0x7FFFFFFFu;
constexpr unsigned kNoKey = 0xFFFFFFFFu;
__device__ __forceinline__ unsigned emb_key(int w, int vocab, int pad_idx)
{
    return emb_is_pad(w, vocab, pad_idx) ? kPadKey : static_cast<unsigned>(w);
}

// The order of up to kEmbSortMax tokens, without a launch of its own: 64 workgroups (128 beyond 8192 tokens), each for the ids of one class.
// What the accumulation needs is that equal ids stand together in ascending position; which id comes before
// which is free, so a class can be any set of ids whose share does not follow from their frequency (frequent words have
// small ids) or their spacing: the low bits of the id with the next two groups of bits folded in (sort_mix).  A workgroup looks at every token
// once, keeps the positions of its ids and counts those of the parts before it, which is where its own begin.  An entry is 32
// bits, what the part leaves of the id and the position: no two are equal, so a part of up to kSortRank entries needs no order on
// its way into LDS (a lane writes its own one after the other) and is sorted by counting the smaller ones of every entry.  Larger
// parts are kept in order and sorted by the rest of the id: a stable least-
// significant-digit radix sort, at most 6 bits per pass.  The lanes of a round of 64 entries that hold the same digit find
// each other with ballots, the lowest takes as many places as they are from the wave's counter of that digit (waves
// apart: nothing depends on timing), in LDS, or in the workspace where a part is larger than kSortLds.  Padding is not
// sorted: what is left of `order` behind the live tokens is filled with it.
// A part larger than kSortRank has a frequent id in it nearly always.  Of four ids that lanes of a wave meet first, the one that most
// lanes do is taken out of the sort: its positions need none, they go to the end of the part's range in the order they are met.
// What bounds it is the latency of its steps, in cycles of the slowest part at 8192 tokens (words, vocabulary 50257): tokens, keys and counts
// 4900, sums 600, the frequent id 2800, into LDS 7100, sort 1800; 17200 together, 26600 when every part went through the radix sort, in order,
// and the frequent id was found by a vote of all lanes.  Whole backward, bf16, in us before and now: 8192 x 1280 words 31.5 / 28.6
// (without dP 31.1 / 27.5), one id everywhere 56 / 54, half of them 43 / 41, multiples of 64 32.5 / 30; 16384 x 1024 words 44.6 / 41 (128 parts);
// 790 x 600 15.7 / 13.4.  One 1024-thread workgroup for all of 8192 tokens took 20 us; with the ids read again from the
// tokens in every round instead of carried, the part of the most frequent word took 19.
constexpr int kSortDigits = 64, kSortLds = 2048, kSortRank = 256;
// How an id is split: `part_bits` low bits choose the part (64 parts; 128 beyond 8192 tokens, where parts of 64 would be too large to
// rank, and where that makes a 31-bit id of a small call fit), the
// rest shares a 32-bit entry with the `pos_bits` bits of a position.
struct EmbSortPlan { int part_bits, pos_bits, passes, pass_bits; bool fits; };
inline EmbSortPlan emb_sort_plan(int64_t rows, int bits)
{
    EmbSortPlan p;
    p.pos_bits = 1;
    while ((static_cast<int64_t>(1) << p.pos_bits) < rows) ++p.pos_bits;
    p.part_bits = rows > 8192 || (bits > 32 - p.pos_bits + 6 && rows <= 256) ? 7 : 6;
    p.fits = rows <= kEmbSortMax && bits <= 32 - p.pos_bits + p.part_bits;
    const int rest = bits > p.part_bits ? bits - p.part_bits : 1;
    p.passes = (rest + 5) / 6;
    p.pass_bits = (rest + p.passes - 1) / p.passes;
    return p;
}
constexpr int kSortLdsBytes = 2 * kSortLds * 4 + 4 * kSortDigits * 4 + 16 * 4;

// An id with its low `part_bits` bits replaced by its class.  Its own inverse: the bits above are the id's.
__device__ __forceinline__ unsigned sort_mix(unsigned id, int part_bits)
{
    return id ^ (((id >> part_bits) ^ (id >> (2 * part_bits))) & ((1u << part_bits) - 1u));
}

// src -> (passes) -> order; src and tmp hold n entries each
__device__ __forceinline__ void emb_sort_part(int* cnt, uint32_t* src, uint32_t* tmp, int n, int part, int2* __restrict__ order,
                                              const EmbSortPlan& pl)
{
    const int passes = pl.passes, pass_bits = pl.pass_bits;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rounds = (n + 255) / 256;
    const int first = wave * rounds * kWave + lane;              // entry of round r: first + 64 r
    const unsigned mask = (1u << pass_bits) - 1u;
    // calls f(whether there is one, the entry, its digit's counter, the lanes of the round with that digit) round by round
    auto walk = [&](int shift, auto&& f) {
        for (int r = 0; r < rounds; ++r) {
            const int i = first + r * kWave;
            const bool valid = i < n;
            const uint32_t e = valid ? src[i] : 0u;
            const unsigned digit = (e >> shift) & mask;
            uint64_t same = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                if (b < pass_bits) {
                    const uint64_t has = __ballot((digit >> b) & 1);
                    same &= ((digit >> b) & 1) ? has : ~has;
                }
            }
            if (!valid) same = 1ull << lane;
            f(valid, e, &cnt[wave * kSortDigits + digit], same);
        }
    };
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pl.pos_bits + pass_bits * pass;
        cnt[threadIdx.x] = 0;                                    // 4 waves x 64 digits
        __syncthreads();
        walk(shift, [&](bool valid, uint32_t, int* c, uint64_t same) {
            if (valid && lane == __builtin_ctzll(same)) *c += __popcll(same);
        });
        __syncthreads();
        if (wave == 0) {                                         // lane = digit: starts in (digit, wave) order
            int c[4], total = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) c[w] = cnt[w * kSortDigits + lane];
#pragma unroll
            for (int w = 0; w < 4; ++w) total += c[w];
            int incl = total;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(incl, o);
                if (lane >= o) incl += v;
            }
            int at = incl - total;
#pragma unroll
            for (int w = 0; w < 4; ++w) { cnt[w * kSortDigits + lane] = at; at += c[w]; }
        }
        __syncthreads();
        const bool last = pass == passes - 1;
        walk(shift, [&](bool valid, uint32_t e, int* c, uint64_t same) {
            const int leader = __builtin_ctzll(same);
            int to = 0;
            if (valid && lane == leader) { to = *c; *c = to + __popcll(same); }
            to = __shfl(to, leader) + __popcll(same & ((1ull << lane) - 1ull));
            if (valid) {
                if (last) order[to] = make_int2(static_cast<int>(e & ((1u << pl.pos_bits) - 1u)),
                                                static_cast<int>(sort_mix((e >> pl.pos_bits) << pl.part_bits | static_cast<unsigned>(part), pl.part_bits)));
                else tmp[to] = e;
            }
        });
        __syncthreads();
        uint32_t* t = src; src = tmp; tmp = t;
    }
}

// inclusive sum over the lanes up to this one (row shifts, then the row totals handed on)
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // row_bcast 15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);      // row_bcast 31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ int wave_total(int scanned) { return __builtin_amdgcn_readlane(scanned, 63); }

// up to kSortRank entries in any order -> order: an entry's place is the number of smaller ones (no two are equal), counted by
// 1, 2 or 4 neighbouring threads per entry.  The entries lie in LDS, kNoKey behind them up to a multiple of sixteen.
__device__ __forceinline__ void emb_rank_part(const uint32_t* src, int n, int part, int2* __restrict__ order, const EmbSortPlan& pl)
{
    if (n == 0) return;                                                   // uniform
    const int each = n <= 64 ? 4 : n <= 128 ? 2 : 1;                      // uniform
    const int i = static_cast<int>(threadIdx.x) / each, q = static_cast<int>(threadIdx.x) % each;
    const uint32_t e = src[min(i, n - 1)];
    int rank = 0;
    for (int k = 16 * q; k < n; k += 16 * each) {
        uvec4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const uvec4*>(src + k + 4 * u);
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += (v[u].x < e ? 1 : 0) + (v[u].y < e ? 1 : 0) + (v[u].z < e ? 1 : 0) + (v[u].w < e ? 1 : 0);
    }
    if (each >= 2) rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xF, 0xF, false);      // quad_perm [1,0,3,2]
    if (each >= 4) rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xF, 0xF, false);      // quad_perm [2,3,0,1]
    if (i < n && q == 0)
        order[rank] = make_int2(static_cast<int>(e & ((1u << pl.pos_bits) - 1u)),
                                static_cast<int>(sort_mix((e >> pl.pos_bits) << pl.part_bits | static_cast<unsigned>(part), pl.part_bits)));
}

__device__ __forceinline__ void emb_sort_body(char* lds, int part, int2* __restrict__ order, uint32_t* __restrict__ spill,
                                              const int32_t* __restrict__ tokens, int rows, const EmbSortPlan& pl,
                                              int vocab, int pad_idx)
{
    const int parts = 1 << pl.part_bits;
    __builtin_amdgcn_s_setprio(3);      // a chain of short steps: its instructions go before those of the dP waves on the same unit
    uint32_t* in_lds = reinterpret_cast<uint32_t*>(lds);                                  // [2][kSortLds]
    int* cnt = reinterpret_cast<int*>(lds + 2 * kSortLds * 4);                            // [4][kSortDigits]
    int* sums = cnt + 4 * kSortDigits;                                                    // [3][4]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rounds = (rows + 255) / 256;
    const int first = wave * rounds * kWave + lane;              // token of round r: first + 64 r
    const int end = min(rows, (wave + 1) * rounds * kWave);      // of the wave's tokens
    constexpr int U = 32;                                        // rounds whose loads are in flight together (8192 tokens, half of the most)
    static_assert(2 * U * 256 >= kEmbSortMax, "two halves");
    unsigned key[U];
    auto load = [&](int r0) {
        int w[U];
        const int left = end - first - r0 * kWave;
#pragma unroll
        for (int g = 0; g < U; g += 8) {
            if (r0 + g < rounds) {                               // uniform; loads only, all in flight
#pragma unroll
                for (int u = g; u < g + 8; ++u) {                // a scalar base and a 32-bit offset
                    const uint32_t at = 4u * static_cast<uint32_t>(min(first + (r0 + u) * kWave, rows - 1));
                    w[u] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(tokens) + at);
                }
            } else {
#pragma unroll
                for (int u = g; u < g + 8; ++u) w[u] = pad_idx;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool there = (u * kWave < left) & (w[u] != pad_idx) & (static_cast<unsigned>(w[u]) < static_cast<unsigned>(vocab));
            const unsigned mixed = sort_mix(static_cast<unsigned>(w[u]), pl.part_bits);      // (selected, not branched over)
            key[u] = there ? mixed : kNoKey;
        }
    };
    const unsigned cls = 0x80000000u | static_cast<unsigned>(parts - 1);        // what of a key says whether and where it belongs
    auto member = [&](unsigned k) { return ((k ^ static_cast<unsigned>(part)) & cls) == 0; };
    int mine = 0, below = 0, live = 0;                           // of the lane, then of the wave
    for (int r0 = 0; r0 < rounds; r0 += U) {
        load(r0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned c = key[u] & cls;
            mine += c == static_cast<unsigned>(part) ? 1 : 0;
            below += c < static_cast<unsigned>(part) ? 1 : 0;
            live += static_cast<int>(key[u]) >= 0 ? 1 : 0;
        }
    }
    // a lane has at most 64 of each, a wave 4096: two of the sums share a register
    const int mine_upto = wave_scan(mine), others = wave_total(wave_scan(below | live << 16));
    if (lane == 0) { sums[wave] = wave_total(mine_upto); sums[4 + wave] = others & 0xFFFF; sums[8 + wave] = others >> 16; }
    __syncthreads();
    int to = 0, n = 0, base = 0, all = 0;                        // the wave's first place in the part; the part's size and begin; live tokens
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int c = sums[w];
        to += w < wave ? c : 0;
        n += c;
        base += sums[4 + w];
        all += sums[8 + w];
    }
    unsigned frequent = kNoKey - 1u;                             // no id
    int tf = 0;                                                  // its first place for the wave, behind the n others
    int lane_to = mine_upto - mine;                              // the lane's first place among the wave's, in any order
    const bool heavy = n > kSortRank;                            // uniform over the workgroup
    if (heavy) {
        unsigned met = kNoKey;                                   // the first id of the part that the lane holds
#pragma unroll
        for (int u = U - 1; u >= 0; --u) met = member(key[u]) ? key[u] : met;
        // each of four lanes spread over the wave proposes its own; the one that most lanes met is the wave's
        const uint64_t has = __ballot(met != kNoKey);
        int most = 0;
        unsigned elect = kNoKey;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint64_t from = has >> (16 * c) << (16 * c);
            if (from == 0) continue;                             // uniform over the wave
            const unsigned id = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(met), __builtin_ctzll(from)));
            const int votes = __popcll(__ballot(met == id));
            if (votes > most) { most = votes; elect = id; }
        }
        __syncthreads();                                         // everyone has read the sums
        if (lane == 0) { sums[wave] = most; sums[4 + wave] = static_cast<int>(elect); }
        __syncthreads();
        most = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (sums[w] > most) { most = sums[w]; frequent = static_cast<unsigned>(sums[4 + w]); }
        int c = 0, nf = 0;
        for (int r0 = rounds > U ? U : 0; r0 >= 0; r0 -= U) {    // the half that is here; the next loop begins with the first one
            if (r0 + U < rounds) load(r0);
#pragma unroll
            for (int u = 0; u < U; ++u) c += key[u] == frequent ? 1 : 0;
        }
        const int c_upto = wave_scan(c);
        lane_to -= c_upto - c;
        if (lane == 0) sums[8 + wave] = wave_total(c_upto);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            tf += w < wave ? sums[8 + w] : 0;
            nf += sums[8 + w];
        }
        to -= tf;
        n -= nf;
    }
    uint32_t* big0 = spill + base;                               // parts are disjoint: base + n <= live tokens <= rows
    uint32_t* big1 = spill + rows + base;
    const bool fits = n <= kSortLds, rank = n <= kSortRank;      // uniform over the workgroup
    lane_to += to;
    const uint64_t before = (1ull << lane) - 1ull;
    auto keep = [&](unsigned k, bool in, int pos) {
        const uint64_t m = __ballot(in);
        if (m != 0) {
            if (in) {
                const int at = to + __popcll(m & before);
                const uint32_t e = (k >> pl.part_bits) << pl.pos_bits | static_cast<uint32_t>(pos);
                if (fits) in_lds[at] = e;
                else big0[at] = e;
            }
            to += __popcll(m);
        }
    };
    for (int r0 = 0; r0 < rounds; r0 += U) {
        if (rounds > U && (r0 > 0 || !heavy)) load(r0);          // up to U rounds they are still here
        if (heavy) {                                             // the frequent id's positions, ascending
            const int id = static_cast<int>(sort_mix(frequent, pl.part_bits));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u % 8 == 0 && r0 + u >= rounds) break;       // uniform
                const bool out = key[u] == frequent;
                const uint64_t m = __ballot(out);
                if (out) order[base + n + tf + __popcll(m & before)] = make_int2(first + (r0 + u) * kWave, id);
                tf += __popcll(m);
                key[u] = out ? kNoKey : key[u];
            }
        }
        if (rank) {                                              // no order needed: a lane writes its own one after the other
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u % 8 == 0 && r0 + u >= rounds) break;
                if (member(key[u])) in_lds[lane_to++] = (key[u] >> pl.part_bits) << pl.pos_bits | static_cast<uint32_t>(first + (r0 + u) * kWave);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u % 8 == 0 && r0 + u >= rounds) break;
                keep(key[u], member(key[u]), first + (r0 + u) * kWave);
            }
        }
    }
    if (rank && threadIdx.x < 16) in_lds[n + threadIdx.x] = kNoKey;
    for (int i = all + part * 256 + static_cast<int>(threadIdx.x); i < rows; i += parts * 256)
        order[i] = make_int2(0, static_cast<int>(kPadKey));
    __syncthreads();
    if (rank) emb_rank_part(in_lds, n, part, order + base, pl);
    else if (fits) emb_sort_part(cnt, in_lds, in_lds + kSortLds, n, part, order + base, pl);
    else emb_sort_part(cnt, big0, big1, n, part, order + base, pl);
}

// ---- the same order for MANY tokens: beyond kEmbSortMax the (token, key) pairs go through the same kind of
// sort over many workgroups, 8 bits per pass over the bits an id can have (two
// passes up to 65535 ids).  A workgroup owns 2048 consecutive entries, striped over its 256
// threads (entry j*256 + i is item j of thread i), so that "round j, wave w, lane l" is ascending
// position.  Per pass: digit histogram per workgroup (integer LDS atomics: the counts do not depend
// on arrival order), exclusive scan of the [digit][workgroup] table (its own kernel only for very
// many workgroups), and the scatter, which hands out slots in position order: the lanes of a wave that hold the same digit find
// each other with 8 ballots, and the four waves take their turns on the running LDS counters.
constexpr int kRadixItems = 8;
constexpr int kRadixBlock = 256 * kRadixItems;
constexpr int kRadixFuseScan = 512;       // up to this many workgroups (2^20 tokens) the scatter scans its own offsets

__device__ __forceinline__ int2 radix_item(const int2* __restrict__ src, const int32_t* __restrict__ tokens, int64_t i,
                                           int vocab, int pad_idx)
{
    if (src) return src[i];
    return make_int2(static_cast<int>(i), static_cast<int>(emb_key(tokens[i], vocab, pad_idx)));   // first pass: the ids themselves
}

__global__ __launch_bounds__(256) void emb_radix_hist(int32_t* __restrict__ hist, const int2* __restrict__ src,
                                                      const int32_t* __restrict__ tokens, int64_t rows, int nblocks,
                                                      int shift, int vocab, int pad_idx)
{
    __shared__ int cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kRadixBlock;
#pragma unroll
    for (int j = 0; j < kRadixItems; ++j) {
        const int64_t i = base + j * 256 + threadIdx.x;
        if (i < rows) atomicAdd(&cnt[(radix_item(src, tokens, i, vocab, pad_idx).y >> shift) & 255], 1);
    }
    __syncthreads();
    hist[static_cast<int64_t>(threadIdx.x) * nblocks + blockIdx.x] = cnt[threadIdx.x];      // digit-major
}

// exclusive scan of n counts in place, one workgroup: every thread owns a contiguous piece
__global__ __launch_bounds__(1024) void emb_radix_scan(int32_t* __restrict__ hist, int64_t n)
{
    __shared__ int wave_sum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t per = (n + 1023) / 1024;
    const int64_t lo = min(n, tid * per), hi = min(n, lo + per);
    int sum = 0;
    for (int64_t i = lo; i < hi; ++i) sum += hist[i];
    int incl = sum;                                              // inclusive scan over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = incl - sum;
    for (int w = 0; w < wave; ++w) before += wave_sum[w];
    for (int64_t i = lo; i < hi; ++i) {
        const int c = hist[i];
        hist[i] = before;
        before += c;
    }
}

// SCANNED: `offs` went through emb_radix_scan.  Otherwise it holds the raw counts and the workgroup
// derives its own 256 offsets: thread = digit adds up its row of the table (all of it, and the part
// before this workgroup), and an exclusive scan over the 256 row sums finishes it; one launch less per
// pass, worth it while a row of the table is short.
template <bool SCANNED>
__global__ __launch_bounds__(256) void emb_radix_scatter(int2* __restrict__ dst, const int32_t* __restrict__ offs,
                                                         const int2* __restrict__ src, const int32_t* __restrict__ tokens,
                                                         int64_t rows, int nblocks, int shift, int vocab, int pad_idx)
{
    __shared__ int next[256];                  // next slot of each digit, for this workgroup's entries
    __shared__ int wave_sum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if constexpr (SCANNED) {
        next[tid] = offs[static_cast<int64_t>(tid) * nblocks + blockIdx.x];
    } else {
        const int32_t* row = offs + static_cast<int64_t>(tid) * nblocks;
        int total = 0, mine = 0;
        const int me = blockIdx.x;
#pragma unroll 8
        for (int b = 0; b < nblocks; ++b) {
            const int c = row[b];
            total += c;
            mine += b < me ? c : 0;
        }
        int incl = total;                                        // inclusive scan of the row sums over the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        int before = incl - total;
        for (int w = 0; w < wave; ++w) before += wave_sum[w];
        next[tid] = before + mine;
    }
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kRadixBlock;
    for (int j = 0; j < kRadixItems; ++j) {                      // uniform trip count: every thread reaches every barrier
        const int64_t i = base + j * 256 + tid;
        const bool valid = i < rows;
        const int2 item = valid ? radix_item(src, tokens, i, vocab, pad_idx) : make_int2(0, 0);
        const int digit = (item.y >> shift) & 255;
        uint64_t same = __ballot(valid);                         // lanes of this wave with my digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t has = __ballot((digit >> b) & 1);
            same &= ((digit >> b) & 1) ? has : ~has;
        }
        if (!valid) same = 0;
        const int below = __popcll(same & ((1ull << lane) - 1ull));
        const int leader = same ? __builtin_ctzll(same) : lane;
        int slot = 0;
        for (int w = 0; w < 4; ++w) {                            // waves in order: ascending position
            if (wave == w && valid && lane == leader) {          // one lane per digit present in the wave
                slot = next[digit];
                next[digit] = slot + __popcll(same);
            }
            __syncthreads();
        }
        slot = __shfl(slot, leader);
        if (valid) dst[slot + below] = item;
    }
}

// The sorted order is cut into units of kEmbUnit entries, ranges of kEmbRange entries and column blocks of 16 packs.  A workgroup takes a
// (range, column block): 16 lanes own a unit's entries, a wave has four units, so no lane idles on a row's last packs, and what a unit's first or last
// run shares with the unit beside it goes over by lane shuffles in a wave and LDS between the four.  A run that crosses the border of a range has
// workgroups of its own (emb_border_run) and is left out here, or leaves its sum of the range in memory (PARTS, emb_range_runs).  The destination rows are fetched together with the dy rows.
// What bounds it is the chain order -> rows -> rows of dE; 4 waves per SIMD at 8192 x 1280.  One wave per (8 entries, 64 packs), which left an fp32 row
// for every run that crossed its entries, and a last launch that added these took 13.1 + 6.0 us there; whole backward, bf16 with dropout, in us before and now:
// 8192 x 1280 words 28.6 / 23.4, distinct 29.0 / 23.7, half of one id 40.5 / 31.8, 16384 x 1024 40.9 / 36.4, 2048 x 768 f16 15.3 / 12.6.  Units of 8 entries,
// ranges before borders and 128 registers forced were slower.
constexpr int kEmbUnit = 4;
// dy is read twice in a call, by token and by position: through the caches (8192 x 1280 24.1 us, 26.2 past them, 16384 x 1024 37.6 / 41.2)
static_assert(kEmbRange == 16 * kEmbUnit, "four waves of four units");

__device__ __forceinline__ bool emb_live_key(int key) { return key >= 0 && key != static_cast<int>(kPadKey); }
// key of an entry; beyond the data kNoKey (-1 as int), which equals no token's key
__device__ __forceinline__ int emb_key_at(const int2* __restrict__ order, int64_t i, int64_t rows)
{
    return i >= 0 && i < rows ? order[i].y : static_cast<int>(kNoKey);
}

// PARTS (beyond the in-LDS sort's tokens): a run that crosses borders is not left out, the range's share of it goes to one of the range's two fp32 rows of `part` ([2 * ranges]
// rows of whole packs: the share of the run that came in, or fills the range, and of the one that goes on), and emb_join adds these.  The columns of a run
// end at 16 workgroups per column block, and in slices of one pack, which read an eighth of a line each; thousands of its rows are too long for them.  Whole backward,
// us, windows of 8 entries / shared columns / an fp32 row per range: words, 1280 bf16, 2^15 tokens 95.5 / 86.6 / 82.1, 2^16 144 / 140 / 121, 2^17 240 / 274 / 210; half of one
// id 2^15 145 / 110 / 81, 2^16 248 / 189 / 119; 500 ids, 1001 f16 2^15 96.0 / 101.2 / 93.8.  Up to 16384 tokens the launch more costs what it gives (8192 x 1280 words 21.5 / 24.1, ids
// without a word's frequencies 16384 x 1280 47.2 / 37.0 / 40.0); beyond, only such ids of narrow rows lose (20480 x 64 uniform 39.2 / 42.8).
template <typename T, bool DROP, bool RAG, bool PARTS>
__device__ __forceinline__ void emb_range_runs(float* lds, T* __restrict__ demb, const T* __restrict__ dy, const int2* __restrict__ order,
                                               float* __restrict__ part, int64_t range, int64_t rows, int cb, const RowPackIO<T, RAG>& io,
                                               float scale, const DropoutParams& d)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, c = cb * 16 + (lane & 15);
    const bool mine = c < io.ppr;
    const int cp = min(c, io.ppr - 1);
    const int64_t base = range * kEmbRange + (wave * 4 + grp) * kEmbUnit;
    // `order` has room for whole ranges: what lies beyond the data is read and not used
    int key[kEmbUnit + 1], tok[kEmbUnit];
#pragma unroll
    for (int k = 0; k < kEmbUnit; k += 2) {
        const uvec4 v = *reinterpret_cast<const uvec4*>(order + base + k);
        tok[k] = static_cast<int>(v.x); key[k] = static_cast<int>(v.y);
        tok[k + 1] = static_cast<int>(v.z); key[k + 1] = static_cast<int>(v.w);
    }
    key[kEmbUnit] = emb_key_at(order, base + kEmbUnit, rows);
    const int prev = emb_key_at(order, base - 1, rows);
    const int before = emb_key_at(order, range * kEmbRange - 1, rows), after = emb_key_at(order, (range + 1) * kEmbRange, rows);
#pragma unroll
    for (int k = 0; k < kEmbUnit; ++k)
        if (base + k >= rows) key[k] = static_cast<int>(kNoKey);
    bool live[kEmbUnit], ends[kEmbUnit];
#pragma unroll
    for (int k = 0; k < kEmbUnit; ++k) live[k] = emb_live_key(key[k]) && (PARTS || (key[k] != before && key[k] != after));
#pragma unroll
    for (int k = 0; k < kEmbUnit; ++k) ends[k] = live[k] && key[k] != key[k + 1];
    const bool first_unit = PARTS && wave == 0 && grp == 0, last_unit = PARTS && wave == 3 && grp == 3;
    if (last_unit) ends[kEmbUnit - 1] = live[kEmbUnit - 1];        // the range's share of a run ends with the range
    RawPack<T> raw[kEmbUnit], dst[kEmbUnit];
#pragma unroll
    for (int k = 0; k < kEmbUnit; ++k) {
        if (live[k]) raw[k] = io.template ahead<false>(dy, tok[k], cp);
        else raw[k] = zero_raw<T>();
    }
#pragma unroll
    for (int k = 0; k < kEmbUnit; ++k) {
        if (ends[k] && !(PARTS && (key[k] == before || key[k] == after))) dst[k] = io.template ahead<false>(demb, key[k], cp);
        else dst[k] = zero_raw<T>();
    }
    auto add_to = [&](int row, const RawPack<T>& to, const float (&a)[8]) {
        if (PARTS && (row == before || row == after)) {
            float* q = part + (2 * range + (row == before ? 0 : 1)) * (static_cast<int64_t>(io.ppr) * kPack) + cp * kPack;
            if (mine) {
                st_f4<false>(q, fvec4{a[0], a[1], a[2], a[3]});
                st_f4<false>(q + 4, fvec4{a[4], a[5], a[6], a[7]});
            }
            return;
        }
        float o[8];
        unpack<T>(io.settle(to, cp), o);
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = fmaf(scale, a[j], o[j]);
        if (mine) io.template store<false>(demb, row, cp, o);
    };
    bool open = !first_unit && live[0] && key[0] == prev;          // the run at hand came from the unit before
    const bool came = open;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, head[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    RawPack<T> head_dst = zero_raw<T>();
    bool head_ends = false;
#pragma unroll
    for (int k = 0; k < kEmbUnit; ++k) {
        if (live[k]) {
            float g[8];
            unpack<T>(io.settle(raw[k], cp), g);
            if constexpr (DROP) {
                float kf[8];
                io.factors(d, tok[k], cp, kf);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaf(g[j], kf[j], acc[j]);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += g[j];
            }
        }
        if (ends[k]) {
            if (open) {
#pragma unroll
                for (int j = 0; j < 8; ++j) head[j] = acc[j];
                head_dst = dst[k];
                head_ends = true;
            } else {
                add_to(key[k], dst[k], acc);
            }
            open = false;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
        }
    }
    // acc: what goes on into the next unit (0 if nothing does); `open` still: the whole unit is the middle of one run
    const bool middle = open;
    const uint64_t middles = __ballot(middle);
    if (middles != 0) {                                            // uniform; group after group
#pragma unroll
        for (int s = 1; s < 4; ++s)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float t = __shfl_up(acc[j], 16);
                if (middle && grp == s) acc[j] += t;
            }
    }
    float* vals = lds;                                             // [4][8][16]
    int* through = reinterpret_cast<int*>(lds + 4 * 128);          // [4]: the whole wave is the middle of one run
    if (grp == 3) {
#pragma unroll
        for (int j = 0; j < 8; ++j) vals[wave * 128 + j * 16 + (lane & 15)] = acc[j];
        if (lane == 63) through[wave] = middles == ~0ull;
    }
    __syncthreads();
    if (__ballot(came && head_ends) == 0) return;
    float in[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) in[j] = __shfl_up(acc[j], 16);
    // the units before this one in the wave are all middles: the sum of the waves before comes on top
    const bool reach = (middles & ((1ull << (16 * grp)) - 1ull)) == (1ull << (16 * grp)) - 1ull;
    if (grp == 0)
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] = 0.0f;
    if (reach) {
        float sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int v = 0; v < wave; ++v) {
            const bool t = through[v] != 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) sum[j] = vals[v * 128 + j * 16 + (lane & 15)] + (t ? sum[j] : 0.0f);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] += sum[j];
    }
    if (came && head_ends) {
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] += head[j];
        add_to(key[0], head_dst, in);
    }
}

// A run that crosses borders of ranges.  Every border that it crosses has a workgroup per column block for it, and these share its
// COLUMNS: each takes a slice of the 16 packs, a power of two, and holds 256 / slice rows of the run at once, so it has as many loads as a range's
// workgroup, whatever the run's length (down to slices of one pack), and no sum has to meet another workgroup's.  The lane groups add their rows in
// ascending position and meet in a butterfly, the waves in LDS: a fixed order.
// (8 in flight: two waves per SIMD fewer, 16384 x 2048 f32 with dropout 87 us, 80 with 4)
constexpr int kEmbBorderRows = 4;                                  // loads in flight per lane
template <typename T, bool DROP, bool RAG>
__device__ __forceinline__ void emb_border_run(float* lds, T* __restrict__ demb, const T* __restrict__ dy, const int2* __restrict__ order,
                                               int64_t border, int64_t rows, int cb, const RowPackIO<T, RAG>& io, float scale,
                                               const DropoutParams& d)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = border * kEmbRange - 32;                  // a view of 64 entries about the border: most runs begin and end in it
    int2 e = make_int2(0, static_cast<int>(kNoKey));
    if (base + lane < rows) e = order[base + lane];
    // every wave reads the same entries and takes the same decisions: the exits are workgroup-uniform
    const int key = __builtin_amdgcn_readlane(e.y, 32);
    if (!emb_live_key(key) || __builtin_amdgcn_readlane(e.y, 31) != key) return;
    const uint64_t run = __ballot(e.y == key);                     // entries of one id stand together
    const int lo = __builtin_ctzll(run), hi = 63 - __builtin_clzll(run);
    // [from, to): the run, or where it leaves the view the ranges that it touches (entries of others are told by their key)
    int64_t from = base + lo, to = base + hi + 1;
    bool seen = true;
    const int here = min(16, io.ppr - cb * 16);                    // packs of the column block
    if (lo == 0) {                                                 // v is the run's first range if the entry before it has another key
        seen = false;
        const int64_t v = border - 1 - lane;
        const uint64_t m = __ballot(v == 0 || (v > 0 && order[v * kEmbRange - 1].y != key));
        const int before = m != 0 ? __builtin_ctzll(m) : 64;       // of the run's borders, this one's index
        // only the first borders have a slice: the others leave here, one look from the start (each of a run's borders looking for its two ends is
        // quadratic in the run: one id in 16384 tokens of 1280 columns bf16 68.3 us, 66.5 like this)
        if (before >= here) return;
        from = (border - 1 - before) * kEmbRange;
    }
    if (hi == 63) {
        seen = false;
        const int64_t end = (rows + kEmbRange - 1) / kEmbRange - 1;     // the last range
        for (int64_t b = border;; b += 64) {
            const int64_t v = b + lane;
            const bool stop = v == end || (v < end && order[(v + 1) * kEmbRange].y != key);
            const uint64_t m = __ballot(stop);
            if (m != 0) { to = min(rows, (b + __builtin_ctzll(m) + 1) * kEmbRange); break; }
        }
    }
    const int64_t first = from / kEmbRange + 1, crossed = (to - 1) / kEmbRange + 1 - first;      // borders
    int width = 16;                                                // of a slice
    while (width >= 2 * here) width >>= 1;
    for (int64_t n = crossed; n >= 2 && width > 1; n >>= 1) width >>= 1;
    if ((border - first) * width >= here) return;                  // fewer slices than borders
    const int groups = 64 / width, grp = lane / width, c = static_cast<int>(border - first) * width + lane % width;
    const bool mine = c < here;
    const int cp = cb * 16 + min(c, here - 1);
    RawPack<T> dst = zero_raw<T>();
    const bool writes = wave == 0 && grp == 0 && mine;
    if (writes) dst = io.template ahead<false>(demb, key, cp);
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    constexpr int U = kEmbBorderRows;
    const int step = 4 * groups, at = wave * groups + grp;
    for (int64_t r0 = from; r0 < to; r0 += U * step) {
        int tok[U];
        bool ok[U];
        RawPack<T> raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = r0 + u * step + at;
            ok[u] = r < to;
            if (seen) {
                tok[u] = __shfl(e.x, static_cast<int>(r - base) & 63);
            } else {
                const int2 x = order[min(r, to - 1)];
                ok[u] = ok[u] && x.y == key;
                tok[u] = x.x;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (ok[u]) raw[u] = io.template ahead<false>(dy, tok[u], cp);
            else raw[u] = zero_raw<T>();
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u * step >= to) break;                        // uniform
            float g[8];
            unpack<T>(io.settle(raw[u], cp), g);
            if constexpr (DROP) {
                float kf[8];
                io.factors(d, tok[u], cp, kf);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaf(g[j], kf[j], acc[j]);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += g[j];
            }
        }
    }
    for (int w = width; w < 64; w <<= 1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += __shfl_xor(acc[j], w);
    }
    if (wave > 0 && grp == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) lds[((wave - 1) * 8 + j) * 16 + lane] = acc[j];
    }
    __syncthreads();
    if (writes) {
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += lds[(w * 8 + j) * 16 + lane];
        float o[8];
        unpack<T>(io.settle(dst, cp), o);
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = fmaf(scale, acc[j], o[j]);
        io.template store<false>(demb, key, cp, o);
    }
}

template <typename T, bool DROP, bool RAG, bool PARTS>
__global__ __launch_bounds__(256) void emb_accumulate(T* __restrict__ demb, const T* __restrict__ dy, const int2* __restrict__ order,
                                                      float* __restrict__ part, int64_t rows, int borders, int ncb, RowPackIO<T, RAG> io,
                                                      float scale, DropoutParams d)
{
    __shared__ float lds[4 * 128 + 4];
    const int unit = static_cast<int>(blockIdx.x) / ncb, cb = static_cast<int>(blockIdx.x) % ncb;
    if (!PARTS && unit < borders) emb_border_run<T, DROP, RAG>(lds, demb, dy, order, unit + 1, rows, cb, io, scale, d);
    else emb_range_runs<T, DROP, RAG, PARTS>(lds, demb, dy, order, part, PARTS ? unit : unit - borders, rows, cb, io, scale, d);
}

// PARTS: the shares of a run that crosses borders of ranges, added in ascending order of the ranges by the workgroup of its first border (the others
// leave), 16 lanes per row, 16 rows at once.  One partial row per 64 entries: the bytes are nothing beside those of dy.
template <typename T, bool RAG>
__global__ __launch_bounds__(256) void emb_join(T* __restrict__ demb, const float* __restrict__ part, const int2* __restrict__ order, int64_t rows,
                                                int ncb, RowPackIO<T, RAG> io, float scale)
{
    __shared__ float lds[3 * 128];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t border = static_cast<int>(blockIdx.x) / ncb + 1, end = (rows + kEmbRange - 1) / kEmbRange - 1;     // the last range
    // the border's two entries and the one before the range in front of it: the same for all threads, so the exits are workgroup-uniform
    const int key = emb_key_at(order, border * kEmbRange, rows);
    if (!emb_live_key(key) || emb_key_at(order, border * kEmbRange - 1, rows) != key) return;
    if (emb_key_at(order, (border - 1) * kEmbRange - 1, rows) == key) return;
    int64_t last = border;                                         // the last range that the run touches
    for (int64_t b = border;; b += 64) {                           // 64 ranges per trip
        const int64_t v = b + lane;
        const uint64_t m = __ballot(v == end || (v < end && order[(v + 1) * kEmbRange].y != key));
        if (m != 0) { last = b + __builtin_ctzll(m); break; }      // `end` stops
    }
    const int c = (static_cast<int>(blockIdx.x) % ncb) * 16 + (lane & 15), cp = min(c, io.ppr - 1);
    const bool writes = threadIdx.x < 16 && c < io.ppr;
    RawPack<T> dst = zero_raw<T>();
    if (writes) dst = io.template ahead<false>(demb, key, cp);
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    constexpr int U = 4;
    const int64_t colsp = static_cast<int64_t>(io.ppr) * kPack;
    for (int64_t v0 = border - 1 + (threadIdx.x >> 4); v0 <= last; v0 += 16 * U) {
        fvec4 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t v = v0 + 16 * u;
            a[u] = fvec4{0, 0, 0, 0};
            b[u] = fvec4{0, 0, 0, 0};
            if (v <= last) {
                const float* q = part + (2 * v + (v < border ? 1 : 0)) * colsp + cp * kPack;
                a[u] = ld_f4<false>(q);
                b[u] = ld_f4<false>(q + 4);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc[0] += a[u].x; acc[1] += a[u].y; acc[2] += a[u].z; acc[3] += a[u].w;
            acc[4] += b[u].x; acc[5] += b[u].y; acc[6] += b[u].z; acc[7] += b[u].w;
        }
    }
#pragma unroll
    for (int w = 16; w < 64; w <<= 1)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += __shfl_xor(acc[j], w);
    if (wave > 0 && lane < 16) {
#pragma unroll
        for (int j = 0; j < 8; ++j) lds[((wave - 1) * 8 + j) * 16 + lane] = acc[j];
    }
    __syncthreads();
    if (writes) {
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += lds[(w * 8 + j) * 16 + lane];
        float o[8];
        unpack<T>(io.settle(dst, cp), o);
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = fmaf(scale, acc[j], o[j]);
        io.template store<false>(demb, key, cp, o);
    }
}

// dP[l,:] += sum over the batch.  256 threads own W packs of one position; 256 / W groups of W lanes take every
// (256 / W)-th sentence each (four or eight loads in flight per lane) and their partial sums are added in group order, so the
// result does not depend on timing.  W = 64 up to 16 sentences (one trip of 4 x 4 loads), and where there are many positions
// to stream (fp32, 20 x 900, hidden 1600: 33 us, 59 as W = 16).  Otherwise 16 lanes per group, four times the sentences in
// flight and four times the workgroups: with few positions and long batches the serial trips were the whole time.  Whole
// backward in us with a token's look before its row's load, and now: 600 sentences of 17, hidden 512 41.6 / 24.8; 333 of 29, 1960 41.0 / 32.8;
// 300 of 50, 640 39.5 / 35.3.
constexpr int kDposWideBatch = 16, kDposManyUnits = 1024;
template <int W> constexpr int dpos_lds_floats() { return (256 / W - 1) * 8 * W; }
constexpr int kEmbLds = dpos_lds_floats<16>() * 4 > kSortLdsBytes ? dpos_lds_floats<16>() * 4 : kSortLdsBytes;

template <typename T, bool DROP, int W, bool RAG>
__device__ __forceinline__ void emb_dpos_body(float* sm, int cb, int l, T* __restrict__ dpos, const T* __restrict__ dy,
                                              const int32_t* __restrict__ tokens, int batch, int len,
                                              const RowPackIO<T, RAG>& io, int vocab, int pad_idx, const DropoutParams& d)
{
    // sentences per lane and trip as W = 16: eight in whole packs (600 sentences of 17, hidden 512: 24.8 us, 26.6 with four), four at any
    // alignment, where eight take 212-256 registers, for the sort too (eight / four: 40 x 200 x 777 f32 with dropout 51.6 / 37.6, bf16 38.8 /
    // 34.3, 333 x 29 x 1961 f32 90.4 / 73.4; the longest batches lose, 1000 x 16 x 301 bf16 41.6 / 44.8, 59 before the tokens were loaded ahead)
    constexpr int U = W == 16 && !RAG ? 8 : 4, G = 256 / W;
    const int lane = threadIdx.x % W, grp = threadIdx.x / W;
    const int cp = cb * W + lane;
    const bool active = cp < io.ppr;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (active) {
        // the next trip's tokens are loaded ahead, without conditions: a load behind a look at its token, one sentence after the
        // other, paid a token's latency each
        int next[U];
        auto fetch = [&](int b0) {
#pragma unroll
            for (int u = 0; u < U; ++u) next[u] = tokens[static_cast<int64_t>(min(b0 + u * G, batch - 1)) * len + l];
        };
        fetch(grp);
        for (int b0 = grp; b0 < batch; b0 += G * U) {
            RawPack<T> raw[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ok[u] = (b0 + u * G < batch) & !emb_is_pad(next[u], vocab, pad_idx);
                if (ok[u]) raw[u] = io.template ahead<false>(dy, static_cast<int64_t>(b0 + u * G) * len + l, cp);
                else raw[u] = zero_raw<T>();
            }
            if (b0 + G * U < batch) fetch(b0 + G * U);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!ok[u]) continue;
                const int64_t t = static_cast<int64_t>(b0 + u * G) * len + l;
                float g[8];
                unpack<T>(io.settle(raw[u], cp), g);
                if constexpr (DROP) {
                    float kf[8];
                    io.factors(d, t, cp, kf);
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[j] = fmaf(g[j], kf[j], acc[j]);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[j] += g[j];
                }
            }
        }
    }
    if (grp > 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) sm[((grp - 1) * 8 + j) * W + lane] = acc[j];
    }
    __syncthreads();
    if (grp == 0 && active) {
#pragma unroll
        for (int w = 0; w < G - 1; ++w)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += sm[(w * 8 + j) * W + lane];
        float o[8];
        unpack<T>(io.template load<false>(dpos, l, cp), o);
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] += acc[j];
        io.template store<false>(dpos, l, cp, o);
    }
}

// The sort is a few workgroups' work, the position gradient a stream over dy; neither needs the other.  One launch holds
// both, the sort first (workgroups 0 .. sorts - 1), so that they overlap instead of running back to back.  Without dP (units = 0) only
// the sort runs, without the sort (many tokens) only dP.
// The sort's registers are the stream's too: with 108 of them (four waves per SIMD, not six) 8192 x 1280 took 1.2 us longer.
template <typename T, bool DROP, int W, bool RAG>
__global__ __launch_bounds__(256) void emb_sort_dpos(int2* __restrict__ order, uint32_t* __restrict__ spill,
                                                     const int32_t* __restrict__ tokens, int64_t rows, int sorts, EmbSortPlan pl,
                                                     T* __restrict__ dpos, const T* __restrict__ dy, int batch, int len,
                                                     RowPackIO<T, RAG> io, int ncb, int vocab, int pad_idx, DropoutParams d)
{
    __shared__ __align__(16) char lds[kEmbLds];
    const int b = static_cast<int>(blockIdx.x) - sorts;
    if (b < 0) emb_sort_body(lds, blockIdx.x, order, spill, tokens, static_cast<int>(rows), pl, vocab, pad_idx);
    else emb_dpos_body<T, DROP, W, RAG>(reinterpret_cast<float*>(lds), b % ncb, b / ncb, dpos, dy, tokens, batch, len, io, vocab, pad_idx, d);
}

template <typename T, bool RAG>
inline void launch_sort_dpos(int2* order, uint32_t* spill, const int32_t* tokens, int64_t rows, bool sort, const EmbSortPlan& pl, T* dpos, const T* dy,
                             int batch, int len, const RowPackIO<T, RAG>& io, int vocab, int pad_idx, const DropoutParams& d, hipStream_t s)
{
    const int ppr = io.ppr;
    const int w = batch <= kDposWideBatch || ceil_div(ppr, 64) * len >= kDposManyUnits ? 64 : 16;
    const int ncb = static_cast<int>(ceil_div(ppr, w));
    const int64_t units = dpos ? static_cast<int64_t>(ncb) * len : 0;
    const int sorts = sort ? 1 << pl.part_bits : 0;
    const dim3 grid(static_cast<unsigned>(sorts + units)), block(256);
    if (grid.x == 0) return;
#define D(DROP, W) hipLaunchKernelGGL((emb_sort_dpos<T, DROP, W, RAG>), grid, block, 0, s, order, spill, tokens, rows, sorts, pl, dpos, dy, batch, len, io, ncb, vocab, pad_idx, d)
    if (d.on) { if (w == 64) D(true, 64); else D(true, 16); }
    else { if (w == 64) D(false, 64); else D(false, 16); }
#undef D
}

template <typename T, bool RAG>
static lsq_status emb_fwd_dispatch(void* out, const int32_t* tokens, const void* emb, const void* pos, int64_t rows,
                                   int len, int hidden, int vocab, int pad_idx, float scale, const DropoutParams& d,
                                   hipStream_t s)
{
    T* o = static_cast<T*>(out);
    const T* e = static_cast<const T*>(emb);
    const T* p = static_cast<const T*>(pos);
    if constexpr (RAG) {
        if (hidden < kEmbFlatColumns || rows * hidden < kEmbFlatElements) {
            hipLaunchKernelGGL((emb_fwd_flat<T>), dim3(static_cast<unsigned>(ceil_div(rows * hidden, 256))), dim3(256), 0, s,
                               o, tokens, e, p, rows, len, hidden, vocab, pad_idx, scale, d);
            return launch_status();
        }
    }
    const RowPackIO<T, RAG> io(hidden);
    // one row per wave up to 65536 rows: 5.9 / 8.0 us at 4096 x 1024 / 8192 x 1280 against 6.6 / 8.15 with four
    int64_t rb = ceil_div(rows, kEmbWaves);
    if (rb > 16384) rb = 16384;
    const dim3 grid(static_cast<unsigned>(ceil_div(io.ppr, 64)), static_cast<unsigned>(rb)), block(256);
    const FastDiv by_len = make_fastdiv(static_cast<uint32_t>(len));
    if (d.on) hipLaunchKernelGGL((emb_fwd_cols<T, true, RAG>), grid, block, 0, s, o, tokens, e, p, rows, len, io, vocab, pad_idx, scale, d, by_len);
    else hipLaunchKernelGGL((emb_fwd_cols<T, false, RAG>), grid, block, 0, s, o, tokens, e, p, rows, len, io, vocab, pad_idx, scale, d, by_len);
    return launch_status();
}

// A launch of 2^32 threads and more is refused, and by then the launches before it have changed dP: no call whose accumulation or position gradient (the
// wide form; the other has fewer than 4096 workgroups) is that large.  All others are smaller.
inline bool emb_bwd_launches(int64_t rows, int len, int hidden, bool dpos)
{
    constexpr int64_t kMost = 0xFFFFFFFFll / 256;                  // workgroups of 256 threads
    const int64_t ranges = ceil_div(rows, kEmbRange), units = rows > kEmbSortMax ? ranges : 2 * ranges - 1;
    return units * ceil_div(hidden, 16 * kPack) <= kMost && (!dpos || ceil_div(hidden, 64 * kPack) * len + 128 <= kMost);       // (128: the sort's)
}

template <typename T, bool RAG>
static lsq_status emb_bwd_dispatch(void* demb, void* dpos, const void* dy, const int32_t* tokens, void* ws,
                                   int batch, int len, int hidden, int vocab, int pad_idx, float scale,
                                   const DropoutParams& d, hipStream_t s)
{
    const int64_t rows = static_cast<int64_t>(batch) * len;
    const EmbBwdPlan plan = emb_bwd_plan(rows, hidden);
    int2* order = reinterpret_cast<int2*>(ws);
    T* de = static_cast<T*>(demb);
    T* dp = static_cast<T*>(dpos);
    const T* g = static_cast<const T*>(dy);
    // the dropout scale 1/(1-p) is carried by the per-element factors; `scale` is the embedding scale
    const RowPackIO<T, RAG> io(hidden);
    int bits = 1;
    while ((static_cast<int64_t>(1) << bits) <= vocab) ++bits;                 // 2^bits > vocab: padding (all ones) comes last
    const int passes = (bits + 7) / 8;
    const EmbSortPlan pl = emb_sort_plan(rows, bits);
    const bool few = pl.fits;
    // the radix sort's second buffer; the in-LDS sort's two words per token for parts that LDS does not hold
    int2* tmp = reinterpret_cast<int2*>(static_cast<char*>(ws) + plan.pair_bytes);
    uint32_t* spill = reinterpret_cast<uint32_t*>(tmp);
    int32_t* hist = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + 2 * plan.pair_bytes);    // [256][radix blocks]
    // the position gradient rides along with the in-LDS sort
    launch_sort_dpos<T, RAG>(order, spill, tokens, rows, few, pl, dp, g, batch, len, io, vocab, pad_idx, d, s);
    if (!few) {
        const int nblocks = plan.radix_blocks;
        const int2* src = nullptr;
        for (int pass = 0; pass < passes; ++pass) {
            int2* dst = (passes - pass) % 2 == 1 ? order : tmp;                      // the last pass lands in `order`
            hipLaunchKernelGGL(emb_radix_hist, dim3(nblocks), dim3(256), 0, s, hist, src, tokens, rows, nblocks, 8 * pass, vocab, pad_idx);
            if (nblocks <= kRadixFuseScan) {
                hipLaunchKernelGGL((emb_radix_scatter<false>), dim3(nblocks), dim3(256), 0, s, dst, hist, src, tokens, rows, nblocks, 8 * pass, vocab, pad_idx);
            } else {
                hipLaunchKernelGGL(emb_radix_scan, dim3(1), dim3(1024), 0, s, hist, static_cast<int64_t>(256) * nblocks);
                hipLaunchKernelGGL((emb_radix_scatter<true>), dim3(nblocks), dim3(256), 0, s, dst, hist, src, tokens, rows, nblocks, 8 * pass, vocab, pad_idx);
            }
            src = dst;
        }
    }
    const int ranges = static_cast<int>(ceil_div(rows, kEmbRange)), ncb = static_cast<int>(ceil_div(io.ppr, 16));
    float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + 2 * plan.pair_bytes + plan.hist_bytes);
    const bool parts = plan.part_bytes != 0;
    const int borders = parts ? 0 : ranges - 1;
    const dim3 grid(static_cast<unsigned>(borders + ranges) * static_cast<unsigned>(ncb)), block(256);
#define A(DROP, PARTS) hipLaunchKernelGGL((emb_accumulate<T, DROP, RAG, PARTS>), grid, block, 0, s, de, g, order, part, rows, borders, ncb, io, scale, d)
    if (parts) { if (d.on) A(true, true); else A(false, true); }
    else { if (d.on) A(true, false); else A(false, false); }
#undef A
    if (parts)
        hipLaunchKernelGGL((emb_join<T, RAG>), dim3(static_cast<unsigned>(ranges - 1) * static_cast<unsigned>(ncb)), block, 0, s, de, part, order, rows, ncb, io, scale);
    return launch_status();
}

}  // namespace lsq

extern "C" lsq_status lsq_embedding_fwd(void* out, const int32_t* tokens, const void* emb, const void* pos,
                                        int32_t batch, int32_t len, int32_t hidden, int32_t vocab, int32_t pad_idx,
                                        float scale, float p, uint64_t seed, uint64_t offset, lsq_dtype dt, void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(batch >= 0 && len >= 0 && hidden > 0 && vocab > 0);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p, seed, offset, &d));
    const int64_t rows = static_cast<int64_t>(batch) * len;
    if (rows == 0) return LSQ_OK;
    LSQ_REQUIRE(out && tokens && emb && pos);
    LSQ_ALIGNED(out); LSQ_ALIGNED(emb); LSQ_ALIGNED(pos);
    LSQ_REQUIRE(rows <= 0x7FFFFFFF);
    LSQ_REQUIRE(ceil_div(rows * hidden, 256) <= 0x7FFFFFFF);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool rag = hidden % kPack != 0;
    switch (dt) {
        case LSQ_F16: return rag ? emb_fwd_dispatch<f16, true>(out, tokens, emb, pos, rows, len, hidden, vocab, pad_idx, scale, d, s) : emb_fwd_dispatch<f16, false>(out, tokens, emb, pos, rows, len, hidden, vocab, pad_idx, scale, d, s);
        case LSQ_BF16: return rag ? emb_fwd_dispatch<bf16, true>(out, tokens, emb, pos, rows, len, hidden, vocab, pad_idx, scale, d, s) : emb_fwd_dispatch<bf16, false>(out, tokens, emb, pos, rows, len, hidden, vocab, pad_idx, scale, d, s);
        default: return rag ? emb_fwd_dispatch<float, true>(out, tokens, emb, pos, rows, len, hidden, vocab, pad_idx, scale, d, s) : emb_fwd_dispatch<float, false>(out, tokens, emb, pos, rows, len, hidden, vocab, pad_idx, scale, d, s);
    }
}

extern "C" lsq_status lsq_embedding_bwd(void* demb, void* dpos, const void* dy, const int32_t* tokens, int32_t batch,
                                        int32_t len, int32_t hidden, int32_t vocab, int32_t pad_idx, float scale,
                                        float p, uint64_t seed, uint64_t offset, void* workspace, size_t workspace_bytes,
                                        lsq_dtype dt, void* stream)
{
    using namespace lsq;
    LSQ_REQUIRE(batch >= 0 && len >= 0 && hidden > 0 && vocab > 0);
    if (!valid_dtype(dt)) return LSQ_UNSUPPORTED_DTYPE;
    DropoutParams d;
    LSQ_REQUIRE(make_dropout(p, seed, offset, &d));
    const int64_t rows = static_cast<int64_t>(batch) * len;
    if (rows == 0) return LSQ_OK;
    LSQ_REQUIRE(rows <= 0x7FFFFFFF / 2);
    LSQ_REQUIRE(emb_bwd_launches(rows, len, hidden, dpos != nullptr));
    LSQ_REQUIRE(demb && dy && tokens);
    LSQ_ALIGNED(demb); LSQ_ALIGNED(dpos); LSQ_ALIGNED(dy); LSQ_ALIGNED(workspace);
    const size_t need = emb_bwd_plan(rows, hidden).total();
    if (!workspace || workspace_bytes < need) return LSQ_WORKSPACE_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    void* ws = workspace;
    const bool rag = hidden % kPack != 0;
    switch (dt) {
        case LSQ_F16: return rag ? emb_bwd_dispatch<f16, true>(demb, dpos, dy, tokens, ws, batch, len, hidden, vocab, pad_idx, scale, d, s) : emb_bwd_dispatch<f16, false>(demb, dpos, dy, tokens, ws, batch, len, hidden, vocab, pad_idx, scale, d, s);
        case LSQ_BF16: return rag ? emb_bwd_dispatch<bf16, true>(demb, dpos, dy, tokens, ws, batch, len, hidden, vocab, pad_idx, scale, d, s) : emb_bwd_dispatch<bf16, false>(demb, dpos, dy, tokens, ws, batch, len, hidden, vocab, pad_idx, scale, d, s);
        default: return rag ? emb_bwd_dispatch<float, true>(demb, dpos, dy, tokens, ws, batch, len, hidden, vocab, pad_idx, scale, d, s) : emb_bwd_dispatch<float, false>(demb, dpos, dy, tokens, ws, batch, len, hidden, vocab, pad_idx, scale, d, s);
    }
}
