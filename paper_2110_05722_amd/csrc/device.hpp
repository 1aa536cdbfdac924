// Device-side building blocks for the gfx950 kernels: storage types, 8-element
// packs (one 128-bit access for fp16/bf16), wave64 reductions on DPP, and the
// Philox4x32-10 dropout stream.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lsq {

using f16 = _Float16;
using bf16 = __bf16;

constexpr int kWave = 64;
constexpr int kPack = 8;   // elements per pack == elements per Philox call

template <typename T> struct alignas(sizeof(T) * 8 > 16 ? 16 : sizeof(T) * 8) Raw8 { T v[8]; };

template <typename T> __device__ __forceinline__ float to_f32(T v) { return static_cast<float>(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v) { return static_cast<T>(v); }

// 128-bit vector types the nontemporal builtins accept.
typedef float fvec4 __attribute__((ext_vector_type(4)));
typedef uint32_t uvec4 __attribute__((ext_vector_type(4)));
typedef uint32_t uvec2 __attribute__((ext_vector_type(2)));

// Streaming accesses carry the nontemporal hint: the tensors on this path are far
// larger than L2 and are touched once per kernel, so keeping their lines only
// evicts data someone else could reuse.  Measured on MI355X it is worth 7 % on a
// plain copy and 10 % on the Adam kernel.
template <bool NT> __device__ __forceinline__ fvec4 ld_f4(const float* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const fvec4*>(p));
    else return *reinterpret_cast<const fvec4*>(p);
}
template <bool NT> __device__ __forceinline__ void st_f4(float* p, fvec4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<fvec4*>(p));
    else *reinterpret_cast<fvec4*>(p) = v;
}
template <bool NT> __device__ __forceinline__ uvec4 ld_u4(const void* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const uvec4*>(p));
    else return *reinterpret_cast<const uvec4*>(p);
}
template <bool NT> __device__ __forceinline__ void st_u4(void* p, uvec4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<uvec4*>(p));
    else *reinterpret_cast<uvec4*>(p) = v;
}
template <bool NT> __device__ __forceinline__ uvec2 ld_u2(const void* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const uvec2*>(p));
    else return *reinterpret_cast<const uvec2*>(p);
}
template <bool NT> __device__ __forceinline__ void st_u2(void* p, uvec2 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<uvec2*>(p));
    else *reinterpret_cast<uvec2*>(p) = v;
}

// 8 consecutive elements starting at a pack-aligned address, widened to fp32.
// fp16/bf16: one global_load_dwordx4; fp32: two.
template <typename T, bool NT = false>
__device__ __forceinline__ void load8(const T* __restrict__ p, float (&f)[8])
{
    if constexpr (sizeof(T) == 2) {
        const uvec4 u = ld_u4<NT>(p);
        const Raw8<T> r = __builtin_bit_cast(Raw8<T>, u);
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = to_f32<T>(r.v[j]);
    } else {
        const fvec4 a = ld_f4<NT>(reinterpret_cast<const float*>(p));
        const fvec4 b = ld_f4<NT>(reinterpret_cast<const float*>(p) + 4);
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
        f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
}

template <typename T, bool NT = false>
__device__ __forceinline__ void store8(T* __restrict__ p, const float (&f)[8])
{
    if constexpr (sizeof(T) == 2) {
        Raw8<T> r;
#pragma unroll
        for (int j = 0; j < 8; ++j) r.v[j] = from_f32<T>(f[j]);
        st_u4<NT>(p, __builtin_bit_cast(uvec4, r));
    } else {
        st_f4<NT>(reinterpret_cast<float*>(p), fvec4{f[0], f[1], f[2], f[3]});
        st_f4<NT>(reinterpret_cast<float*>(p) + 4, fvec4{f[4], f[5], f[6], f[7]});
    }
}

// A pack in its storage form (4 registers for fp16/bf16, 8 for fp32).  Kernels load the
// raw packs of a whole row first and widen them afterwards: all loads of the row are then
// in flight together, and a prefetched row costs half the registers of its fp32 form.
template <typename T, int = sizeof(T)> struct RawPack;
template <typename T> struct RawPack<T, 2> { uvec4 u; };
template <typename T> struct RawPack<T, 4> { fvec4 a, b; };

template <typename T, bool NT = false>
__device__ __forceinline__ RawPack<T> load_raw(const T* __restrict__ p)
{
    RawPack<T> r;
    if constexpr (sizeof(T) == 2) {
        r.u = ld_u4<NT>(p);
    } else {
        r.a = ld_f4<NT>(reinterpret_cast<const float*>(p));
        r.b = ld_f4<NT>(reinterpret_cast<const float*>(p) + 4);
    }
    return r;
}

template <typename T, bool NT = false>
__device__ __forceinline__ void store_raw(T* __restrict__ p, const RawPack<T>& r)
{
    if constexpr (sizeof(T) == 2) {
        st_u4<NT>(p, r.u);
    } else {
        st_f4<NT>(reinterpret_cast<float*>(p), r.a);
        st_f4<NT>(reinterpret_cast<float*>(p) + 4, r.b);
    }
}

template <typename T>
__device__ __forceinline__ RawPack<T> zero_raw()
{
    RawPack<T> r;
    if constexpr (sizeof(T) == 2) r.u = uvec4{0u, 0u, 0u, 0u};
    else { r.a = fvec4{0.f, 0.f, 0.f, 0.f}; r.b = r.a; }
    return r;
}

// Hide a packed row from the optimiser: a kernel that walks the same packs in several passes
// re-widens them in each pass instead of keeping 8 fp32 registers per pack alive in between.
template <typename T>
__device__ __forceinline__ void opaque(RawPack<T>& r)
{
    if constexpr (sizeof(T) == 2) asm volatile("" : "+v"(r.u));
    else asm volatile("" : "+v"(r.a), "+v"(r.b));
}

template <typename T>
__device__ __forceinline__ void unpack(const RawPack<T>& r, float (&f)[8])
{
    if constexpr (sizeof(T) == 2) {
        const Raw8<T> h = __builtin_bit_cast(Raw8<T>, r.u);
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = to_f32<T>(h.v[j]);
    } else {
        f[0] = r.a.x; f[1] = r.a.y; f[2] = r.a.z; f[3] = r.a.w;
        f[4] = r.b.x; f[5] = r.b.y; f[6] = r.b.z; f[7] = r.b.w;
    }
}

// fp32 -> storage form (one rounding per element), the inverse of unpack
template <typename T>
__device__ __forceinline__ RawPack<T> pack_raw(const float (&f)[8])
{
    RawPack<T> r;
    if constexpr (sizeof(T) == 2) {
        Raw8<T> h;
#pragma unroll
        for (int j = 0; j < 8; ++j) h.v[j] = from_f32<T>(f[j]);
        r.u = __builtin_bit_cast(uvec4, h);
    } else {
        r.a = fvec4{f[0], f[1], f[2], f[3]};
        r.b = fvec4{f[4], f[5], f[6], f[7]};
    }
    return r;
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// fp32 packs of a group of G lanes that hold G consecutive packs.  A pack is two 16-byte accesses, and with pack = lane each of them covers every
// second 16 bytes: half of each line, twice, which with nontemporal hints moves half lines to and from memory.  Here lane l holds pack
// (l / 2) + (l % 2) G / 2: its accesses are the 16-byte pieces l and G + l of the group, which cover it without gaps, and each pair of lanes exchanges one
// piece.  Both lanes of a pair have to be there; `ok` says whether the lane's own pack is (the packs that are there come first in the group).
// 16-bit packs are one access: pack = lane.  fp32, us with pack = lane and like this, inputs cold: bias+dropout+residual forward / backward 16384 x 1024
// 40.0 / 37.6 and 32.8 / 30.0 (the copy of the forward's bytes 32), 8192 x 1280 26.3 / 23.5 and 22.0 / 20.5, 2000 x 1024 7.2 / 8.4 and 6.5 / 7.9; GELU with dropout
// 16384 x 1024 29.4 / 43.8 and 25.0 / 38.5, 8192 x 1280 20.5 / 32.4 and 18.6 / 27.9.  Without the hints, pack = lane: 37.1 / 35.7 and 28.7 / 40.9.
template <typename T, int G>
struct LanePacks {
    static constexpr bool kPaired = sizeof(T) == 4 && G >= 8;      // (below, no line is covered either way)
    static __device__ __forceinline__ int pack(int l)
    {
        if constexpr (kPaired) return (l & ~(G - 1)) | ((l & (G - 1)) >> 1) | ((l & 1) * (G / 2));
        else return l;
    }
    static __device__ __forceinline__ fvec4 other(const fvec4& v)  // the other lane's of the pair: quad_perm [1,0,3,2]
    {
        return fvec4{dpp_mov<0xB1>(v.x), dpp_mov<0xB1>(v.y), dpp_mov<0xB1>(v.z), dpp_mov<0xB1>(v.w)};
    }
    static __device__ __forceinline__ bool other(bool ok) { return __builtin_amdgcn_update_dpp(0, ok ? 1 : 0, 0xB1, 0xF, 0xF, false) != 0; }
    template <bool NT>
    static __device__ __forceinline__ void load_into(RawPack<T>& r, const T* p, bool ok)      // p: the lane's own pack; r stays where it is not there
    {
        if constexpr (kPaired) {
            const bool odd = threadIdx.x & 1, ok2 = other(ok);
            const float* a = reinterpret_cast<const float*>(p) + (odd ? 4 - 4 * G : 0);
            if (odd ? ok2 : ok) r.a = ld_f4<NT>(a);
            if (odd ? ok : ok2) r.b = ld_f4<NT>(a + 4 * G);        // settled where it is used: the exchange would wait for it
        } else {
            if (ok) r = load_raw<T, NT>(p);
        }
    }
    template <bool NT>
    static __device__ __forceinline__ RawPack<T> load(const T* p, bool ok)
    {
        RawPack<T> r = zero_raw<T>();
        load_into<NT>(r, p, ok);
        return r;
    }
    static __device__ __forceinline__ RawPack<T> settle(const RawPack<T>& r)
    {
        if constexpr (kPaired) {
            const bool odd = threadIdx.x & 1;
            const fvec4 t = other(odd ? r.a : r.b);
            RawPack<T> o;
            o.a = odd ? t : r.a;
            o.b = odd ? r.b : t;
            return o;
        } else {
            return r;
        }
    }
    template <bool NT>
    static __device__ __forceinline__ void store(T* p, const RawPack<T>& r, bool ok)
    {
        if constexpr (kPaired) {
            const float f[8] = {r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w};
            store<NT>(p, f, ok);
        } else {
            if (ok) store_raw<T, NT>(p, r);
        }
    }
    template <bool NT>
    static __device__ __forceinline__ void move(T* p, const RawPack<T>& r)        // what load() has read, whole groups, to where the lane's pack goes
    {
        if constexpr (kPaired) {
            float* a = reinterpret_cast<float*>(p) + (threadIdx.x & 1 ? 4 - 4 * G : 0);
            st_f4<NT>(a, r.a);
            st_f4<NT>(a + 4 * G, r.b);
        } else {
            store_raw<T, NT>(p, r);
        }
    }
    template <bool NT>
    static __device__ __forceinline__ void store(T* p, const float (&f)[8], bool ok)
    {
        if constexpr (kPaired) {
            const bool odd = threadIdx.x & 1, ok2 = other(ok);
            const fvec4 q0 = {f[0], f[1], f[2], f[3]}, q1 = {f[4], f[5], f[6], f[7]};
            const fvec4 t = other(odd ? q0 : q1);
            float* a = reinterpret_cast<float*>(p) + (odd ? 4 - 4 * G : 0);
            if (odd ? ok2 : ok) st_f4<NT>(a, odd ? t : q0);
            if (odd ? ok : ok2) st_f4<NT>(a + 4 * G, odd ? q1 : t);
        } else {
            if (ok) store8<T, NT>(p, f);
        }
    }
};

// Make eight fp32 values exist as fp32 before they are narrowed: without it the compiler may fold
// a final fma into the conversion (v_fma_mixlo_f16: one rounding instead of two), and it takes
// that decision instantiation by instantiation, so two kernels that must agree bit for bit would not.
__device__ __forceinline__ void pin_f32(float (&f)[8])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(f[j]));
}

// 4 consecutive elements (one 128-bit access of fp32, one 64-bit access of fp16/bf16).
template <typename T> struct alignas(sizeof(T) * 4 > 16 ? 16 : sizeof(T) * 4) Raw4 { T v[4]; };

template <typename T, bool NT = false>
__device__ __forceinline__ void load4(const T* __restrict__ p, float (&f)[4])
{
    if constexpr (sizeof(T) == 2) {
        const uvec2 u = ld_u2<NT>(p);
        const Raw4<T> r = __builtin_bit_cast(Raw4<T>, u);
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = to_f32<T>(r.v[j]);
    } else {
        const fvec4 a = ld_f4<NT>(reinterpret_cast<const float*>(p));
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    }
}

template <typename T, bool NT = false>
__device__ __forceinline__ void store4(T* __restrict__ p, const float (&f)[4])
{
    if constexpr (sizeof(T) == 2) {
        Raw4<T> r;
#pragma unroll
        for (int j = 0; j < 4; ++j) r.v[j] = from_f32<T>(f[j]);
        st_u2<NT>(p, __builtin_bit_cast(uvec2, r));
    } else {
        st_f4<NT>(reinterpret_cast<float*>(p), fvec4{f[0], f[1], f[2], f[3]});
    }
}

// ---------------------------------------------------------------- reductions
// All-reduce over aligned groups of WIDTH lanes (a power of two <= 64) inside one
// wave64.  Lanes 1..15 apart are reached with DPP (quad permutes and row mirrors,
// no LDS traffic); 16 apart with a 32-lane swizzle; the last step of a full-wave
// reduction reads the four row results through scalar registers.
struct OpSum { static __device__ __forceinline__ float apply(float a, float b) { return a + b; } };
struct OpMax { static __device__ __forceinline__ float apply(float a, float b) { return fmaxf(a, b); } };

//
// PAIRED: the lanes hold packs as LanePacks of groups of 8 do, and the groups of 8 add in the order of the PACK's index (lane bits 1, 2, 0 are pack bits
// 0, 1, 2): the result is, bit for bit, that of the same packs with pack = lane, so the two forms may be chosen by what is faster.
template <int WIDTH, typename Op, bool PAIRED = false>
__device__ __forceinline__ float group_allreduce(float v)
{
    static_assert(WIDTH == 1 || WIDTH == 2 || WIDTH == 4 || WIDTH == 8 || WIDTH == 16 || WIDTH == 32 || WIDTH == 64, "");
    if constexpr (PAIRED) {
        static_assert(WIDTH >= 8, "");
        v = Op::apply(v, dpp_mov<0x4E>(v));                          // 2 apart
        v = Op::apply(v, dpp_mov<0x1B>(dpp_mov<0x141>(v)));          // 4 apart: quad_perm [3,2,1,0] of the half mirror
        v = Op::apply(v, dpp_mov<0xB1>(v));                          // 1 apart
    } else {
        if constexpr (WIDTH >= 2) v = Op::apply(v, dpp_mov<0xB1>(v));    // quad_perm [1,0,3,2]
        if constexpr (WIDTH >= 4) v = Op::apply(v, dpp_mov<0x4E>(v));    // quad_perm [2,3,0,1]
        if constexpr (WIDTH >= 8) v = Op::apply(v, dpp_mov<0x141>(v));   // row_half_mirror
    }
    if constexpr (WIDTH >= 16) v = Op::apply(v, dpp_mov<0x140>(v));  // row_mirror
    if constexpr (WIDTH == 32) {
        // swap with the lane 16 away inside each half-wave (bit-mask mode: and 0x1F, xor 0x10)
        float o = __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
        v = Op::apply(v, o);
    }
    if constexpr (WIDTH == 64) {
        const int iv = __builtin_bit_cast(int, v);
        float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 0));
        float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16));
        float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 32));
        float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 48));
        v = Op::apply(Op::apply(r0, r1), Op::apply(r2, r3));
    }
    return v;
}

// A half-wave's sum of packs in lane pairs of groups of 32: pack bits 0..3 are lane bits 1..4 and bit 4 is lane bit 0, so this adds over them in that order
// and is, bit for bit, group_sum<32> of the same packs with pack = lane.
__device__ __forceinline__ float paired_half_wave_sum(float v)
{
    v += dpp_mov<0x4E>(v);                                           // 2 apart
    v += dpp_mov<0x1B>(dpp_mov<0x141>(v));                           // 4 apart
    v += dpp_mov<0x128>(v);                                          // 8 apart: row_ror:8
    v += __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));      // 16 apart
    return v + dpp_mov<0xB1>(v);                                     // 1 apart
}

template <int WIDTH, bool PAIRED = false> __device__ __forceinline__ float group_sum(float v) { return group_allreduce<WIDTH, OpSum, PAIRED>(v); }
template <int WIDTH> __device__ __forceinline__ float group_max(float v) { return group_allreduce<WIDTH, OpMax>(v); }

// Block-wide all-reduce for NWAVES waves; `scratch` holds NWAVES floats of LDS.
// Every thread of the block must call it; it contains two barriers.
template <int NWAVES, typename Op, bool PAIRED = false>
__device__ __forceinline__ float block_allreduce(float v, float* scratch)
{
    v = group_allreduce<64, Op, PAIRED>(v);
    if constexpr (NWAVES == 1) return v;
    const int wave = threadIdx.x >> 6;
    __syncthreads();                    // scratch may still be read from a previous call
    if ((threadIdx.x & 63) == 0) scratch[wave] = v;
    __syncthreads();
    float r = scratch[0];
#pragma unroll
    for (int w = 1; w < NWAVES; ++w) r = Op::apply(r, scratch[w]);
    return r;
}

// -------------------------------------------------------------------- Philox
// Philox4x32-10 (Salmon et al., SC'11).  One call yields 128 bits = eight 16-bit
// dropout lanes, so a pack of 8 elements costs one call.
struct DropoutParams {
    uint32_t key0, key1;      // seed
    uint32_t ctr2, ctr3;      // offset
    uint32_t t16;             // keep iff r16 >= t16
    uint32_t on;              // p > 0: draw and scale (a p so small that t16 rounds to 0 keeps everything, still scaled)
    float scale;              // 1 / (1 - p)
};

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
    constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = static_cast<uint64_t>(M0) * c0;
        const uint64_t p1 = static_cast<uint64_t>(M1) * c2;
        // three-input xor in one VALU operation (truth table 0x96); the round keys stay scalar
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p1 >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p0 >> 32), c3, k1, 0x96);
        c1 = static_cast<uint32_t>(p1);
        c3 = static_cast<uint32_t>(p0);
        c0 = n0;
        c2 = n2;
        k0 += W0;
        k1 += W1;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Workgroup -> tile for kernels that stream large tensors one tile per workgroup.  Consecutive workgroups of a
// launch go to the eight XCDs in turn, each with its own L2 and address-translation cache; with tile = workgroup
// every XCD walks every small piece of every tensor.  Here an XCD takes a run of CHUNK consecutive tiles out of
// every eight runs, so that it streams about a megabyte of each tensor at a stretch.  The last, partial group of
// eight runs keeps its order; the map is a permutation of 0..nb-1.
template <int CHUNK>
__device__ __forceinline__ int64_t xcd_chunked(int64_t b, int64_t nb)
{
    if constexpr (CHUNK <= 1) return b;
    constexpr int64_t kGroup = 8 * static_cast<int64_t>(CHUNK);
    const int64_t first = b / kGroup * kGroup;
    if (first + kGroup > nb) return b;
    const int64_t r = b - first;
    return first + (r % 8) * CHUNK + r / 8;
}

// The same with the runs of a group handed to the XCDs in an order that rotates from group to group: XCDs receive
// their workgroups in strict rotation whatever their load, so when the cost of a tile depends on its position
// in a period that the group length divides (padded sentence tails in a criterion batch), fixed runs would give
// one XCD all the cheap tiles.
template <int CHUNK>
__device__ __forceinline__ int64_t xcd_chunked_rotating(int64_t b, int64_t nb)
{
    if constexpr (CHUNK <= 1) return b;
    constexpr int64_t kGroup = 8 * static_cast<int64_t>(CHUNK);
    const int64_t grp = b / kGroup, first = grp * kGroup;
    if (first + kGroup > nb) return b;
    const int64_t r = b - first;
    return first + ((r + grp) % 8) * CHUNK + r / 8;
}

// (column block, row block) of a workgroup of a [column blocks, row blocks] grid.
// ORDER 0: as launched (column blocks fastest); 1: row blocks fastest.
struct GridBlock { int col; int row; };
template <int ORDER>
__device__ __forceinline__ GridBlock grid_block()
{
    if constexpr (ORDER == 1) {
        const unsigned lin = blockIdx.x + gridDim.x * blockIdx.y;
        return {static_cast<int>(lin / gridDim.y), static_cast<int>(lin % gridDim.y)};
    } else {
        return {static_cast<int>(blockIdx.x), static_cast<int>(blockIdx.y)};
    }
}

// keep[j] (as 0.0f / scale) for the 8 elements of pack `g` (flat element index / 8).
__device__ __forceinline__ void dropout_factors8(const DropoutParams& d, uint64_t g, float (&k)[8])
{
    uint32_t w[4];
    philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), d.ctr2, d.ctr3, d.key0, d.key1, w);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        k[2 * j] = (w[j] & 0xFFFFu) >= d.t16 ? d.scale : 0.0f;
        k[2 * j + 1] = (w[j] >> 16) >= d.t16 ? d.scale : 0.0f;
    }
}

// v = keep ? v : 0 for the 8 elements of pack `g`: a dropped infinity or NaN becomes 0, which a factor of 0 would not make it.
__device__ __forceinline__ void dropout_keep8(const DropoutParams& d, uint64_t g, float (&v)[8])
{
    uint32_t w[4];
    philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), d.ctr2, d.ctr3, d.key0, d.key1, w);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[2 * j] = (w[j] & 0xFFFFu) >= d.t16 ? v[2 * j] : 0.0f;
        v[2 * j + 1] = (w[j] >> 16) >= d.t16 ? v[2 * j + 1] : 0.0f;
    }
}

// factors from the sixteen 16-bit lanes of two groups, from lane s (0..7) on.  The words are pinned as single registers: left as arrays,
// `by4 ? w[1] : w[0]` becomes an access by a selected address, which puts the array into LDS or scratch memory (feed-forward
// forward of 500 x 1027: 16.7 us).
__device__ __forceinline__ void dropout_lanes8(const DropoutParams& d, unsigned s, uint32_t (&lo)[4], uint32_t (&hi)[4], float (&k)[8])
{
    uint32_t l0 = lo[0], l1 = lo[1], l2 = lo[2], l3 = lo[3], h0 = hi[0], h1 = hi[1], h2 = hi[2], h3 = hi[3];
    asm volatile("" : "+v"(l0), "+v"(l1), "+v"(l2), "+v"(l3), "+v"(h0), "+v"(h1), "+v"(h2), "+v"(h3));
    const bool by4 = s & 4u, by2 = s & 2u, by1 = s & 1u;
    const uint32_t a0 = by4 ? l2 : l0, a1 = by4 ? l3 : l1, a2 = by4 ? h0 : l2, a3 = by4 ? h1 : l3;
    const uint32_t a4 = by4 ? h2 : h0, a5 = by4 ? h3 : h1;
    const uint32_t b0 = by2 ? a1 : a0, b1 = by2 ? a2 : a1, b2 = by2 ? a3 : a2, b3 = by2 ? a4 : a3, b4 = by2 ? a5 : a4;
    const uint32_t w[4] = {by1 ? (b0 >> 16) | (b1 << 16) : b0, by1 ? (b1 >> 16) | (b2 << 16) : b1,
                           by1 ? (b2 >> 16) | (b3 << 16) : b2, by1 ? (b3 >> 16) | (b4 << 16) : b3};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        k[2 * j] = (w[j] & 0xFFFFu) >= d.t16 ? d.scale : 0.0f;
        k[2 * j + 1] = (w[j] >> 16) >= d.t16 ? d.scale : 0.0f;
    }
}

// The factors of the 8 elements from flat element `e` on, at any alignment: the two groups that they touch are drawn and the
// sixteen 16-bit lanes shifted down by e % 8 (e is the same for all lanes of a row walk up to multiples of 8: the shifts'
// conditions are uniform).
__device__ __forceinline__ void dropout_factors8_any(const DropoutParams& d, uint64_t e, float (&k)[8])
{
    const uint64_t g = e >> 3;
    uint32_t lo[4], hi[4];
    philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), d.ctr2, d.ctr3, d.key0, d.key1, lo);
    philox4x32_10(static_cast<uint32_t>(g + 1), static_cast<uint32_t>((g + 1) >> 32), d.ctr2, d.ctr3, d.key0, d.key1, hi);
    dropout_lanes8(d, static_cast<unsigned>(e) & 7u, lo, hi, k);
}

// The same where lane i of the wave holds pack cp + i of one row: the second group is the next lane's first one, so a lane draws one
// group and takes the other's words from its neighbour.  All 64 lanes call it; lane 63 has no neighbour and holds no pack
// of its own (kRagLanes packs per wave).
constexpr int kRagLanes = 63;
__device__ __forceinline__ void dropout_factors8_row(const DropoutParams& d, uint64_t e, float (&k)[8])
{
    uint32_t lo[4], hi[4];
    const uint64_t g = e >> 3;
    philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), d.ctr2, d.ctr3, d.key0, d.key1, lo);
#pragma unroll
    for (int j = 0; j < 4; ++j)      // wave_shl 1
        hi[j] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo[j]), 0x130, 0xF, 0xF, false));
    dropout_lanes8(d, static_cast<unsigned>(e) & 7u, lo, hi, k);
}

// a pack moved down by s elements (0..7), zeros from above
__device__ __forceinline__ RawPack<float> shift_down(const RawPack<float>& r, int s)
{
    const bool by4 = s & 4, by2 = s & 2, by1 = s & 1;
    const fvec4 z = {0.f, 0.f, 0.f, 0.f};
    const fvec4 a = by4 ? r.b : r.a, b = by4 ? z : r.b;
    const fvec4 c = by2 ? fvec4{a.z, a.w, b.x, b.y} : a, d = by2 ? fvec4{b.z, b.w, 0.f, 0.f} : b;
    RawPack<float> o;
    o.a = by1 ? fvec4{c.y, c.z, c.w, d.x} : c;
    o.b = by1 ? fvec4{d.y, d.z, d.w, 0.f} : d;
    return o;
}
template <typename T>
__device__ __forceinline__ RawPack<T> shift_down(const RawPack<T>& r, int s)
{
    const bool by4 = s & 4, by2 = s & 2, by1 = s & 1;
    const uvec4 a = by4 ? uvec4{r.u.z, r.u.w, 0u, 0u} : r.u;
    const uvec4 b = by2 ? uvec4{a.y, a.z, a.w, 0u} : a;
    RawPack<T> o;
    o.u = by1 ? uvec4{(b.x >> 16) | (b.y << 16), (b.y >> 16) | (b.z << 16), (b.z >> 16) | (b.w << 16), b.w >> 16} : b;
    return o;
}

// ------------------------------------------------------------------ rows of any length
// A [rows, hidden] tensor walked in packs of 8 columns counted from each row's start.  RAG = false: hidden is a whole
// number of packs, every access aligned.  RAG = true: any hidden.  Rows then start at any element, so a pack is a 128-bit access
// that is aligned to the element only (the hardware takes it; it may touch two lines), the last pack of a row has
// hidden % 8 elements and goes element by element, and a pack's dropout lanes come from two groups.
typedef uint32_t any4 __attribute__((ext_vector_type(4), aligned(2)));
template <typename T, bool RAG>
struct RowPackIO {
    int hidden, ppr;                                             // columns; packs per row, the cut one included
    __host__ __device__ explicit RowPackIO(int h) : hidden(h), ppr(RAG ? (h + kPack - 1) / kPack : h / kPack) {}

    __device__ __forceinline__ int64_t element(int64_t row, int cp) const { return RAG ? row * hidden + cp * kPack : (row * ppr + cp) * kPack; }
    // A load in two steps, so that many can be in flight: `ahead` only loads, `settle` (at the first use) makes the pack of it.
    template <bool NT>
    __device__ __forceinline__ RawPack<T> load(const T* __restrict__ base, int64_t row, int cp) const
    {
        return settle(ahead<NT>(base, row, cp), cp);
    }
    __device__ __forceinline__ RawPack<T> settle(const RawPack<T>& r, int cp) const
    {
        if constexpr (!RAG) return r;
        const int left = hidden - cp * kPack;
        return shift_down(r, left < kPack && hidden >= kPack ? kPack - left : 0);
    }
    template <bool NT>
    __device__ __forceinline__ RawPack<T> ahead(const T* __restrict__ base, int64_t row, int cp) const
    {
        const T* p = base + element(row, cp);
        if constexpr (!RAG) return load_raw<T, NT>(p);
        const int left = hidden - cp * kPack;
        if (hidden < kPack) {                                    // uniform: rows shorter than a pack
            RawPack<T> r;
            if constexpr (sizeof(T) == 2) {
                const uint16_t* q = reinterpret_cast<const uint16_t*>(p);
                auto at = [&](int j) { const uint32_t v = q[j < left ? j : 0]; return j < left ? v : 0u; };
                r.u = uvec4{at(0) | at(1) << 16, at(2) | at(3) << 16, at(4) | at(5) << 16, at(6) | at(7) << 16};
            } else {
                auto at = [&](int j) { const float v = p[j < left ? j : 0]; return j < left ? v : 0.0f; };
                r.a = fvec4{at(0), at(1), at(2), at(3)};
                r.b = fvec4{at(4), at(5), at(6), at(7)};
            }
            return r;
        }
        // the cut pack: the row's last 8 elements, shifted down (in settle) by those that belong to the pack before (no branch;
        // one load per element behind branches took 0.8 us each, 14 of them in a row in the embedding's forward)
        const int s = left < kPack ? kPack - left : 0;
        RawPack<T> r;
        if constexpr (sizeof(T) == 2) {
            r.u = *reinterpret_cast<const any4*>(p - s);
        } else {
            r.a = __builtin_bit_cast(fvec4, static_cast<uvec4>(*reinterpret_cast<const any4*>(p - s)));
            r.b = __builtin_bit_cast(fvec4, static_cast<uvec4>(*reinterpret_cast<const any4*>(p - s + 4)));
        }
        return r;
    }
    template <bool NT>
    __device__ __forceinline__ void put(T* base, int64_t row, int cp, const RawPack<T>& r) const
    {
        T* p = base + element(row, cp);
        if constexpr (!RAG) {
            store_raw<T, NT>(p, r);
        } else {
            const int left = hidden - cp * kPack;
            if (left >= kPack) {
                if constexpr (sizeof(T) == 2) {
                    *reinterpret_cast<any4*>(p) = r.u;
                } else {
                    *reinterpret_cast<any4*>(p) = __builtin_bit_cast(uvec4, r.a);
                    *reinterpret_cast<any4*>(p + 4) = __builtin_bit_cast(uvec4, r.b);
                }
            } else if constexpr (sizeof(T) == 2) {
                uint16_t* q = reinterpret_cast<uint16_t*>(p);
#pragma unroll
                for (int j = 0; j < 7; ++j)
                    if (j < left) q[j] = static_cast<uint16_t>(r.u[j / 2] >> (16 * (j & 1)));
            } else {
#pragma unroll
                for (int j = 0; j < 7; ++j)
                    if (j < left) p[j] = j < 4 ? r.a[j & 3] : r.b[j & 3];
            }
        }
    }
    template <bool NT>
    __device__ __forceinline__ void store(T* base, int64_t row, int cp, const float (&f)[8]) const
    {
        put<NT>(base, row, cp, pack_raw<T>(f));
    }
    __device__ __forceinline__ void factors(const DropoutParams& d, int64_t row, int cp, float (&k)[8]) const
    {
        if constexpr (RAG) dropout_factors8_any(d, static_cast<uint64_t>(element(row, cp)), k);
        else dropout_factors8(d, static_cast<uint64_t>(row * ppr + cp), k);
    }
};

// The factor for one element (element-strided paths and the ragged last pack of a flat walk: one Philox call per element).
__device__ __forceinline__ float dropout_factor1(const DropoutParams& d, uint64_t e)
{
    uint32_t w[4];
    const uint64_t g = e >> 3;
    philox4x32_10(static_cast<uint32_t>(g), static_cast<uint32_t>(g >> 32), d.ctr2, d.ctr3, d.key0, d.key1, w);
    const uint32_t lane = static_cast<uint32_t>(e) & 7u;
    const uint32_t word = lane < 2 ? w[0] : lane < 4 ? w[1] : lane < 6 ? w[2] : w[3];
    const uint32_t r16 = (word >> (16u * (lane & 1u))) & 0xFFFFu;
    return r16 >= d.t16 ? d.scale : 0.0f;
}

}  // namespace lsq
