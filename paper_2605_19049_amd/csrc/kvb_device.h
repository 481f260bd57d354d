// kvb -- KVBuffer-style Gated DeltaNet decoding, HIP kernels for gfx950 behind the C ABI of
// include/kvb.h.  This header holds what the translation units share: device helpers, the
// argument structs of the kernels, and the launch plumbing.
//   kvb_step_kernel.h    kvb_step_kernel and kvb_buffer_step_kernel (decode); instantiated per
//                        (input type, record type) by kvb_step_f32.hip, kvb_step_bf16.hip,
//                        kvb_step_bf16_r16.hip, kvb_step_f16.hip, kvb_step_f16_r16.hip
//   kvb_verify_kernel.h  kvb_verify_mfma_kernel; instantiated by kvb_verify_bf16.hip, _f16.hip, _f32.hip
//   kvb_flush.hip        kvb_flush_mfma_kernel, kvb_flush_rows_kernel, kvb_compact_kernel
//   kvb_direct.hip       kvb_direct_mfma_kernel, kvb_direct_rows_kernel
//   kvb_api.hip          argument checks, the extern "C" entry points, the kernel timer
//
// Element types (Sec. 4.1: 16-bit vectors and records beside a fp32 state): TIn is the type of
// q, k, v and of the buffered keys (float, bf16_t or f16_t), TRec that of the buffered delta
// values (float, or TIn when that is 16-bit); outputs are fp32 or TIn, chosen at run time at the
// final store.  All arithmetic is fp32, or on 16-bit pieces of fp32 values with fp32 sums.
//
// Work decomposition: one 256-thread workgroup per (request b, v-head h), in
// kvb_buffer_step_kernel per request and one or two v-heads; the committed state S0[dk][dv] (fp32, dv contiguous, 64 KB at
// d = 128) is streamed exactly once per call.  Besides the state a unit needs
// its buffered keys k_l, delta values u_l and cumulative log decays G_l (paper
// App. A.1, the paragraph after Eq. 16), a few KB.
//   kvb_step_kernel         decode, one token: vector ALUs; a thread owns
//                           4 adjacent dv columns of 16 state rows (16-byte loads)
//   kvb_buffer_step_kernel  decode without a state: one workgroup per (b, one or two v-heads of a qk-head)
//   kvb_verify_mfma_kernel  verify: matrix cores; a wave owns 32 dv columns (16 at d <= 64)
//   kvb_flush_mfma_kernel   deferred state update, 16-bit inputs / d = 128: matrix cores on exact
//                           16-bit pieces of the fp32 factor
//   kvb_flush_rows_kernel   the same for the other types and head sizes: fp32 matrix instruction
//   kvb_direct_mfma_kernel  short contexts, 16-bit inputs / d = 128: matrix cores throughout
//   kvb_direct_rows_kernel  short contexts, other types and head sizes: fp32 matrix instruction, block row by block row
//
// Notation follows App. A.1: gamma_i = exp(G_i), Gamma_il = exp(G_i - G_l).

#ifndef KVB_DEVICE_H
#define KVB_DEVICE_H

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <tuple>
#include <type_traits>

#include "kvb.h"

struct kvb_timer {
    hipEvent_t start, stop;
};

namespace kvb_impl {

constexpr int NT = 256;      // threads per workgroup
constexpr int NW = NT / 64;  // wavefronts per workgroup
constexpr int FILL_MASK = 0xFFFF;
constexpr int TICKET_ONE = 1 << 16;

struct bf16_t {
    uint16_t bits;
};
struct f16_t {
    uint16_t bits;
};

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float((uint32_t)x.bits << 16); }
__device__ __forceinline__ float to_f32(f16_t x) { return (float)__builtin_bit_cast(_Float16, x.bits); }

// Rounding to a storage type, to nearest even (the hardware conversions of gfx950).
template <typename T>
__device__ __forceinline__ T from_f32(float x);
template <>
__device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <>
__device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return bf16_t{__builtin_bit_cast(uint16_t, (__bf16)x)}; }
template <>
__device__ __forceinline__ f16_t from_f32<f16_t>(float x) { return f16_t{__builtin_bit_cast(uint16_t, (_Float16)x)}; }
// x as the storage type T will hold it
template <typename T>
__device__ __forceinline__ float rounded_to(float x) { return to_f32(from_f32<T>(x)); }

// The two 16-bit elements packed in one word, and two floats packed into one.
template <typename T>
__device__ __forceinline__ float2 unpack_pair(uint32_t w)
{
    if constexpr (__is_same(T, bf16_t)) {
        return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xFFFF0000u));
    } else {
        const f16x2_t h = __builtin_bit_cast(f16x2_t, w);
        return make_float2((float)h[0], (float)h[1]);
    }
}
template <typename T>
__device__ __forceinline__ uint32_t pack_pair(float lo, float hi)
{
    return (uint32_t)from_f32<T>(lo).bits | ((uint32_t)from_f32<T>(hi).bits << 16);
}

// 8 consecutive elements starting at p (p is 16-byte aligned) as untouched bits: issuing a load and converting its result are
// kept apart so that no wait lands between two loads.
template <typename T>
struct Raw8 {
    uint4 w;
};
template <>
struct Raw8<float> {
    float4 a, b;
};
__device__ __forceinline__ Raw8<float> load_raw8(const float *p)
{
    return Raw8<float>{*reinterpret_cast<const float4 *>(p), *reinterpret_cast<const float4 *>(p + 4)};
}
template <typename T>
__device__ __forceinline__ Raw8<T> load_raw8(const T *p)
{
    return Raw8<T>{*reinterpret_cast<const uint4 *>(p)};
}
__device__ __forceinline__ void unpack8(const Raw8<float> &r, float (&o)[8])
{
    o[0] = r.a.x; o[1] = r.a.y; o[2] = r.a.z; o[3] = r.a.w;
    o[4] = r.b.x; o[5] = r.b.y; o[6] = r.b.z; o[7] = r.b.w;
}
template <typename T>
__device__ __forceinline__ void unpack8(const Raw8<T> &r, float (&o)[8])
{
    const float2 a = unpack_pair<T>(r.w.x), b = unpack_pair<T>(r.w.y), c = unpack_pair<T>(r.w.z), d = unpack_pair<T>(r.w.w);
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
    o[4] = c.x; o[5] = c.y; o[6] = d.x; o[7] = d.y;
}

// 4 and 2 consecutive elements of a record array (delta values), raw and converted.
template <typename T>
struct Raw4 {
    uint2 w;
};
template <>
struct Raw4<float> {
    float4 a;
};
__device__ __forceinline__ Raw4<float> load_raw4(const float *p) { return Raw4<float>{*reinterpret_cast<const float4 *>(p)}; }
template <typename T>
__device__ __forceinline__ Raw4<T> load_raw4(const T *p) { return Raw4<T>{*reinterpret_cast<const uint2 *>(p)}; }
__device__ __forceinline__ float4 unpack4(const Raw4<float> &r) { return r.a; }
template <typename T>
__device__ __forceinline__ float4 unpack4(const Raw4<T> &r)
{
    const float2 a = unpack_pair<T>(r.w.x), b = unpack_pair<T>(r.w.y);
    return make_float4(a.x, a.y, b.x, b.y);
}
template <typename T>
struct Raw2 {
    uint32_t w;
};
template <>
struct Raw2<float> {
    float2 a;
};
__device__ __forceinline__ Raw2<float> load_raw2(const float *p) { return Raw2<float>{*reinterpret_cast<const float2 *>(p)}; }
template <typename T>
__device__ __forceinline__ Raw2<T> load_raw2(const T *p) { return Raw2<T>{*reinterpret_cast<const uint32_t *>(p)}; }
__device__ __forceinline__ float2 unpack2r(const Raw2<float> &r) { return r.a; }
template <typename T>
__device__ __forceinline__ float2 unpack2r(const Raw2<T> &r) { return unpack_pair<T>(r.w); }

// Stores of results.  A plain store leaves its line in the XCD's L2, and a kernel ends by writing all such lines back: the
// next one waits for that.  These go through to memory as they are made (device scope, nobody is ordered by them) or, NT,
// past the caches, for what a state that is streamed too leaves behind.  With plain stores / through, us: kvb_decode_flush, 8
// steps of 8 requests of 32 heads 49.5 / 46.1, of 24 103.3 / 96.6, 16 steps of 64 437 / 433; kvb_verify and commit of 24
// requests of 16 heads, fp32, 20.2 / 19.0.  PLAIN: a plain store all the same, for what is read back soon (kvb_decode_flush,
// small folds by kvb_flush) and for the parts of a line that end a short launch (kvb_direct); the lines are measured there.
template <bool NT, bool PLAIN = false, typename T>
__device__ __forceinline__ void put(T *p, const T &x)
{
    static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16);
    typedef uint32_t v2 __attribute__((ext_vector_type(2)));
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    using Bits = std::conditional_t<sizeof(T) == 2, uint16_t, std::conditional_t<sizeof(T) == 4, uint32_t, std::conditional_t<sizeof(T) == 8, v2, v4>>>;
    if constexpr (NT)
        __builtin_nontemporal_store(__builtin_bit_cast(Bits, x), reinterpret_cast<Bits *>(p));
    else if constexpr (PLAIN)
        *reinterpret_cast<Bits *>(p) = __builtin_bit_cast(Bits, x);
    else if constexpr (sizeof(T) == 16)
        // (the widest that there is an atomic store of is 8 bytes.  The compiler does not look inside: for two wait states no
        // vector instruction may overwrite the data of a store of more than 8 bytes, and it places them behind its own stores only)
        asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(__builtin_bit_cast(v4, x)) : "memory");
    else if constexpr (sizeof(T) == 8)
        __hip_atomic_store(reinterpret_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        __hip_atomic_store(reinterpret_cast<Bits *>(p), __builtin_bit_cast(Bits, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A plain or non-temporal store of 16 bytes at a scalar address and the lane's offset (a register to a store's address, not two: with
// two the fold of fp32 inputs and 64-record windows spilled 4, and 8 steps of 8 requests took 45.3 us instead of 45.0).
template <bool NT>
__device__ __forceinline__ void put_at(float *base, uint32_t lane_at, const float4 &x)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    v4f *p = reinterpret_cast<v4f *>(reinterpret_cast<char *>(base) + lane_at);
    const v4f v = {x.x, x.y, x.z, x.w};
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}
// The same of already-rounded or to-be-rounded values into an array of type T.
template <bool NT = false>
__device__ __forceinline__ void store2(float *p, float x, float y) { put<NT>(reinterpret_cast<float2 *>(p), make_float2(x, y)); }
template <bool NT = false, typename T>
__device__ __forceinline__ void store2(T *p, float x, float y) { put<NT>(reinterpret_cast<uint32_t *>(p), pack_pair<T>(x, y)); }
// The same as streaming (non-temporal) stores, for results that this kernel does not read again.
__device__ __forceinline__ void store2_nt(float *p, float x, float y)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(v2f{x, y}, reinterpret_cast<v2f *>(p));
}
template <typename T>
__device__ __forceinline__ void store2_nt(T *p, float x, float y)
{
    static_assert(sizeof(T) == 2, "a 16-bit storage type");
    __builtin_nontemporal_store(pack_pair<T>(x, y), reinterpret_cast<uint32_t *>(p));
}
template <bool NT = false, bool PLAIN = false>
__device__ __forceinline__ void store4(float *p, const float4 &v) { put<NT, PLAIN>(reinterpret_cast<float4 *>(p), v); }
template <bool NT = false, typename T>
__device__ __forceinline__ void store4(T *p, const float4 &v)
{
    put<NT>(reinterpret_cast<uint2 *>(p), make_uint2(pack_pair<T>(v.x, v.y), pack_pair<T>(v.z, v.w)));
}
template <bool NT = false, bool PLAIN = false, typename T>
__device__ __forceinline__ void store1(T *p, float x) { put<NT, PLAIN>(p, from_f32<T>(x)); }

// The output array has a run-time element type (KVB_F32 or the 16-bit input type TIn): the
// stores sit at the end of every kernel, where a uniform branch costs nothing.
template <typename TIn>
struct Out {
    void *p;
    bool wide;   // fp32 elements
    template <bool NT = false, bool PLAIN = false>
    __device__ __forceinline__ void put1(size_t i, float x) const
    {
        if (sizeof(TIn) == 4 || wide)
            store1<NT, PLAIN>(static_cast<float *>(p) + i, x);
        else
            store1<NT, PLAIN>(static_cast<TIn *>(p) + i, x);
    }
    __device__ __forceinline__ void put2(size_t i, float x, float y) const
    {
        if constexpr (sizeof(TIn) == 4) {
            store2(static_cast<float *>(p) + i, x, y);
        } else {
            if (wide)
                store2(static_cast<float *>(p) + i, x, y);
            else
                store2(static_cast<TIn *>(p) + i, x, y);
        }
    }
    // element i0 + i, i0 a scalar (64-bit) and i the lane's (its byte offset in 32 bits)
    __device__ __forceinline__ void put2_nt(size_t i0, uint32_t i, float x, float y) const
    {
        if (sizeof(TIn) == 4 || wide)
            store2_nt(reinterpret_cast<float *>(static_cast<char *>(p) + 4 * i0 + 4 * i), x, y);
        else if constexpr (sizeof(TIn) == 2)
            store2_nt(reinterpret_cast<TIn *>(static_cast<char *>(p) + 2 * i0 + 2 * i), x, y);
    }
    template <bool NT = false>
    __device__ __forceinline__ void put4(size_t i, const float4 &v) const
    {
        if constexpr (sizeof(TIn) == 4) {
            store4<NT>(static_cast<float *>(p) + i, v);
        } else {
            if (wide)
                store4<NT>(static_cast<float *>(p) + i, v);
            else
                store4<NT>(static_cast<TIn *>(p) + i, v);
        }
    }
};

// v_mfma_f32_16x16x32 on 16-bit operands of type T given as raw bits (8 elements per lane).
template <typename T>
__device__ __forceinline__ f32x4_t mfma16x32(const uint4 &a, const uint4 &b, const f32x4_t &c)
{
    if constexpr (__is_same(T, bf16_t))
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                       c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b),
                                                      c, 0, 0, 0);
}

// Waits until the matrix instructions that produce these values have written them.  The compiler
// inserts such waits itself, but where a block of matrix instructions is skipped by a branch it looked back
// along the path through that block only, and the other path read a register before its sum had arrived; sums
// that end in such blocks are therefore settled by hand before anything else reads them.  (The wait states from
// a matrix instruction to a vector read of its result: 16-bit 16x16x32 8, fp32 16x16x4 10.)
constexpr int SETTLE_16BIT = 8, SETTLE_FP32 = 10;
template <int STATES>
__device__ __forceinline__ void settle(f32x4_t &x)
{
    asm volatile("s_nop %1" : "+v"(x) : "n"(STATES - 1));
}
template <int STATES>
__device__ __forceinline__ void settle(f32x4_t &x, f32x4_t &y)
{
    asm volatile("s_nop %2" : "+v"(x), "+v"(y) : "n"(STATES - 1));
}
template <int STATES, int N>
__device__ __forceinline__ void settle(f32x4_t (&x)[N][2])
{
    settle<STATES>(x[0][0], x[0][1]);   // (volatile: the ones below stay behind it)
#pragma unroll
    for (int i = 1; i < N; ++i)
        asm volatile("" : "+v"(x[i][0]), "+v"(x[i][1]));
}

// Whether the matrix products of a wave came out finite: cut into 16-bit pieces, or multiplied as whole tiles with
// their zeros, an infinity or a value out of range becomes NaN, and every kernel of that kind then does the wave's part
// again in fp32 over the exact terms.  largest: the largest magnitude so far, NaN once there was one.
__device__ __forceinline__ float largest(float so_far, float x, float y)
{
    // (v_maximum3_f32, which hands NaN on)
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(so_far, __builtin_fabsf(x)), __builtin_fabsf(y));
}
__device__ __forceinline__ float largest(float so_far, const f32x4_t &x)
{
    return largest(largest(so_far, x[0], x[1]), x[2], x[3]);
}
__device__ __forceinline__ bool all_finite(float largest)
{
    // (as bits: the compiler turned "< Inf" into "!= Inf", which NaN passes)
    return __all(__float_as_uint(largest) < 0x7F800000u);
}

// One 16-byte piece of the state tile.  STREAM: non-temporal load, for a state that will
// not be read again before the last-level cache has turned over (measured on MI355X:
// +14% at 1 GiB of state per call, -5% at 128 MiB, which the 256 MB cache keeps).
template <bool STREAM>
__device__ __forceinline__ float4 load_state4(const float4 *p)
{
    if constexpr (STREAM) {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
        return make_float4(t.x, t.y, t.z, t.w);
    } else {
        return *p;
    }
}

// The same for an 8-byte piece.
template <bool STREAM>
__device__ __forceinline__ float2 load_state2(const float *p)
{
    if constexpr (STREAM) {
        typedef float v2f __attribute__((ext_vector_type(2)));
        const v2f t = __builtin_nontemporal_load(reinterpret_cast<const v2f *>(p));
        return make_float2(t.x, t.y);
    } else {
        return *reinterpret_cast<const float2 *>(p);
    }
}

__device__ __forceinline__ void fma4(float4 &acc, float c, const float4 &x)
{
    acc.x = fmaf(c, x.x, acc.x);
    acc.y = fmaf(c, x.y, acc.y);
    acc.z = fmaf(c, x.z, acc.z);
    acc.w = fmaf(c, x.w, acc.w);
}

// The workgroups of one request share fill[slot].  Every wave reads the word when it starts, and its value decides a
// branch; then comes a barrier, and behind it the workgroup's first thread adds to bits 16.., which says that ALL waves
// of its workgroup have read.  (Without the barrier a wave that has yet to read could find the word complete and take the
// new fill for the old one.)  The barrier is bare: it waits for the waves, not for their memory operations.  Relaxed
// ordering is enough and matters: the reads have completed when the word is added to (their values decided branches),
// and nothing else is communicated through it.  Acquire / release ordering at device scope would make every workgroup
// write back and invalidate its L2, which costs more than the kernel's whole memory traffic.
//
// advance_fill: the usual way.  Nobody waits for the word: each workgroup adds its share and the shares of all of them
// add up to new - old.  The first workgroup's share holds the change of the count and a negative number of workgroups,
// so the word is negative from then on until the last share brings bits 16.. back to zero.  A wave that finds it
// negative reads the new count and knows the old one from it (fill_before, fill_before_commit); a positive word holds
// the old count.  The atomics return nothing, so no wave's end waits for them: with a ticket that came back to the
// workgroup holding it, which is what this replaced, 64 requests of 32 heads took 469 us for 16 steps of
// kvb_decode_flush and take 460, a single request 74.6 and 71.2, 13 of 8 heads 97.3 and 94.7.
//
// Additions to one 128-byte line pass one at a time, about 10 ns each, whatever the word or the XCD, and reads of the line
// queue behind them.  With the fills of 32 slots to a line that is what bounded launches of a few hundred workgroups on
// (KVB_STORE_FILL_APART gives each slot a line).  Packed / apart, us: kvb_decode_flush, 8 steps of 8 requests of 32 heads 61.2 / 49.7,
// 16 requests 86.6 / 73.0, 24 114 / 104, d = 64 8 requests 56.9 / 39.8, 60 requests 127 / 98; kvb_verify and commit of 24
// requests 28.7 / 26.4; kvb_direct and 16 steps of kvb_decode without a state, 24 contexts, 121.7 / 106.2; one request 60.5 / 60.9.
//
// publish_fill: a ticket that comes back; whoever holds the last one stores the new plain count.  For changes from
// which the old count does not follow (a fold that was due earlier, or by kvb_flush; a commit cut off at cap), where
// the word is positive throughout.  It is taken once the loads are in flight (take_ticket) and looked at at the end.
// All of these hold the barrier, so every thread of the workgroup calls them (advance_fill_read, take_ticket: those
// behind a barrier of the caller's are called by all, too).
constexpr int MAX_FILL_WG = 1 << 15;   // workgroups of a request that bits 16.. can count, the sign apart
__host__ __device__ inline int fill_share(bool first, int nwg, int change)   // nwg <= MAX_FILL_WG
{
    return first ? change - (nwg - 1) * TICKET_ONE : TICKET_ONE;
}
// the fill before a token was appended to it; folded: what it was if that token brought it to zero
__host__ __device__ inline int fill_before(int word, int folded)
{
    const int low = word & FILL_MASK;
    return word >= 0 ? low : low > 0 ? low - 1 : folded;
}
// the fill before `accepted` > 0 records were committed
__host__ __device__ inline int fill_before_commit(int word, int accepted)
{
    return (word & FILL_MASK) - (word < 0 ? accepted : 0);
}
__device__ __forceinline__ void advance_fill_read(int32_t *word, bool first, int nwg, int change)   // every wave is known to have read the word
{
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(word, fill_share(first, nwg, change), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void advance_fill(int32_t *word, bool first, int nwg, int change)
{
    __builtin_amdgcn_s_barrier();
    advance_fill_read(word, first, nwg, change);
}
__device__ __forceinline__ int take_ticket(int32_t *word)
{
    __builtin_amdgcn_s_barrier();
    return threadIdx.x == 0 ? __hip_atomic_fetch_add(word, TICKET_ONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
}
__device__ __forceinline__ void publish_if_last(int32_t *word, int ticket, int nwg, int new_fill)   // thread 0
{
    // Opaque to the optimiser: otherwise the shift below is hoisted next to the atomic and
    // the wave waits there for the ticket (and for every load it issued before it).
    asm volatile("" : "+v"(ticket));
    if ((ticket >> 16) == nwg - 1)
        __hip_atomic_store(word, new_fill, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_fill(int32_t *word, int nwg, int new_fill)
{
    const int ticket = take_ticket(word);
    if (threadIdx.x == 0)
        publish_if_last(word, ticket, nwg, new_fill);
}

template <bool NT = false, bool PLAIN = false>
__device__ __forceinline__ void store_raw8(float *p, const Raw8<float> &r)
{
    store4<NT, PLAIN>(p, r.a);
    store4<NT, PLAIN>(p + 4, r.b);
}
template <bool NT = false, bool PLAIN = false, typename T>
__device__ __forceinline__ void store_raw8(T *p, const Raw8<T> &r)
{
    put<NT, PLAIN>(reinterpret_cast<uint4 *>(p), r.w);
}

// x / d for a scalar d > 0, x >= 0.  The division stands ahead of the load of slot[b], the head of every dependent chain;
// in general it is some fifteen dependent instructions through the vector ALU, and head counts are powers of two mostly:
// 16 steps of one request 62.7 -> 61.7 us, of 64 430 -> 427, kvb_direct of 2 contexts 8.8 -> 8.6.  Other head counts pay for the test; Hv / Hk comes with the arguments, so that one
// division is left behind the slot: 217 contexts of 9 heads of 32 12.1 us before the test, 12.3 with it and both, 12.0 so; 16
// steps of one request of 32 heads 57.0 -> 55.9.
__host__ __device__ inline int quotient(int x, int d)
{
    return (d & (d - 1)) == 0 ? x >> __builtin_ctz(d) : x / d;
}

// s, behind the loads of all that is listed: from here on they are in scalar registers, requested ahead and waited for together
// with s.  Left alone the compiler requested the argument block in four pieces and waited for each in turn, for the first (the head
// counts of a division) even ahead of the load of s: that chain is the start of every workgroup.  us without and with: 16 steps of
// kvb_decode_flush of one request 61.2 / 59.7, 8 steps of 8 requests 47.0 / 45.2, 16 steps of 64 441 / 436; kvb_verify and commit of 24
// requests 24.3 / 23.6, of 7 trees 19.8 / 19.0; 16 steps of kvb_decode without a state, 24 contexts, 104.5 / 100.4.  (Not a volatile statement: behind one the compiler takes memory as changed and loads scalars, the fill among them,
// through the vector memory path, where each waits for every load before it.)
template <typename A, typename B, typename C, typename D, typename E, typename F, typename G>
__device__ __forceinline__ int with_registers(int s, A a, B b, C c, D d, E e, F f, G g)
{
    asm("" : "+s"(s) : "s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f), "s"(g));
    return s;
}
template <typename A, typename B, typename C, typename D, typename E, typename F, typename G, typename... T>
__device__ __forceinline__ int with_registers(int s, A a, B b, C c, D d, E e, F f, G g, T... t)
{
    asm("" : "+s"(s) : "s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f), "s"(g));
    return with_registers(s, t...);
}

// Which unit a workgroup of kvb_direct takes, whose work grows with the context: the heads of a request are dealt
// over all XCDs, one qk-head with its r v-heads (which share keys and queries through the XCD's L2) at a time; with
// whole requests on one XCD, the XCD that drew the longest contexts set the
// end of the launch (256 contexts of ~U(1,64): 118 -> 110 us; 96 of ~U(1,128): 130 -> 115 us).  The order of the requests is
// another matter (longest_first).
// Rounds of 8 qk-heads are dealt, one to an XCD; the units of the qk-heads that are left (fewer than 8) go one by one.
// Where some are left, from 1024 units on (four workgroups a CU; below that all run at once, and what the v-heads of a
// qk-head share is worth less than spreading contexts of one length over the CUs).  Against unit = workgroup id, d =
// 128 unless said, contexts of ~U(1, 64): 255 requests of 4/8 heads 32.9 -> 32.3 us, up to 128 tokens 80.3 -> 77.4; 255
// of 2/16 heads, fp16, 46.2 -> 43.6; 101 of 4/16 heads 26.0 -> 26.8, up to 112 tokens 57.9 -> 56.7, d = 64 26.6 -> 25.4;
// dealt all the same below the line: 61 of 4/8 heads 14.1 -> 14.1, 13 of 4/8 11.1 -> 11.3, 77 of 3/9 16.9 -> 17.6.
// The rule in one word: rounds in the upper 20 bits, r in the lower 12 (0 rounds: unit = workgroup id).
__host__ __device__ inline int deal_of(int blocks, int r)
{
    const int rounds = r < 4096 && (blocks % (8 * r) == 0 || blocks >= 1024) ? blocks / (8 * r) : 0;
    return (rounds < 0x7FFFF ? rounds : 0x7FFFF) << 12 | (r & 4095);
}
__host__ __device__ inline int dealt_unit(int x, int deal)
{
    const int r = deal & 4095, rounds = deal >> 12, j = x / 8;
    if (x >= 8 * r * rounds)
        return x;
    const int of = quotient(j, r);
    return (of * 8 + x % 8) * r + j - of * r;
}

// The same for the kernels whose workgroups share a request's fill word, over n workgroups of which each qk-head has r: dealt in
// rounds of 8 qk-heads, or XCD x works on one contiguous eighth, so that what the heads of a request read in common is in one L2,
// or unit = workgroup id.  In one word, steps and a power of two, without a branch ahead of the load of the slot: workgroup
// x = 8 j + c takes c * (the upper 27 bits) + 8 (j & -run) + (j & run - 1), run = 1 << the lower 5 bits.
// Dealt, the requests that fold (and write their states back) are no XCD's alone.  Eighths / dealt, with a
// line to each fill word, us: kvb_decode_flush, 16 steps of 64 requests of
// 32 heads 436 / 397, 4 of 500 935 / 917, 8 of 24 96.4 / 92.4, of 16 67.1 / 62.7, of 32 of 16 69.8 / 67.4; below 512 units it
// depends on where the states lie, 8 steps of 12 of 32 heads 52.0 / 50.0, of 20 of 16 53.2 / 52.9 or 63.2, of 60 of 8 60.9 / 64.4.
// kvb_decode without a state, 128 requests 424 / 417, 24 99.7 / 103, 60 of 16 heads 48.2 / 49.0.  kvb_verify and commit, both alike
// (one dealt and the other not is 1 to 6 % slower than either): 128 requests 88.6 / 83.6, 300 182 / 173, 60 of 16 heads 32.7 / 31.7,
// 24 of 32 23.8 / 23.3, 24 of 16 18.5 / 18.5, 40 of 8 19.7 / 20.2.  The fold after kvb_direct, which deals at any size, of 10 contexts
// 28.9 / 27.9, of 100 126 / 124.
// Packed fill words (32 slots to a line): dealt, the additions to a line come from all XCDs, which is dearest where the slots of a batch are
// neighbours.  Only kvb_decode_flush at d = 128 below 832 units is faster so in any order of slots; all else stays in eighths.  Before units were dealt
// and results sent through / eighths / dealt, slots in order and (at random), us: kvb_decode_flush, 16 steps at C = 8, 16 requests of 32 heads 190 /
// 188 / 162 (162 / 155 / 152), 20 223 / 214 / 202 (201 / 198 / 160), 24 226 / 218 / 213 (214 / 212 / 206), 28 234 / 239 / 249 (234 / 231 / 228), 31 242 /
// 247 / 274 (254 / 267 / 253), 48 360 / 360 / 388 (362 / 361 / 352), 64 451 / 459 / 553 (458 / 469 / 450), 48 of 16 206 / 211 / 200 (205 / 209 / 200), 60 of 16 232 /
// 235 / 266 (233 / 255 / 246); threshold 1, 24 277 / 263 / 272 (266 / 269 / 268), 31 316 / 317 / 360 (314 / 337 / 335).  kvb_decode and kvb_flush, 16 steps
// at C = 16, 24 280 / 257 / 263 (276 / 250 / 276), 64 532 / 501 / 641 (615 / 578 / 557); kvb_decode, 8 steps, 24 100 / 97 / 104 (94 / 94 / 93), 32 114 /
// 111 / 134 (111 / 108 / 118), 64 185 / 180 / 247 (200 / 198 / 198); kvb_direct of up to 16 tokens and fold, 24 29.7 / 28.2 / 30.4 (29.6 / 27.4 / 27.9).  Slots at
// random: d = 64, kvb_decode_flush, 60 requests 124 / 121 / 131, 200 210 / 211 / 254; kvb_verify and commit, 24 requests 32.5 / 31.2 / 31.6, 48 46.9 / 43.8 /
// 46.1, 128 87.3 / 86.3 / 87.9, 300 188 / 189 / 184; kvb_decode without a state, 128 requests 21.3 / 21.0 / 22.4.
constexpr int DEAL_STEP = 512, DEAL_BUFFER_STEP = 1024, DEAL_SPEC = 512;   // the least units (workgroups) to deal
constexpr int PACKED_END = 832, LEVEL_STEP = 1024, NO_DEALING = 0x7FFFFFFF;
// Where every step folds, no XCD has less to do, and whole eighths keep what the heads of a request share, and the state from one step to the
// next, in one L2: at threshold 1 (d = 128: from 1024 units on), and at 2 of a streamed state, nothing is dealt.  Eighths / dealt, us a step of
// threshold 1: 16 requests of 32 heads 10.5 / 10.0, 24 16.3 / 14.5, 28 19.0 / 17.4 to 19.5, 32 20.6 / 20.7, 48 29.8 / 30.4, 64 39.1 / 40.6 (fp16 39.6 /
// 41.0), 96 57.8 / 59.9, 128 82.0 / 81.1, 256 184 / 186; fp32, 24 15.8 / 14.6; 96 of 8 heads 16.3 / 14.6, 128 20.6 / 20.8, 400 60.7 / 62.7; d = 64, 32 of 16
// heads 5.65 / 5.80, 200 19.2 / 19.6; 4 steps of 400 of 32 1175 / 1223.  Threshold 2, 16 steps: 64 requests 583 / 515, 128 (8) 537 / 509, streamed,
// 256 1120 / 1140, 400 (4 steps) 873 / 892; threshold 3, streamed, 256 1022 / 1005.
// kvb_flush without accepted drafts comes behind kvb_direct, which deals at any size, or behind kvb_decode.  The two are alike, or a fold
// has its state and records in other L2s than its decode: so kvb_decode deals at any size as well.  kvb_decode in eighths and the fold dealt /
// both in eighths / both dealt, 16 steps of kvb_decode and kvb_flush: C = 16, 4 requests of 32 heads 102.9 / 98.6 / 99.4, 8 124 / 117 / 114, 15
// 159 / 151 / 156; C = 1, 4 requests 169 / 137 / 144, 8 233 / 164 / 181, 15 393 / 242 / 265 (before all this 175, 240, 315); kvb_direct and the
// fold, 10 contexts dealt / the fold in eighths 31.8 / 36.1, 15 36.3 / 40.3.  kvb_decode alone, 8 steps of 4 requests, eighths / dealt 39.7 /
// 38.8, 8 39.2 / 39.6 to 44.8 with where the states lie, 15 61.6 / 58.2.
// From how many units on kvb_step_kernel deals, with n of them (threshold: 0 where it does not fold; appends: not for kvb_verify of one
// draft, which goes with its commit; apart: a line to each fill word)
inline int step_deals_from(int d, int n, int threshold, bool stream, bool appends, bool apart)
{
    const bool level = threshold > 0 && threshold <= (stream ? 2 : 1) && (d < 128 || n >= LEVEL_STEP);
    if (!apart)
        return d == 128 && threshold > 0 && n < PACKED_END ? DEAL_STEP : NO_DEALING;
    return level ? NO_DEALING : threshold == 0 && appends ? 0 : DEAL_STEP;
}
// kvb_flush where (nearly) every request folds, d = 128: behind a dealt kvb_verify or kvb_decode the fold is faster in eighths all the same, from
// 768 units on and while it has not much more state than the last-level cache holds (3584 units; 4096 are 256 MiB).  Dealt before and dealt / dealt
// before and eighths / both in eighths, which kvb_verify and kvb_decode cannot know to take (before all this), us: commits of 4 drafts at threshold 1,
// 16 requests of 32 heads (2 drafts) 19.1 / 24.6 / 16.4 (22.1), 24 29.9 / 28.5 / 24.1 (30.6), 40 (2) 46.8 / 42.2 / 38.2 (44.3), 64 70.3 / 63.7 /
// 61.4 (67.2), 96 99.6 / 91.6 / 89.0 (94.6), 112 (2) 120.7 / 115.8 / 116.0 (116.8), 128 140 / 150 / 138 (140), fp32, 64 73.0 / 69.7 / 68.9 (71.6),
// 200 of 8 heads 57.8 / 53.5 / 49.8 (54.9); at threshold 2, 40 44.1 / 41.2 / 38.0 (43.9), 2 drafts 37.0 / 39.7 / 36.3 (42.1), 96 90.8 / 86.5 / 85.0
// (89.5), 2 drafts 77.6 / 76.9 / 76.2 (80.2), 200 of 8 heads 53.7 / 50.2 / 46.9 (51.9); at threshold 3, 64 57.2 / 57.1 / 55.3 (60.0), at 4 49.2 / 53.8 / 52.7 (58.0).  16 steps of kvb_decode
// and kvb_flush at threshold 1, 24 443 / 426 / 359 (481), 64 1070 / 965 / 907 (1003), 96 1520 / 1398 / 1348 (1454), 128 (8 steps) 1034 / 1062 / 988
// (994); at threshold 2, 64 718 / 773 / 737 (789).  Up to two drafts, all folded in their round, stay slower than before from 4096 units on: one,
// 128 requests 129 / 135 / 124 (125), 200 206 / 207 / 202 (201); two, 128 137 (136), fp16 135 (132).
// The fold behind kvb_direct, dealt / eighths (before): up to 64 tokens, 24 contexts 38.0 / 39.3 (40.3), 64 83.6 / 86.7 (88.2), fp32, 48 87 / 97 (100); up
// to 16, 24 27.5 / 28.1 (29.9), 48 48.3 / 48.5 (49.6), fp16 45.5 / 43.8 (45.8), 96 90.9 / 89.9 (91.6), fp32, 48 53.6 / 51.4 (55.2).  So without accepted
// drafts, eighths are for buffers of up to 16 records.  (Streamed, 4096 units and more, dealt / eighths: 128 contexts of up to 64 154.8 / 159.5
// (158.9); the kernel by itself over the same 64 records a request again and again, though, 115 / 105 (104).)
// d = 64, dealt as behind / in eighths: commits at threshold 1, 60 requests of 16 heads 13.2 / 17.4 (17.7), 200 31.5 / 35.0 (37.6).
constexpr int LEVEL_FOLD = 768, LEVEL_FOLD_2 = 1536, LEVEL_FOLD_END = 3840;   // units: at threshold 1, at 2, and below
// the same for kvb_flush (commits: of accepted drafts), and for the others
inline int fold_deals_from(int d, int n, bool commits, int threshold, int cap, bool apart)
{
    const bool level = commits ? threshold == 1 || (threshold == 2 && n >= LEVEL_FOLD_2) : threshold == 1 && cap <= 16;
    if (!apart || (d == 128 && level && n >= LEVEL_FOLD && n < LEVEL_FOLD_END))
        return NO_DEALING;
    return commits ? DEAL_SPEC : 0;
}
inline int deals_from(int least, bool apart) { return apart ? least : NO_DEALING; }
inline int unit_deal(int n, int r, int least)
{
    const bool small = n < 1 << 29;
    if (small && n >= least && (r & (r - 1)) == 0 && r < 1 << 26 && n % 8 == 0 && n / 8 % r == 0)
        return (int)((uint32_t)r << 5 | (uint32_t)__builtin_ctz(r));
    return small && n % 8 == 0 ? (int)((uint32_t)(n / 8) << 5 | 31u) : 1 << 5;
}
__host__ __device__ inline int unit_of(uint32_t x, uint32_t deal)
{
    const uint32_t j = x >> 3, rest = j & ((1u << (deal & 31u)) - 1u);
    return (int)((x & 7u) * (deal >> 5) + 8u * (j - rest) + rest);
}

// The byte offset of one of 16 rows, cut off where `left` rows follow the first; own: the row times the stride.  (In 32 bits, so
// the rows behind the sixteenth are no part of the product: 127 rows leave 32 bits from 132105 heads on.)
__host__ __device__ inline uint32_t row_of_16(uint32_t own, int left, uint32_t stride)
{
    const uint32_t last = (uint32_t)(left < 15 ? left : 15) * stride;
    return own < last ? own : last;
}

// Whether kvb_direct takes the longest contexts first (how: ranked_request in kvb_direct.hip).  The sort costs every
// workgroup 0.3 to 0.6 us and shortens the end of the launch, so it needs contexts whose work differs.
// us a call in the order of the batch / sorted, 32 heads unless said:
//   up to 128 tokens, d = 128: 96 contexts, bf16, 109 / 100; 128 of up to 100, fp16, 103 / 94; 400 of up to 112, fp16,
//     473 / 451; 8 23.5 / 24.1; 4 29.0 / 29.6
//   up to 64 tokens, d = 128, bf16: 256 contexts 105 / 106; 128 57 / 58; 96 46.6 / 47.6; 64 32.7 / 29.7; 24 16.7 / 16.4;
//     16 16.5 / 15.2; 12 15.5 / 14.0; 8 12.8 / 13.4; fp16: 256 84 / 86; 96 37.9 / 37.8; 40 20.5 / 18.2; 8 11.7 / 12.2;
//     heads of 8: 100 contexts 22.4 / 17.0, 45 13.6 / 13.1, 13 11.7 / 12.3
//   up to 64 tokens, block rows: d = 64, heads of 16: 48 contexts 19.4 / 16.7, 100 32.0 / 27.7, 24 12.6 / 13.3, 8 9.4 / 10.2;
//     500 of 32 heads and up to 40 139 / 153; fp32, d = 128: 40 48.2 / 43.8, 100 93 / 89; d = 32: 60 23.9 / 23.2
// Below the lower lines all workgroups run at once; beyond the upper one the end is a small part of the launch, and
// mixed lengths share the memory better (up to 128 tokens the work differs too much for that).
// Short contexts (sorted / in the order of the batch, mean over 8 batches of ~U(1, Lmax); longest context in the columns):
//                                  8..16       20     24     28     32     36     40     48     64
//   d = 128, bf16,  768 units      1.07        0.93   0.93   0.96   0.97   0.96   0.94   0.88   0.95
//                  1280                        1.13   1.14   1.03   1.02   1.04   1.05   1.00   0.99
//                  2048            1.13..1.17  0.98   1.02   1.00   1.00   0.97   0.96   0.97   0.93
//   d = 128, fp16, 1280                        0.97   0.97   0.93   0.95   0.92   0.93   0.87   0.89
//                  1632                        1.10   1.12   1.07   1.04   1.04   0.99   0.96   0.97
//   d = 128, fp32,  800                        1.04   0.98   0.94   0.91   0.92   0.89   0.93   0.87
//                  1280            1.14        1.08   1.06   1.01   1.04   1.03   1.00   0.97   0.94
//                  1632                        1.10   1.04   1.05   1.05   1.01   0.99   0.97   0.95
//   d = 64,  bf16, 1280            1.09        0.95   0.93   0.90   0.91   0.94   0.90   0.91   0.91
//                  2048            1.14        1.02   1.01   1.01   1.00   0.98   0.95   0.95   0.93
//   d = 32,  fp16, 1632                        1.06   1.03   0.97   0.97   1.00   0.98   0.89   0.88
// Up to 16 tokens all contexts are of one class and there is nothing to sort.  Launches of about one round of workgroups
// gain from 20 tokens on, larger ones later.
inline bool longest_first(int blocks, int Lmax, int d, int in_dtype)
{
    const bool fp32 = d == 128 && in_dtype == KVB_F32;
    if (blocks < (d == 128 && !fp32 ? 320 : 512))
        return false;
    if (Lmax > 64)
        return true;
    const bool one_round = blocks <= (d <= 64 || in_dtype == KVB_F16 ? 1280 : 1024);
    const int least = d <= 64 ? (one_round ? 20 : 28) : !one_round ? 40 : fp32 ? 36 : 20;
    return blocks <= 2560 && Lmax >= least;
}
// The leading argument of kvb_direct's kernels: Hv, or with its sign bit set a batch of B (<= MAX_RANKED) requests to be
// sorted in bits 16.., Hv in the rest.
constexpr int MAX_RANKED = 2 * NT;
__host__ __device__ inline int rank_lead(int B, int Hv, bool rank)
{
    return rank && B > 1 && B <= MAX_RANKED && Hv < 65536 ? (int)(0x80000000u | (uint32_t)B << 16 | (uint32_t)Hv) : Hv;
}

struct Store {
    float *state;
    void *buf_k;   // input type
    void *buf_u;   // record type
    float *buf_G;
    int32_t *fill;
    int32_t *status;
    int32_t n_slots;
    // Paged record buffers (Sec. 3.1: blocks of 8 or 16 records from a pool shared by all requests).
    // block_table == nullptr: slot s owns the records s*cap .. s*cap+cap-1 of each head, as one block.
    const int32_t *block_table;   // [n_slots, max_blocks] block ids
    int32_t block_size;           // records per block, a power of two (cap when not paged)
    int32_t max_blocks;           // row length of block_table (1 when not paged)
    int32_t n_blocks;             // blocks in the pools; ids are clamped into 0..n_blocks-1
    int32_t fill_lg;              // the fill of slot s is word s << fill_lg (0, or 5 with KVB_STORE_FILL_APART)
    bool apart() const { return fill_lg != 0; }   // (on the host)
    // (of one workgroup's slot: a word that the request's other workgroups may be adding to)
    __device__ __forceinline__ int32_t *fill_of(int s) const { return fill + ((size_t)s << fill_lg); }
};

// Where record l of the request lives.  The record arrays are [blocks, heads, block_size, ...]:
// a head's records inside a block are contiguous.  Without a block table the block is the slot
// and block_size is cap, which is the contiguous layout.  Each wave keeps its own copy of the
// request's block-table row in LDS (written and read by the same wave, so no barrier), filled
// from one small vector load that is issued before the state loads and therefore never waits
// for them.
constexpr int MAX_BLOCKS = KVB_MAX_BLOCKS;   // cap <= 128, block_size >= 8
// PAGED is a compile-time switch of every kernel: the contiguous layout then costs nothing
// (measured: a run-time flag cost the decode step 2 %; and a dummy load from fill[s] in its
// place doubled the step time, every wave's first load queueing behind the ticket atomics
// that the other heads of the request issue on that word).
template <bool PAGED>
struct Pages {
    const int *tab;   // this wave's LDS copy of the row
    int s, bs, lg;
    __device__ __forceinline__ int blk(int l) const
    {
        if constexpr (PAGED)
            return tab[l >> lg];
        else
            return s;
    }
    __device__ __forceinline__ int off(int l) const { return PAGED ? (l & (bs - 1)) : l; }
    // row of the first record that the block of record l holds of head `head` (H heads per block), in units of one record
    __device__ __forceinline__ size_t block_row(int l, int H, int head) const
    {
        const size_t unit = (size_t)blk(l) * H + head;
        return PAGED ? unit << lg : unit * bs;
    }
    // row of record l
    __device__ __forceinline__ size_t row(int l, int H, int head) const { return block_row(l, H, head) + off(l); }
};
// The records of one head as an array of rows of E elements (a scalar address and 32 bits of offset where the rows of a
// slot are contiguous: with 64-bit arithmetic for each load a wave alone on its SIMD spends a microsecond on addresses).
template <int E, typename T, bool PAGED>
struct Rows {
    using Byte = std::conditional_t<std::is_const_v<T>, const char, char>;
    T *p;   // contiguous: record 0 of the head; paged: the pool
    Pages<PAGED> pg;
    int H, head;
    __device__ __forceinline__ T *at(int l0, int l, int e) const   // of record l0 + l, l0 a scalar
    {
        if constexpr (PAGED)
            return at(l0 + l, e);
        else
            return reinterpret_cast<T *>(reinterpret_cast<Byte *>(p + l0 * E) + (uint32_t)((l * E + e) * (int)sizeof(T)));
    }
    __device__ __forceinline__ T *at(int l, int e) const   // element e of record l
    {
        // (through a byte pointer: through an integer the compiler loses the address space and emits flat accesses)
        // Paged: the block in 64 bits, by a shift, and 32 bits inside it.  Row by row in 64 bits a load took three
        // multiplications and more registers than kernels at the edge of their budget have: kvb_decode with fp32 inputs and
        // a 64-record window spilled values of loads in flight, each a wait for all of them (150 requests of 32 heads, 48
        // records, four steps 343 us, 263 so; 298 before records had this form at all).
        if constexpr (PAGED)
            return reinterpret_cast<T *>(reinterpret_cast<Byte *>(p) + (pg.block_row(l, H, head) * (E * sizeof(T)) +
                                                                        (uint32_t)((pg.off(l) * E + e) * (int)sizeof(T))));
        else
            return reinterpret_cast<T *>(reinterpret_cast<Byte *>(p) + (uint32_t)((l * E + e) * (int)sizeof(T)));
    }
};
template <int E, bool PAGED, typename T>
__device__ __forceinline__ Rows<E, T, PAGED> make_rows(T *pool, const Pages<PAGED> &pg, int H, int head)
{
    return Rows<E, T, PAGED>{PAGED ? pool : pool + ((size_t)pg.s * H + head) * pg.bs * E, pg, H, head};
}
// The lane's entry of the block-table row (lanes >= max_blocks repeat the last entry).
template <bool PAGED>
__device__ __forceinline__ int load_block_id(const Store &st, int s, int lane)
{
    if constexpr (PAGED)
        return st.block_table[(size_t)s * st.max_blocks + min(lane, st.max_blocks - 1)];
    else
        return 0;
}
template <bool PAGED>
__device__ __forceinline__ Pages<PAGED> make_pages(const Store &st, int s, int cap, int *tab, int lane, int id)
{
    Pages<PAGED> pg;
    pg.tab = tab;
    pg.s = s;
    if constexpr (PAGED) {
        if (lane < MAX_BLOCKS)
            tab[lane] = min(max(id, 0), st.n_blocks - 1);
        __builtin_amdgcn_wave_barrier();   // the lookups below stay behind this store (same wave, so no more is needed)
        pg.bs = st.block_size;
        pg.lg = 31 - __builtin_clz(st.block_size);
    } else {
        pg.bs = cap;
        pg.lg = 0;
    }
    return pg;
}

// (r, in the arguments of every kernel: Hv / Hk, the v-heads of a qk-head)
struct StepArgs {
    Store st;
    const int32_t *slot;
    const void *q, *k, *v;
    const float *g, *beta;
    void *out;
    int32_t out_wide;   // fp32 outputs (otherwise the 16-bit input type)
    int32_t Hk, Hv, r, cap, T;
    float scale;
    int32_t advance;    // 1: decode (fill += T after the step); 0: verify (fill untouched)
    int32_t threshold;  // fused decode + flush only: fold the buffer into the state once it holds this many
    int32_t stream_state;  // non-temporal state loads
    // kvb_verify_tree: parent[b][i] in {-1, 0..i-1} of draft i.  When `tree` is 0 the drafts are
    // a chain and `parent` points at some other readable array of at least B*T words (its
    // values are ignored), so that the kernels can load it without a branch.
    const int32_t *parent;
    int32_t tree;
};

struct FlushArgs {
    Store st;
    const int32_t *slot;
    const int32_t *accepted;
    int32_t Hk, Hv, r, cap, threshold;
    int32_t stream;   // non-temporal state loads and stores
};

struct DirectArgs {
    Store st;
    const int32_t *slot;
    const int32_t *len;
    const void *q, *k, *v;
    const float *g, *beta;
    void *out;
    int32_t out_wide;   // fp32 outputs (otherwise the 16-bit input type)
    int32_t Hk, Hv, r, cap, Lmax;
    float scale;
};

struct CompactArgs {
    Store st;
    const int32_t *slot;
    const int32_t *path;
    const int32_t *path_len;
    int32_t Hk, Hv, r, cap, T;
};

// ---------------------------------------------------------------------------
// launch plumbing (host)
// ---------------------------------------------------------------------------
// The timer that the calling thread armed for its next launch, and what its last launch
// returned (kvb_api.hip).
extern thread_local kvb_timer *g_armed;
extern thread_local hipError_t g_launch_status;

// One kernel launch.  If this thread armed a timer, the launch carries its two events so
// that they hold the kernel's own begin / end timestamps.  The runtime's return code is kept
// in g_launch_status (the runtime's "last error" is left alone: it may hold some other
// library's error, which is neither ours to report nor ours to clear).
template <typename... Params, typename... Args>
void launch(void (*kernel)(Params...), int blocks, hipStream_t stream, const Args &...a)
{
    static_assert(sizeof...(Params) == sizeof...(Args), "one argument per kernel parameter");
    std::tuple<std::remove_cv_t<Params>...> params{a...};
    void *argv[sizeof...(Params)];
    std::apply([&](auto &...p) { int i = 0; ((argv[i++] = &p), ...); }, params);
    kvb_timer *t = g_armed;
    g_armed = nullptr;
    if (t)
        g_launch_status = hipExtLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(blocks), dim3(NT), argv, 0,
                                             stream, t->start, t->stop, 0);
    else
        g_launch_status = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(blocks), dim3(NT), argv, 0, stream);
}

// Picks the paged or the contiguous instance of a kernel template whose last parameter is PAGED;
// the arguments after `a` are the kernel's name and its leading template arguments.  They take
// (slot, Hv, dealing of the units) as three plain leading arguments ahead of the argument struct: the build preloads the first
// kernel-argument words into scalar registers at wave launch, so the load of slot[b] -- the head of every dependent
// chain -- goes out at once.
#define LAUNCH_LEAD(blocks, deal, stream, a, ...)                                    \
    do {                                                                             \
        if ((a).st.block_table)                                                      \
            launch(__VA_ARGS__, true>, blocks, stream, (a).slot, (a).Hv, deal, a);   \
        else                                                                         \
            launch(__VA_ARGS__, false>, blocks, stream, (a).slot, (a).Hv, deal, a);  \
    } while (0)

// The compiled (input type, record type) pairs: fp32 records with any input type, 16-bit records
// of the input's own 16-bit type.  Calls f.template operator()<TIn, TRec>().
template <typename F>
int dispatch_types(int in_dtype, int rec_dtype, F &&f)
{
    const bool wide = rec_dtype == KVB_F32;
    if (in_dtype == KVB_F32 && wide)
        f.template operator()<float, float>();
    else if (in_dtype == KVB_BF16 && wide)
        f.template operator()<bf16_t, float>();
    else if (in_dtype == KVB_BF16 && rec_dtype == KVB_BF16)
        f.template operator()<bf16_t, bf16_t>();
    else if (in_dtype == KVB_F16 && wide)
        f.template operator()<f16_t, float>();
    else if (in_dtype == KVB_F16 && rec_dtype == KVB_F16)
        f.template operator()<f16_t, f16_t>();
    else
        return KVB_EUNSUPPORTED;
    return KVB_OK;
}
// The same for the 16-bit input types alone (the matrix-core kernels).
template <typename F>
int dispatch_types16(int in_dtype, int rec_dtype, F &&f)
{
    const bool wide = rec_dtype == KVB_F32;
    if (in_dtype == KVB_BF16 && wide)
        f.template operator()<bf16_t, float>();
    else if (in_dtype == KVB_BF16 && rec_dtype == KVB_BF16)
        f.template operator()<bf16_t, bf16_t>();
    else if (in_dtype == KVB_F16 && wide)
        f.template operator()<f16_t, float>();
    else if (in_dtype == KVB_F16 && rec_dtype == KVB_F16)
        f.template operator()<f16_t, f16_t>();
    else
        return KVB_EUNSUPPORTED;
    return KVB_OK;
}

// Calls f.template operator()<D, TIn, TRec>() for the compiled head sizes and type pairs.
template <typename F>
int dispatch(int dk, int in_dtype, int rec_dtype, F &&f)
{
    if (dk != 32 && dk != 64 && dk != 128)
        return KVB_EUNSUPPORTED;
    return dispatch_types(in_dtype, rec_dtype, [&]<typename TIn, typename TRec>() {
        if (dk == 32)
            f.template operator()<32, TIn, TRec>();
        else if (dk == 64)
            f.template operator()<64, TIn, TRec>();
        else
            f.template operator()<128, TIn, TRec>();
    });
}

// v-heads of a workgroup of kvb_buffer_step_kernel (the measurements stand there); blocks: B * Hv, wide: fp32 inputs,
// apart: a line to each fill word.
inline int buffer_step_heads(int d, bool wide, int Hk, int Hv, int cap, int blocks, bool apart)
{
    if (!apart)
        return Hv > Hk && blocks >= (d == 128 ? 256 : 96) ? 2 : 1;
    const bool one = d == 128 && wide && cap > 64 && Hv <= MAX_FILL_WG;
    return Hv > Hk && blocks >= 320 && !one ? 2 : 1;
}
// Workgroups that add to a request's fill word when a token is appended.
inline int step_workgroups(const StepArgs &a, int d, bool wide, int blocks)
{
    const int hb = a.st.state ? 1 : buffer_step_heads(d, wide, a.Hk, a.Hv, a.cap, blocks, a.st.apart());
    return a.Hk * ((a.r + hb - 1) / hb);
}

// One launcher per translation unit.  They return KVB_EUNSUPPORTED for a head size or type pair
// that is not compiled; none of them checks the launch (the caller does).
template <typename TIn, typename TRec>
int launch_step_typed(int dk, const StepArgs &a, int blocks, hipStream_t stream);   // kvb_step_*.hip, one unit per pair
template <typename TIn, typename TRec>
void launch_verify_typed(int dk, const StepArgs &a, int blocks, hipStream_t stream);   // kvb_verify_*.hip, one unit per input type
int launch_flush(int dk, int in_dtype, int rec_dtype, const FlushArgs &a, int blocks, hipStream_t stream);    // kvb_flush.hip
int launch_compact(int dk, int in_dtype, int rec_dtype, const CompactArgs &a, int blocks, hipStream_t stream);
int launch_direct(int dk, int in_dtype, int rec_dtype, const DirectArgs &a, int blocks, hipStream_t stream);  // kvb_direct.hip

}  // namespace kvb_impl
#endif  // KVB_DEVICE_H
