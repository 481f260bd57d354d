// kvb_flush_rows_kernel and kvb_flush_mfma_kernel (the deferred state update as its own launch), kvb_compact_kernel.
#include "kvb_device.h"

namespace kvb_impl {

// N adjacent elements of which the first lies at a multiple of N (accesses of at most 16 bytes each).
template <int N, typename T>
__device__ __forceinline__ void copy_row(T *dst, const T *src)
{
    constexpr int M = N * sizeof(T) > 16 ? 16 / sizeof(T) : N;
    struct __attribute__((aligned(M * sizeof(T)))) Piece {
        T x[M];
    };
#pragma unroll
    for (int i = 0; i < N; i += M) {
        const Piece p = *reinterpret_cast<const Piece *>(src + i);
        *reinterpret_cast<Piece *>(dst + i) = p;
    }
}

// ---------------------------------------------------------------------------
// kvb_flush: S <- gamma_{m-1} S + sum_{l<m} Gamma_{m-1,l} k_l^T u_l   (Eq. 16, last line)
// for fp32 inputs and for head sizes 32 and 64, on v_mfma_f32_16x16x4_f32 (exact products, fp32 sums).
//
// A call of these sizes moves little, so it is bound by the chain inside a workgroup: the vector-ALU
// kernel that this replaces staged 16 records at a time in LDS and waited for memory once a tile.
// Here nothing is staged and no wave waits for another: the contraction index is the record, lane
// (lq = lane / 16, lm = lane % 16) holds record 4 step + lq of a step, and a chunk of records and the
// state are requested together, the next chunk before this one is multiplied.
// A wave owns RT x CT tiles of 16 x 16: tile row mi of row tile rt is state row RW + RT mi + rt (the
// lane's RT key elements are adjacent), tile column ni of column tile t is column CW + CT ni + t
// (16 lanes read a 128-byte segment of a row at d >= 64).
// 48 requests of 16 heads, d = 64, 1..64 records: 16.9 -> 11.8 us (start of launch to end); 24 of 16 heads, d = 128, fp32, of which
// one in six folds up to 20 records: 11.9 -> 7.8 us.
// ---------------------------------------------------------------------------
template <int D, typename TIn, typename TRec, bool PAGED>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : D == 64 ? 3 : 4)))
void kvb_flush_rows_kernel(const int32_t *slot_arg, int32_t Hv_arg, int32_t deal_arg, const FlushArgs a)
{
    constexpr int RT = D == 128 ? 8 : D == 64 ? 2 : 1;   // 16-row tiles of a wave
    constexpr int CT = D == 32 ? 1 : 2;                  // 16-column tiles of a wave
    constexpr int ST = D == 128 ? 2 : 8;                 // contraction steps (of 4 records) a chunk
    __shared__ int sBlk[NW][MAX_BLOCKS];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int lm = lane % 16, lq = lane / 16;
    const int lb = unit_of(blockIdx.x, deal_arg);
    const int b = quotient(lb, Hv_arg);
    const int32_t slot = slot_arg[b];
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    const int s = with_registers(slot, a.accepted, a.st.fill, a.st.state, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.st.n_slots, a.st.fill_lg, a.Hk, a.Hv, a.r, a.cap,
                                 a.threshold, a.st.status);
    const int h = lb - b * Hv_arg;
    const int hk = quotient(h, a.r);
    const int cap = a.cap;

    if (s < 0 || s >= a.st.n_slots)
        return;
    const int blk_id = load_block_id<PAGED>(a.st, s, lane);
    const int word = *a.st.fill_of(s);
    int nacc = a.accepted ? a.accepted[b] : 0;
    if (nacc < 0)
        nacc = 0;
    const int f = fill_before_commit(word, nacc);
    int m = f + nacc;
    if (m > cap) {
        m = cap;
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
    }
    // (no state: a KV-only context, Sec. 3.4 -- the call then only commits accepted drafts)
    const bool do_flush = a.st.state != nullptr && m >= a.threshold && m > 0;
    if (!do_flush) {
        // (fill only moves when something was accepted)
        if (m != f + nacc)
            publish_fill(a.st.fill_of(s), a.Hv, m);
        else if (nacc > 0)
            advance_fill(a.st.fill_of(s), h == 0, a.Hv, nacc);
        return;
    }
    const size_t unit = (size_t)s * a.Hv + h;
    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, cap, sBlk[wave], lane, blk_id);
    const auto krec = make_rows<D>(static_cast<const TIn *>(a.st.buf_k), pg, a.Hk, hk);
    const auto urec = make_rows<D>(static_cast<const TRec *>(a.st.buf_u), pg, a.Hv, h);
    const auto Grec = make_rows<1>(static_cast<const float *>(a.st.buf_G), pg, a.Hv, h);
    const int RW = D == 128 ? 0 : 16 * RT * (wave / 2);                              // first row of the wave
    const int CW = D == 128 ? 16 * CT * wave : 16 * CT * (wave % 2);                 // and column
    const int row0 = RW + RT * lm, col0 = CW + CT * lm;

    // a chunk as raw bits; an index past m is clamped to record 0 and its value dropped
    struct Chunk {
        TIn k[ST][RT];
        TRec u[ST][CT];
        float G[ST];
    };
    auto load_chunk = [&](int l0, Chunk &x) {
#pragma unroll
        for (int j = 0; j < ST; ++j) {
            const int l = l0 + 4 * j + lq;
            const int lc = l < m ? l : 0;
            copy_row<RT>(x.k[j], krec.at(lc, row0));
            copy_row<CT>(x.u[j], urec.at(lc, col0));
            x.G[j] = *Grec.at(lc, 0);
        }
    };
    const float Glast = *Grec.at(m - 1, 0);
    Chunk cur;
    load_chunk(0, cur);
    // row r + RT 4 lq of the wave's columns: a scalar address and the lane's offset
    float *sp = a.st.state + unit * D * D;
    const uint32_t lane_at = (uint32_t)((RW + RT * 4 * lq) * D + col0) * 4;
    auto state_at = [&](int r) { return reinterpret_cast<float *>(reinterpret_cast<char *>(sp + r * D) + lane_at); };
    float sreg[RT][4][CT];   // the lane's rows RW + RT (4 lq + v) + rt
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            copy_row<CT>(sreg[rt][v], state_at(RT * v + rt));
    __builtin_amdgcn_sched_barrier(0);
    const int ticket = take_ticket(a.st.fill_of(s));

    // the sums, apart from the state, so that nothing waits for it before the end
    f32x4_t acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < CT; ++t)
            acc[rt][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int l0 = 0; l0 < m; l0 += 4 * ST) {
        const Chunk x = cur;
        if (l0 + 4 * ST < m)   // uniform
            load_chunk(l0 + 4 * ST, cur);
#pragma unroll
        for (int j = 0; j < ST; ++j) {
            if (l0 + 4 * j < m) {   // uniform
                const bool in = l0 + 4 * j + lq < m;
                const float w = expf(Glast - x.G[j]);
                float kf[RT], uf[CT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    kf[rt] = to_f32(x.k[j][rt]);
                // slots past m are zero in both factors (0 * Inf is NaN).  They are in the last step; looked for in every
                // step at d = 64, where a branch costs more, and chunk by chunk at d = 32 (against leaving them alone:
                // d = 128 49.2 -> 49.6 us at 64 x 16 fp32 records of 32 heads, every step 50.8; d = 64 112.3 -> 112.5 at
                // 500 x 16, the last step 113.3; d = 32 49.9 -> 50.8 at 500 x 30 fp16 records, 52.4, 52.9)
                if (RT == 2 || l0 + 4 * (RT == 1 ? ST : j + 1) > m) {   // uniform
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        kf[rt] = in ? kf[rt] : 0.0f;
                }
#pragma unroll
                for (int t = 0; t < CT; ++t)
                    uf[t] = in ? w * to_f32(x.u[j][t]) : 0.0f;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int t = 0; t < CT; ++t)
                        acc[rt][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[rt], uf[t], acc[rt][t], 0, 0, 0);
            }
        }
    }
    const float gam = expf(Glast);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float o[CT];
#pragma unroll
            for (int t = 0; t < CT; ++t)
                o[t] = fmaf(gam, sreg[rt][v][t], acc[rt][t][v]);
            if constexpr (CT == 2)
                store2(state_at(RT * v + rt), o[0], o[CT - 1]);
            else
                store1(state_at(RT * v + rt), o[0]);
        }
    if (tid == 0)
        publish_if_last(a.st.fill_of(s), ticket, a.Hv, 0);
}

// ---------------------------------------------------------------------------
// kvb_flush for 16-bit keys and d = 128, on the matrix cores.
//
// The rank-m update is the dense contraction K^T (Diag(Gamma) U), dk x m by m x dv.  The keys
// are bf16 or fp16 as stored, so they are exact operands of v_mfma_f32_16x16x32_{bf16,f16}; the
// other factor x = Gamma_l u_l is fp32 (also when u_l itself is a 16-bit record: the decay
// weight is not) and is cut into pieces of the keys' type, x = x1 + x2 (+ x3), each piece the
// leading bits of what is left, taken off by an exact subtraction, so that k * x = sum k * x_p
// holds to the last piece and the sum is accumulated in fp32 as before.  bf16 pieces carry 8
// significand bits: three of them give all 24 bits of a fp32 record; two (16 bits, 2^-17
// relative) are far below the 2^-9 rounding a bf16 record already carries.  fp16 pieces carry
// 11 bits: two give 22 bits (2^-23 relative, the rounding of fp32 itself is 2^-24); a piece
// below the fp16 range (6e-8) is dropped, an absolute error that small against delta values
// of order one.  A fp32 record may be larger than a fp16 piece can be (65504): a column that holds such a
// value is scaled by a power of two before it is cut, and its sums are scaled back (SCALED; three bf16 pieces
// of the record and two of the key, exact without a scale, cost 92 us instead of 76 for 64 requests of 32
// heads and 128 records, the scale 78).  The 16-bit instruction runs at 16 times the rate of the fp32 matrix
// instruction, so even three products come at about 5 times that rate and 10 times the rate
// of plain vector-ALU FMAs, which is what bounds the vector-ALU kernel above from 16 records on.
//
// Operand layout (lane = 16 lq + lm): A holds A[lm][8 lq + j], B holds B[8 lq + j][lm],
// j = 0..7, the result D[4 lq + v][lm], v = 0..3.  The contraction index is the record,
// 32 records per instruction.  Which state row a tile row stands for, and which column a tile
// column, is free, and chosen so that every global access is a whole row segment:
//   tile row mi of row tile rt    = state row 8 mi + rt: one 16-byte load of k_l[8 lm .. 8 lm + 7]
//                                   holds the lane's element of all 8 row tiles of record l;
//   tile column ni of column tile t = column 32 wave + 2 ni + t: u and the state are accessed
//                                   as float2, 16 lanes to a 128-byte line.
// A lane ends up with rows 32 lq .. 32 lq + 31 of its column pair.  A wave owns 32 columns of
// all rows and needs nothing from the other waves: the kernel has no barrier.
// MULTI: more than one 32-record chunk (cap > 32); the sums then stay in registers across the
// chunks, otherwise each row tile is finished and stored as soon as its six products are done.
// STREAM: the state is read with non-temporal loads AND written back with non-temporal stores,
// for a state too large to be found in the last-level cache at its next use.  Only the two
// together pay: measured at 256 MiB of state and 64 records, 138 us with either or neither,
// 107 us with both (a state that passes through the cache in one direction still turns it
// over); at 128 MiB, which the cache keeps, they cost 10 %.
// PLAIN: a state that is not streamed is stored plainly and stays in the L2 (launch_flush: when), else through it.
// ---------------------------------------------------------------------------
template <typename TIn, typename TRec, bool MULTI, bool STREAM, bool PLAIN, bool PAGED>
// (register budgets: 3 workgroups per CU, 2 where the sums persist)
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(MULTI ? 2 : 3)))
void kvb_flush_mfma_kernel(const int32_t *slot_arg, int32_t Hv_arg, int32_t deal_arg, const FlushArgs a)
{
    // (the three leading arguments are a.slot, a.Hv and the dealing of the units: preloaded into scalar registers
    // at wave launch, so that the load of slot[b] does not wait for the fetch of the argument block)
    constexpr int D = 128;
    constexpr int CH = 32;   // records per chunk
    // pieces of the fp32 factor (see above)
    constexpr int NP = (__is_same(TIn, bf16_t) && sizeof(TRec) == 4) ? 3 : 2;
    // fp16 pieces of fp32 records: out of range is scaled (see above)
    constexpr bool SCALED = __is_same(TIn, f16_t) && sizeof(TRec) == 4;
    __shared__ int sBlk[NW][MAX_BLOCKS];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;   // (a scalar)
    const int lm = lane % 16, lq = lane / 16;
    const int lb = unit_of(blockIdx.x, deal_arg);
    const int b = quotient(lb, Hv_arg);
    const int32_t slot = slot_arg[b];
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    const int s = with_registers(slot, a.accepted, a.st.fill, a.st.state, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.st.n_slots, a.st.fill_lg, a.Hk, a.Hv, a.r, a.cap,
                                 a.threshold, a.st.status);
    const int h = lb - b * Hv_arg;
    const int hk = quotient(h, a.r);
    const int cap = a.cap;

    if (s < 0 || s >= a.st.n_slots)
        return;
    const int word = *a.st.fill_of(s);
    int nacc = a.accepted ? a.accepted[b] : 0;
    if (nacc < 0)
        nacc = 0;
    const int f = fill_before_commit(word, nacc);
    int m = f + nacc;
    if (m > cap) {
        m = cap;
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
    }
    const bool do_flush = a.st.state != nullptr && m >= a.threshold && m > 0;
    if (!do_flush) {
        if (m != f + nacc)
            publish_fill(a.st.fill_of(s), a.Hv, m);
        else if (nacc > 0)
            advance_fill(a.st.fill_of(s), h == 0, a.Hv, nacc);
        return;
    }
    const size_t unit = (size_t)s * a.Hv + h;
    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, cap, sBlk[wave], lane, load_block_id<PAGED>(a.st, s, lane));
    const auto krec = make_rows<D>(static_cast<const TIn *>(a.st.buf_k), pg, a.Hk, hk);
    const auto urec = make_rows<D>(static_cast<const TRec *>(a.st.buf_u), pg, a.Hv, h);
    const auto Grec = make_rows<1>(static_cast<const float *>(a.st.buf_G), pg, a.Hv, h);
    const float Glast = *Grec.at(m - 1, 0);
    const int col2 = 32 * wave + 2 * lm;

    // records 32 c + 8 lq + j of chunk c as raw bits; an index past m is clamped to record 0
    // (finite values that meet a zero weight)
    uint4 kraw[8];
    Raw2<TRec> uraw[8];
    float Graw[8];
    auto load_chunk = [&](int c) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int l = CH * c + 8 * lq + j;
            const int lc = l < m ? l : 0;
            kraw[j] = *reinterpret_cast<const uint4 *>(krec.at(lc, 8 * lm));
            uraw[j] = load_raw2(urec.at(lc, col2));
            Graw[j] = *Grec.at(lc, 0);
        }
    };
    // first chunk, then the state tile: loads retire in issue order, and the products of the
    // first chunk run while the state is in flight
    load_chunk(0);
    __builtin_amdgcn_sched_barrier(0);
    // State row tiles in flight: a window of 4 of the 8, refilled tile by tile as the results are
    // stored (all 8 in flight measured the same and cost a workgroup per CU).
    constexpr int WIN = 4;
    // row r + 32 lq of the wave's columns: a scalar address and the lane's offset
    float *sp = a.st.state + unit * D * D;
    const uint32_t lane_at = (uint32_t)(32 * lq * D + col2) * 4;
    auto state_at = [&](int r) { return reinterpret_cast<float *>(reinterpret_cast<char *>(sp + r * D) + lane_at); };
    float2 sreg[WIN][4];
    auto issue_state = [&](int rt) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            sreg[rt % WIN][v] = load_state2<STREAM>(state_at(8 * v + rt));
        __builtin_amdgcn_sched_barrier(0);   // issue in the order they are consumed
    };
#pragma unroll
    for (int rt = 0; rt < WIN; ++rt)
        issue_state(rt);
    const int ticket = take_ticket(a.st.fill_of(s));

    // B operands of a chunk: piece p of Gamma_l u_l[col2 + t], 8 records to a lane.  down, up: the power of two that
    // column t is cut at and its inverse, the same in the four lanes that hold the column
    uint4 bop[2][NP];
    float down[2] = {1.0f, 1.0f}, up[2] = {1.0f, 1.0f};
    f32x4_t acc[MULTI ? 8 : 1][2];   // the sums, where they persist
#pragma unroll
    for (int rt = 0; rt < (MULTI ? 8 : 1); ++rt)
        acc[rt][0] = acc[rt][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto build_b = [&](int c) {
        float w[8];
        float2 uf[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            w[j] = CH * c + 8 * lq + j < m ? expf(Glast - Graw[j]) : 0.0f;
            uf[j] = unpack2r(uraw[j]);
        }
        if constexpr (SCALED) {
            float big = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                big = largest(big, w[j] * uf[j].x * down[0], w[j] * uf[j].y * down[1]);
            if (__any(big > 65504.0f)) {   // (NaN is none of this)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    float most = 0.0f;
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        most = fmaxf(most, fabsf(w[j] * (t ? uf[j].y : uf[j].x)));
                    most = fmaxf(most, __shfl_xor(most, 16));
                    most = fmaxf(most, __shfl_xor(most, 32));
                    const int e = (int)(__float_as_uint(most) >> 23);   // 2^(e - 127) <= most < 2^(e - 126)
                    if (most * down[t] > 65504.0f && e < 255) {
                        const float to = __uint_as_float((uint32_t)(127 + 127 + 14 - e) << 23);   // most * to < 2^15
                        const float by = to * up[t];
#pragma unroll
                        for (int rt = 0; rt < (MULTI ? 8 : 1); ++rt)
                            acc[rt][t] *= by;
                        down[t] = to;
                        up[t] = __uint_as_float((uint32_t)(127 + e - 127 - 14) << 23);
                    }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float r[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                r[j] = w[j] * (t ? uf[j].y : uf[j].x) * down[t];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                // the leading significand bits of what is left; the rest is exact in fp32
                uint32_t top[8];   // the piece, in the upper half of the word
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if constexpr (__is_same(TIn, bf16_t)) {
                        top[j] = __builtin_bit_cast(uint32_t, r[j]) & 0xFFFF0000u;
                        r[j] -= __builtin_bit_cast(float, top[j]);
                    } else {
                        const f16_t hp = from_f32<f16_t>(r[j]);
                        top[j] = (uint32_t)hp.bits << 16;
                        r[j] -= to_f32(hp);
                    }
                }
                uint4 w4;
                w4.x = (top[0] >> 16) | top[1];
                w4.y = (top[2] >> 16) | top[3];
                w4.z = (top[4] >> 16) | top[5];
                w4.w = (top[6] >> 16) | top[7];
                bop[t][p] = w4;
            }
        }
    };
    // A operand of row tile rt: element rt of each record's 8-element slice
    auto build_a = [&](int rt) {
        uint32_t d[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t w = rt / 2 == 0 ? kraw[j].x : rt / 2 == 1 ? kraw[j].y : rt / 2 == 2 ? kraw[j].z : kraw[j].w;
            d[j] = rt % 2 ? (w >> 16) : (w & 0xFFFFu);
        }
        uint4 w4;
        w4.x = d[0] | (d[1] << 16);
        w4.y = d[2] | (d[3] << 16);
        w4.z = d[4] | (d[5] << 16);
        w4.w = d[6] | (d[7] << 16);
        return w4;
    };
    auto products = [&](int rt, f32x4_t &c0, f32x4_t &c1) {
        const uint4 aop = build_a(rt);
#pragma unroll
        for (int p = NP - 1; p >= 0; --p) {   // smallest pieces first
            c0 = mfma16x32<TIn>(aop, bop[0][p], c0);
            c1 = mfma16x32<TIn>(aop, bop[1][p], c1);
        }
    };
    const float gam = expf(Glast);
    auto finish = [&](int rt, const f32x4_t &c0, const f32x4_t &c1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float2 o;
            o.x = fmaf(gam, sreg[rt % WIN][v].x, c0[v] * up[0]);
            o.y = fmaf(gam, sreg[rt % WIN][v].y, c1[v] * up[1]);
            put<STREAM, PLAIN>(reinterpret_cast<float2 *>(state_at(8 * v + rt)), o);
        }
        if (rt + WIN < 8) {
            __builtin_amdgcn_sched_barrier(0);
            issue_state(rt + WIN);
        }
    };
    if constexpr (!MULTI) {
        build_b(0);
#pragma unroll
        for (int rt = 0; rt < 8; ++rt) {
            f32x4_t c0 = {0.f, 0.f, 0.f, 0.f}, c1 = {0.f, 0.f, 0.f, 0.f};
            products(rt, c0, c1);
            finish(rt, c0, c1);
        }
    } else {
        const int nchunk = (m + CH - 1) / CH;
        for (int c = 0; c < nchunk; ++c) {
            if (c > 0)
                load_chunk(c);
            build_b(c);
#pragma unroll
            for (int rt = 0; rt < 8; ++rt)
                products(rt, acc[rt][0], acc[rt][1]);
        }
#pragma unroll
        for (int rt = 0; rt < 8; ++rt)
            finish(rt, acc[rt][0], acc[rt][1]);
    }
    if (tid == 0)
        publish_if_last(a.st.fill_of(s), ticket, a.Hv, 0);
}

// ---------------------------------------------------------------------------
// kvb_compact: after kvb_verify_tree, the records of the accepted root path
// (nodes path[0] < path[1] < ...) move from positions f + path[j] to f + j, so that
// the accepted drafts are a prefix of the T new records and kvb_flush(accepted)
// commits them (Sec. 3.3, Eq. 8: the state is updated from the accepted tokens
// only).  A few KB a unit: bound by the chain of loads, so every thread carries one 16-byte piece of one record of
// each array, all moves are requested at once, and the stores come behind a barrier (a record may be the source of one
// move and the destination of another).  7 requests of 32 heads, 8 nodes, fp16, verified, compacted and committed: 22.1 us a
// pass move by move, 21.1 at once.
// ---------------------------------------------------------------------------
template <int D, typename TIn, typename TRec, bool PAGED>
__global__ __launch_bounds__(NT) void kvb_compact_kernel(const int32_t *slot_arg, int32_t Hv_arg, const CompactArgs a)
{
    constexpr int PU = D * sizeof(TRec) / 16, PK = D * sizeof(TIn) / 16;   // pieces of a record
    static_assert(KVB_MAX_DRAFTS * PU <= NT && KVB_MAX_DRAFTS * PK <= NT, "a thread to each piece");
    __shared__ int sBlk[NW][MAX_BLOCKS];
    const int tid = threadIdx.x, lane = tid % 64;
    const int b = quotient(blockIdx.x, Hv_arg);
    const int32_t slot = slot_arg[b];
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    const int s = with_registers(slot, a.path, a.path_len, a.st.fill, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.st.n_slots, a.st.fill_lg, a.Hk, a.Hv, a.r, a.cap, a.T,
                                 a.st.status);
    const int h = (int)blockIdx.x - b * Hv_arg;
    const int r = a.r, hk = quotient(h, r);
    if (s < 0 || s >= a.st.n_slots)
        return;
    const int blk_id = load_block_id<PAGED>(a.st, s, lane);
    // node j of the path in lane j, and in the threads of piece row j
    const int32_t *path = a.path + (size_t)b * a.T;
    const int ju = tid / PU, jk = tid / PK;
    const int pj = path[min(lane, a.T - 1)], pu = path[min(ju, a.T - 1)], pk = path[min(jk, a.T - 1)];
    const int n = a.path_len[b];
    const int f = *a.st.fill_of(s) & FILL_MASK;
    const int before = __shfl_up(pj, 1);
    const bool wrong = lane < n && lane < a.T && (pj <= (lane > 0 ? before : -1) || pj >= a.T);
    if (n < 0 || n > a.T || f + a.T > a.cap || __any(wrong)) {   // uniform
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_BADPATH);
        return;
    }
    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, a.cap, sBlk[tid / 64], lane, blk_id);
    const auto krec = make_rows<D>(static_cast<TIn *>(a.st.buf_k), pg, a.Hk, hk);
    const auto urec = make_rows<D>(static_cast<TRec *>(a.st.buf_u), pg, a.Hv, h);
    const auto Grec = make_rows<1>(a.st.buf_G, pg, a.Hv, h);
    const bool mu = ju < n && pu != ju, mk = h == hk * r && jk < n && pk != jk, mG = tid < n && pj != tid;
    const int eu = tid % PU * (16 / (int)sizeof(TRec)), ek = tid % PK * (16 / (int)sizeof(TIn));
    uint4 u = {0, 0, 0, 0}, k = {0, 0, 0, 0};
    float G = 0.0f;
    if (mu)
        u = *reinterpret_cast<const uint4 *>(urec.at(f + pu, eu));
    if (mk)
        k = *reinterpret_cast<const uint4 *>(krec.at(f + pk, ek));
    if (mG)
        G = *Grec.at(f + pj, 0);
    // (the values are here before any thread stores)
    asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w), "+v"(k.x), "+v"(k.y), "+v"(k.z), "+v"(k.w), "+v"(G));
    __syncthreads();
    if (mu)
        put<false>(reinterpret_cast<uint4 *>(urec.at(f + ju, eu)), u);
    if (mk)
        put<false>(reinterpret_cast<uint4 *>(krec.at(f + jk, ek)), k);
    if (mG)
        put<false>(Grec.at(f + tid, 0), G);
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
int launch_flush(int dk, int in_dtype, int rec_dtype, const FlushArgs &a, int blocks, hipStream_t stream)
{
    const int deal = unit_deal(blocks, a.r, fold_deals_from(dk, blocks, a.accepted != nullptr, a.threshold, a.cap, a.st.apart()));
    // Folds of up to 32 records without accepted drafts, of 257 to 512 units: their states (16 to 32 MiB) stay in the L2s for whoever comes next.
    // kvb_direct and fold again and again, through / plain (plain before), us: 25 of 16 heads up to 19 tokens 21.6 / 18.8 (20.5), 9 of 32 up to 12 17.3 / 15.6
    // (17.9), 48 of 9 up to 22 22.3 / 19.8 (20.8).  With more records, more units or accepted drafts through is faster: 23 of 16 up to 39 21.9 / 22.8, 17
    // up to 103 36.3 / 37.3, 109 up to 17 47.7 / 52.9; commits 1 to 5 %.  (A branch in the kernel instead of an instance: 90 of 32 up to 31 92.8 / 96.5.)
    const bool plain = !a.accepted && blocks > 256 && blocks <= 512;
    if (dk == 128 && in_dtype != KVB_F32)   // the matrix-core kernel
        return dispatch_types16(in_dtype, rec_dtype, [&]<typename TIn, typename TRec>() {
            if (a.cap <= 32) {
                if (a.stream)
                    LAUNCH_LEAD(blocks, deal, stream, a, kvb_flush_mfma_kernel<TIn, TRec, false, true, false);
                else if (plain)
                    LAUNCH_LEAD(blocks, deal, stream, a, kvb_flush_mfma_kernel<TIn, TRec, false, false, true);
                else
                    LAUNCH_LEAD(blocks, deal, stream, a, kvb_flush_mfma_kernel<TIn, TRec, false, false, false);
            } else {
                if (a.stream)
                    LAUNCH_LEAD(blocks, deal, stream, a, kvb_flush_mfma_kernel<TIn, TRec, true, true, false);
                else
                    LAUNCH_LEAD(blocks, deal, stream, a, kvb_flush_mfma_kernel<TIn, TRec, true, false, false);
            }
        });
    return dispatch(dk, in_dtype, rec_dtype, [&]<int D, typename TIn, typename TRec>() {
        if constexpr (!(D == 128 && sizeof(TIn) == 2))
            LAUNCH_LEAD(blocks, deal, stream, a, kvb_flush_rows_kernel<D, TIn, TRec);
    });
}

int launch_compact(int dk, int in_dtype, int rec_dtype, const CompactArgs &a, int blocks, hipStream_t stream)
{
    return dispatch(dk, in_dtype, rec_dtype, [&]<int D, typename TIn, typename TRec>() {
        if (a.st.block_table)
            launch(kvb_compact_kernel<D, TIn, TRec, true>, blocks, stream, a.slot, a.Hv, a);
        else
            launch(kvb_compact_kernel<D, TIn, TRec, false>, blocks, stream, a.slot, a.Hv, a);
    });
}

}  // namespace kvb_impl
