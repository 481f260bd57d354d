// kvb_verify_mfma_kernel: kvb_verify / kvb_verify_tree.  Template code
// only; kvb_verify_bf16.hip, kvb_verify_f16.hip and kvb_verify_f32.hip instantiate it for their input type.
#ifndef KVB_VERIFY_KERNEL_H
#define KVB_VERIFY_KERNEL_H

#include "kvb_device.h"

namespace kvb_impl {

// N adjacent columns of a state row or a delta-value row, converted and as raw bits.
template <int N>
struct Cols {
    float x[N];
};
template <bool STREAM, int N>
__device__ __forceinline__ Cols<N> load_cols(const float *p)
{
    if constexpr (N == 2) {
        const float2 t = load_state2<STREAM>(p);
        return Cols<N>{{t.x, t.y}};
    } else {
        return Cols<N>{{*p}};
    }
}
template <typename T, int N>
struct RawCols {
    Raw2<T> w;
};
template <typename T>
struct RawCols<T, 1> {
    T w;
};
template <int N, typename T>
__device__ __forceinline__ RawCols<T, N> load_raw_cols(const T *p)
{
    if constexpr (N == 2)
        return RawCols<T, N>{load_raw2(p)};
    else
        return RawCols<T, N>{*p};
}
template <typename T, int N>
__device__ __forceinline__ Cols<N> unpack_cols(const RawCols<T, N> &r)
{
    if constexpr (N == 2) {
        const float2 t = unpack2r(r.w);
        return Cols<N>{{t.x, t.y}};
    } else {
        return Cols<N>{{to_f32(r.w)}};
    }
}

// 16 bytes of a key or query row as fp32, and a 16 x 16 tile of dot products: a lane holds the same
// pieces of row lm of both factors, so which element a contraction slot stands for is free.
template <typename T, int N>
__device__ __forceinline__ void unpack_piece(const uint4 &w, float (&o)[N])
{
    if constexpr (sizeof(T) == 2) {
        unpack8(Raw8<T>{w}, o);
    } else {
        o[0] = __uint_as_float(w.x); o[1] = __uint_as_float(w.y); o[2] = __uint_as_float(w.z); o[3] = __uint_as_float(w.w);
    }
}
template <typename T, int N>
__device__ __forceinline__ f32x4_t dot_tile(const uint4 (&a)[N], const uint4 (&b)[N])
{
    f32x4_t c = {0.f, 0.f, 0.f, 0.f};
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int st = 0; st < N; ++st)
            c = mfma16x32<T>(a[st], b[st], c);
        return c;
    } else {   // (short chains: see CHAINS below)
#pragma unroll
        for (int s0 = 0; s0 < N; s0 += 4) {
            f32x4_t e[4];
#pragma unroll
            for (int x = 0; x < 4; ++x)
                e[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = s0; st < s0 + 4 && st < N; ++st) {
                e[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[st].x), __uint_as_float(b[st].x), e[0], 0, 0, 0);
                e[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[st].y), __uint_as_float(b[st].y), e[1], 0, 0, 0);
                e[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[st].z), __uint_as_float(b[st].z), e[2], 0, 0, 0);
                e[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[st].w), __uint_as_float(b[st].w), e[3], 0, 0, 0);
            }
            c += (e[0] + e[1]) + (e[2] + e[3]);
        }
        return c;
    }
}

// ---------------------------------------------------------------------------
// kvb_verify on the matrix cores.
//
// With T drafts the step is a pair of small dense contractions (Sec. 3.3, Eq. 7; Eq. 15):
//   stage 1   C1[m][l] = W[m] . k_l        W = [k_0..k_7 ; q_0..q_7] (16 x dk, 16-bit),
//             l over the buffered and the new keys  -> v_mfma_f32_16x16x32_{bf16,f16}; fp32 keys: 16x16x4_f32
//   stage 2   acc[m][:] = sum_rows sW[row][m] S0[row][:] + sum_{l<f} cW[l][m] u_l[:]
//             (16 x (dk + f)) . ((dk + f) x dv), fp32 operands -> v_mfma_f32_16x16x4_f32
// where sW[row][m] = -gamma_i k_i[row] (m = i) or gamma_i q_i[row] (m = 8 + i) and
// cW[l][m] = -/+ Gamma_il C1[m][l].  The cost of stage 2 does not depend on T <= 8.
// Each wave owns D / 4 dv columns (d = 32: two waves own 16) for all rows, so no reduction
// across waves is needed; at d = 128 a lane loads 2 adjacent columns (16 lanes x 8 B = one
// 128-byte line per row).  MFMA layouts: see kvb_direct_mfma_kernel; for 16x16x4 fp32
// lane l supplies A[l%16][l/16] and B[l/16][l%16] and receives C[4*(l/16)+v][l%16].
// fp32 inputs and the head sizes 32 and 64 came here from the vector ALU, where every draft cost its own
// multiply-adds for every state row and record.  Verify and commit, 24 requests of 16 heads, fp32, 5 drafts:
// 31.5 -> 21.1 us; with the commit's own move off the vector ALU, 150 of 16 heads, fp32, 3 drafts: 100 -> 68 us;
// 200 of 32, d = 64, 4 drafts: 92 -> 55 us.
// With a workgroup to a CU, every phase is as long as its instructions: the drafts' decays are worked out a draft to a
// lane (draft after draft in scalar registers took 1.0 us, now 0.23) and record addresses are 32-bit offsets: 7 requests
// of 32 heads, 8 tree drafts, fp16, with compaction and commit, 24.5 -> 23.9 us (every workgroup 8.8 -> 7.8).
// What concerns the drafts alone (their decays, their weights among themselves) is worked out while the state is in flight
// and stays in registers, from where the substitution takes it as scalars; only the weights of the buffered records cross
// waves behind the state.  Against one set of key tiles for records and drafts behind the state, a table of the weights in LDS and
// results by whole rows (112 registers now at d = 128 with 16 records and 134 with 64, were 118 and 161): 200 requests of 32
// heads of 32 34.5 -> 28.9 us, of 64 46.7 -> 45.0; 60 of 64, 64 records, 23.3 -> 22.2; 100 of 32 heads of 128, 96 records, 7
// drafts 85.4 -> 83.5; 24, 16 records, 24.7 -> 24.2; 300 182 -> 182 (memory).
// ---------------------------------------------------------------------------
template <int D, typename TIn, typename TRec, int WREC, bool HAS_STATE, bool STREAM, bool PAGED>
// (register budgets: at least 4 waves per SIMD with a record window of 16 or 32, 3 with the 64-record window or with
// fp32 keys of 128, whose operands take twice the registers; without a state 2, which keeps the sums out of the
// accumulation registers, where settle() could not hold them)
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(!HAS_STATE ? 2 : (WREC <= 32 ? 4 : 3) - (D * sizeof(TIn) > 256))))
void kvb_verify_mfma_kernel(const int32_t *slot_arg, int32_t Hv_arg, int32_t deal_arg, const StepArgs a)
{
    // (the three leading arguments are a.slot, a.Hv and the dealing of the units: preloaded into scalar registers
    // at wave launch, so that the load of slot[b] does not wait for the fetch of the argument block)
    constexpr int CT = D == 128 ? 2 : 1;                      // adjacent columns of a lane
    constexpr int WC = 16 * CT;                               // columns of a wave
    constexpr int NWC = D / WC;                               // waves that own columns (d = 32: the other two repeat them)
    constexpr int EW = 16 / (int)sizeof(TIn);                 // elements of a 16-byte piece of a key row
    constexpr int NWA = D / (4 * EW);                         // pieces of a row that a lane holds (lq 0..3 side by side)
    constexpr int TMX = KVB_MAX_DRAFTS;                       // 8
    constexpr int NTILE = KVB_MAX_CAP / 16;                   // tiles of 16 buffered keys
    static_assert((WREC + 15) / 16 <= NW, "a wave holds one tile of the window's keys");
    constexpr int WQ = WREC / 4;                              // record quads held in registers
    constexpr bool TAIL = WREC >= 64;
    constexpr bool EARLY = HAS_STATE;   // state loads issued before the fill is known
    static_assert(TMX == 8, "row m of W is draft m % 8");

    __shared__ __attribute__((aligned(16))) float sW[D][16];
    __shared__ __attribute__((aligned(16))) float cW[NTILE * 16][16];   // weights of the buffered records
    __shared__ __attribute__((aligned(16))) float fin[16][D];
    __shared__ int sBlk[NW][MAX_BLOCKS];
    // fp32 inputs, whose products are 16 times as long: the weights of the drafts are one wave's work, beside the key tiles
    constexpr bool ONE_WAVE = sizeof(TIn) == 4;
    __shared__ float4 sPair[ONE_WAVE ? 64 : 1];
    // by draft, each wave's own copy: the log decay from the committed context to the draft, its exponential, the ancestors
    __shared__ __attribute__((aligned(16))) float sRel[NW][TMX], sDec[NW][TMX];
    __shared__ __attribute__((aligned(16))) int sAnc[NW][TMX];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;   // (a scalar)
    const int lb = unit_of(blockIdx.x, deal_arg);
    const int b = quotient(lb, Hv_arg);
    const int32_t slot = slot_arg[b];
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    const int s = with_registers(slot, a.q, a.k, a.v, a.g, a.beta, a.parent, a.st.state, a.st.fill, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.st.n_slots, a.st.fill_lg,
                                 a.T);
    const int h = lb - b * Hv_arg;
    const int r = a.r;
    const int hk = quotient(h, r);
    const int T = a.T;
    const int cap = a.cap;

    if (s < 0 || s >= a.st.n_slots)
        return;
    const size_t unit = (size_t)s * a.Hv + h;
    const TIn *qin = static_cast<const TIn *>(a.q);
    const TIn *kin = static_cast<const TIn *>(a.k);
    const TIn *vin = static_cast<const TIn *>(a.v);
    const Out<TIn> out{a.out, a.out_wide != 0};
    const int blk_id = load_block_id<PAGED>(a.st, s, lane);

    const int lm = lane % 16, lq = lane / 16;   // MFMA row/column index and k index of this lane
    const int col2 = WC * (wave % NWC) + CT * lm;

    // ---- 1. loads that need only the request index: raw bits, clamped addresses, no branches
    // row lm of W (draft lm % 8; k for lm < 8, q above), piece lq of each four
    const int wi = min(lm % 8, T - 1);
    const TIn *wrow = (lm < 8 ? kin : qin) + (((size_t)b * T + wi) * a.Hk + hk) * D + EW * lq;
    uint4 wa[NWA];
#pragma unroll
    for (int st = 0; st < NWA; ++st)
        wa[st] = *reinterpret_cast<const uint4 *>(wrow + 4 * EW * st);

    // scalars of draft lane % 8, one vector load each (a scalar load per draft costs a round trip each while the chip
    // is streaming)
    const int di = lane % 8;
    const uint32_t go = (uint32_t)min(di, T - 1) * a.Hv;
    float g_raw = (a.g + (size_t)b * T * a.Hv + h)[go];
    float beta_mine = (a.beta + (size_t)b * T * a.Hv + h)[go];
    int par_raw = a.parent[(size_t)b * T + min(di, T - 1)];

    // ---- 2. the state: rows 4 st + lq, the wave's columns --------------------
    // EARLY: the state's address needs the slot only, so its loads go out before the fill is
    // known and before the long scalar prologue; the records follow and are consumed after the
    // state (the decay gamma_i of row i is then applied to the finished sum over state rows).
    // State row-quads in flight per wave.  EARLY keeps half of the tile in registers and refills a
    // register pair as soon as its quad has gone through the matrix cores: 32 registers less, which
    // is what lets a fourth workgroup onto each CU (the kernel is bound by how well its waves hide
    // each other's waits, not by bytes in flight).
    constexpr int WIN = EARLY && D == 128 ? 16 : D / 4;
    Cols<CT> sreg[WIN];
    const float *sp = a.st.state + (HAS_STATE ? unit * D * D + col2 : 0);
    auto load_quad = [&](int st) { return load_cols<STREAM, CT>(sp + (size_t)(4 * st + lq) * D); };
    auto issue_state = [&]() {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < WIN; ++st) {
            sreg[st] = load_quad(st);
            __builtin_amdgcn_sched_barrier(0);   // issue in the order they are consumed
        }
    };
    if constexpr (EARLY)
        issue_state();

    const int f = *a.st.fill_of(s) & FILL_MASK;
    if (f + T > cap) {
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
        return;
    }
    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, cap, sBlk[wave], lane, blk_id);
    const auto krec = make_rows<D>(static_cast<TIn *>(a.st.buf_k), pg, a.Hk, hk);
    const auto urec = make_rows<D>(static_cast<TRec *>(a.st.buf_u), pg, a.Hv, h);
    const auto Grec = make_rows<1>(a.st.buf_G, pg, a.Hv, h);

    // ---- 3. loads that need the fill ------------------------------------------
    float G_prev = f > 0 ? *Grec.at(f - 1, 0) : 0.0f;
    // this wave's tile of buffered keys: key 16 wave + lm, 16-byte pieces lq
    uint4 kt[NWA];
    float Gn;
    {
        const int n = 16 * wave + lm, nc = n < f ? n : 0;
        const TIn *kp = krec.at(nc, EW * lq);
        Gn = *Grec.at(nc, 0);
#pragma unroll
        for (int st = 0; st < NWA; ++st)
            kt[st] = *reinterpret_cast<const uint4 *>(kp + 4 * EW * st);
    }
    // buffered delta values: quad sq = records 4 sq .. 4 sq + 3, this lane: record 4 sq + lq,
    // columns col2 (d = 128: and the next)
    RawCols<TRec, CT> uq[WQ];
#pragma unroll
    for (int sq = 0; sq < WQ; ++sq) {
        const int l = 4 * sq + lq;
        uq[sq] = load_raw_cols<CT>(static_cast<const TRec *>(urec.at(l < f ? l : 0, col2)));
    }
    __builtin_amdgcn_sched_barrier(0);

    // Drafts form a chain (kvb_verify) or a tree (kvb_verify_tree): the decay of a draft runs along its own root path,
    // and bit j of its mask is set iff draft j is a strict ancestor.  Lane i of every eight works out draft i: the sum
    // over the ancestors in the order of the path (which is that of their indices), the ancestors by following parents
    // packed four bits a draft.  A parent index that does not precede its child is taken as -1 and flagged.
    int anc = (1 << di) - 1;
    asm volatile("" : "+v"(par_raw));   // (its load stays above, out of the branch)
    if (a.tree) {   // uniform
        const bool bad = par_raw < -1 || par_raw >= di;
        const int up = bad ? 0 : par_raw + 1;   // parent + 1
        uint32_t parents = 0;                   // of draft j in bits 4 (j + 1) ..
#pragma unroll
        for (int j = 0; j < TMX - 1; ++j)
            parents |= (uint32_t)__builtin_amdgcn_readlane(up, j) << (4 * (j + 1));
        anc = 0;
        uint32_t at = up;
#pragma unroll
        for (int j = 0; j < TMX - 1; ++j) {
            anc |= (1 << at) >> 1;
            at = parents >> (4 * at) & 15u;
        }
        if (__any(bad && di < T) && tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_BADPATH);
    }
    // Decays are taken from the committed context on (the record before the drafts), whose own decay comes with the records,
    // behind the state: exp(G_i) = exp(G_prev) exp(rel_i), and of record l exp(G_i - G_l) = exp(G_prev - G_l) exp(rel_i), so that
    // all that concerns the drafts alone is ready before the state is.  Whatever a lane needs of other drafts it reads from the
    // wave's table in LDS (an array indexed at run time would live in scratch memory, whose loads share the counter of the
    // state loads).
    float rel = 0.0f;    // of draft lane % 8, the row of W that this lane loaded
    float decRow[4];     // exp(rel) of the draft of accumulator row 4 lq + v: draft v (lq even) or 4 + v (lq odd); 0 past the drafts
    auto draft_decays = [&]() {
        const int path = anc | 1 << di;
#pragma unroll
        for (int j = 0; j < TMX; ++j) {
            const float gj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, g_raw), j));
            rel += path >> j & 1 ? gj : 0.0f;
        }
        if (lane < TMX) {
            sRel[wave][lane] = rel;
            sDec[wave][lane] = lane < T ? expf(rel) : 0.0f;
            sAnc[wave][lane] = anc;
        }
        __builtin_amdgcn_wave_barrier();   // (the same wave reads them)
        const float4 d4 = *reinterpret_cast<const float4 *>(&sDec[wave][4 * (lq % 2)]);
        decRow[0] = d4.x; decRow[1] = d4.y; decRow[2] = d4.z; decRow[3] = d4.w;
    };
    // Weights of the drafts among themselves, in every wave's registers: row m = 4 lq + v of W against key lm of it, seen by the
    // draft's descendants (q rows: and by itself).  Where they are used they are scalars.
    float pair_w[4];
    auto draft_tile = [&]() {
        const f32x4_t c1 = dot_tile<TIn>(wa, wa);
        const float4 r4 = *reinterpret_cast<const float4 *>(&sRel[wave][4 * (lq % 2)]);
        const int4 a4 = *reinterpret_cast<const int4 *>(&sAnc[wave][4 * (lq % 2)]);
        const float relRow[4] = {r4.x, r4.y, r4.z, r4.w};
        const int ancRow[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int m = 4 * lq + v, i = m % 8;
            const bool isq = m >= 8;
            const bool ok = i < T && lm < T && ((ancRow[v] >> lm & 1) || (isq && lm == i));
            const float w = expf(relRow[v] - rel);   // (lane lm < 8: draft lm)
            pair_w[v] = ok ? (isq ? w : -w) * c1[v] : 0.0f;
            asm volatile("" : "+v"(pair_w[v]));
        }
    };
    auto scalar_of = [](float x, int from) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), from));
    };

    // ---- 4. weights of the state rows ------------------------------------------
    // The sums.  One chain of multiply-adds holds a rounding of the whole sum for each of its terms, which for fp32
    // inputs and the small head sizes showed against the vector ALU's row groups; there two chains run for SETTLE
    // contraction steps and are then added to the total (24 requests, fp32, 5 drafts: 1.2e-7 off 64 bits like the
    // vector ALU, one chain 2.2e-7).
    constexpr bool CHAINS = !(D == 128 && sizeof(TIn) == 2);
    constexpr int NACC = CHAINS ? 2 : 1, SETTLE = D == 128 ? 8 : 4;
    f32x4_t acc[CT], part[NACC][CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < NACC; ++n)
            part[n][t] = acc[t];
    }
    auto add = [&](int step, int t, float w, float x) {
        f32x4_t &c = CHAINS ? part[step % NACC][t] : acc[t];
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(w, x, c, 0, 0, 0);
    };
    auto add_chains = [&]() {
        if constexpr (CHAINS) {
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                acc[t] += part[0][t] + part[NACC - 1][t];
                part[0][t] = part[NACC - 1][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    const bool live = lm % 8 < T;
    {
        const float sg = !live ? 0.0f : lm < 8 ? -1.0f : 1.0f;
        // piece st of the rows belongs to wave st % 4 and covers state rows 4 EW st + EW lq ..
#pragma unroll
        for (int g = 0; g < NWA; g += NW) {
            // (component by component: a select between two uint4 objects is compiled as a select
            // between their addresses, which puts them in scratch memory)
            uint4 mine = wa[g];
#pragma unroll
            for (int j = 1; j < NW; ++j) {
                const uint4 other = wa[g + j < NWA ? g + j : g];
                mine.x = wave == j ? other.x : mine.x;
                mine.y = wave == j ? other.y : mine.y;
                mine.z = wave == j ? other.z : mine.z;
                mine.w = wave == j ? other.w : mine.w;
            }
            if (g + wave < NWA) {   // uniform
                float x[EW];
                unpack_piece<TIn>(mine, x);
#pragma unroll
                for (int e = 0; e < EW; ++e)
                    sW[4 * EW * (g + wave) + EW * lq + e][lm] = sg * x[e];
            }
        }
    }
    auto state_rows = [&]() {
#pragma unroll
        for (int st = 0; st < D / 4; ++st) {
            const float aw = sW[4 * st + lq][lm];
            const Cols<CT> sv = sreg[st % WIN];
#pragma unroll
            for (int t = 0; t < CT; ++t)
                add(st, t, aw, sv.x[t]);
            if (st % SETTLE == SETTLE - 1)
                add_chains();
            if (st + WIN < D / 4) {   // the freed registers take the quad WIN further on
                __builtin_amdgcn_sched_barrier(0);
                sreg[st % WIN] = load_quad(st + WIN);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    __syncthreads();   // sW complete
    __builtin_amdgcn_sched_barrier(0);
    draft_decays();
    if constexpr (!ONE_WAVE)
        draft_tile();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (HAS_STATE)
        state_rows();
    // pins the sums, and whatever derives from the loads younger than the state, to this
    // point: pure arithmetic is otherwise free to drift across the fences
    if constexpr (CT == 2)
        asm volatile("" : "+v"(acc[CT - 1]));
    asm volatile("" : "+v"(acc[0]), "+v"(G_prev));
    __builtin_amdgcn_sched_barrier(0);
    // v of this wave's columns (used by its first WC lanes in the last stage)
    const int colf = WC * (wave % NWC) + lane % WC;
    // (the lane's address of draft 0, which the compiler is kept from taking apart, and a scalar 64-bit row: an offset of rows and
    // columns in 32 bits of elements would wrap from 4.8 million heads on, and a scalar address for each row cost 200 requests
    // of 32 heads of 64 35.0 us instead of 34.3 and 34.5.  A draft's step fits 32 bits: the host checks it)
    const uint32_t v_step = (uint32_t)a.Hv * (uint32_t)(D * sizeof(TIn));
    uint64_t v_at = reinterpret_cast<uint64_t>(vin + ((size_t)b * T * a.Hv + h) * D + colf);
    asm volatile("" : "+v"(v_at));
    using VBits = std::conditional_t<sizeof(TIn) == 4, float, uint16_t>;
    TIn v_raw[TMX];
#pragma unroll
    for (int i = 0; i < TMX; ++i) {
        const uint64_t row = (uint64_t)(uint32_t)min(i, T - 1) * v_step;
        v_raw[i] = __builtin_bit_cast(TIn, *reinterpret_cast<const VBits __attribute__((address_space(1))) *>(v_at + row));
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (HAS_STATE) {
        // acc*[v] is row m = 4 lq + v = draft m % 8: apply its gamma
        const float base = expf(G_prev);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[t][v] *= base * decRow[v];
    }

    // ---- 5. stage 1: decayed dot products with every buffered key -------
    auto key_tile = [&](int tile, const uint4(&kk)[NWA], float Gkey) {
        const f32x4_t c1 = dot_tile<TIn>(wa, kk);
        // this lane: rows m = 4 lq + v of W against key n
        const int n = 16 * tile + lm;
        const float w = lq < 2 ? -expf(G_prev - Gkey) : expf(G_prev - Gkey);   // (k rows are negated)
        float o[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            o[v] = n < f ? w * decRow[v] * c1[v] : 0.0f;
        *reinterpret_cast<float4 *>(&cW[n][4 * lq]) = make_float4(o[0], o[1], o[2], o[3]);
    };
    if (16 * wave < f && 16 * wave < WREC)   // uniform
        key_tile(wave, kt, Gn);
    for (int tile = NW + wave; TAIL && 16 * tile < f; tile += NW) {   // keys beyond the register window
        const int n = 16 * tile + lm, nc = n < f ? n : 0;
        const TIn *kp = krec.at(nc, EW * lq);
        uint4 kk[NWA];
#pragma unroll
        for (int st = 0; st < NWA; ++st)
            kk[st] = *reinterpret_cast<const uint4 *>(kp + 4 * EW * st);
        key_tile(tile, kk, *Grec.at(nc, 0));
    }
    if constexpr (ONE_WAVE) {
        if (wave == NW - 1) {   // (whose key tile is the last to fill)
            draft_tile();
            sPair[lane] = make_float4(pair_w[0], pair_w[1], pair_w[2], pair_w[3]);
        }
    }
    __syncthreads();
    if constexpr (ONE_WAVE) {
        const float4 w4 = sPair[lane];
        pair_w[0] = w4.x; pair_w[1] = w4.y; pair_w[2] = w4.z; pair_w[3] = w4.w;
    }

    // ---- 6. stage 2 on the fp32 matrix cores: records (and, if not yet done, state rows)
    const int nquad = (f + 3) / 4;
#pragma unroll
    for (int sq = 0; sq < WQ; ++sq) {
        if (sq < nquad) {   // uniform
            const bool ok = 4 * sq + lq < f;
            const float aw = cW[4 * sq + lq][lm];   // (zero past the records)
            const Cols<CT> uv = unpack_cols(uq[sq]);
#pragma unroll
            for (int t = 0; t < CT; ++t)
                add(sq, t, aw, ok ? uv.x[t] : 0.0f);
            if (sq % SETTLE == SETTLE - 1)
                add_chains();
        }
    }
    // records beyond the register window: four quads to a round trip (requested together, clamped)
    for (int s0 = WQ; TAIL && s0 < nquad; s0 += 4) {
        RawCols<TRec, CT> u4r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = 4 * (s0 + j) + lq;
            u4r[j] = load_raw_cols<CT>(static_cast<const TRec *>(urec.at(l < f ? l : 0, col2)));
        }
        Cols<CT> u4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            u4[j] = unpack_cols(u4r[j]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = 4 * (s0 + j) + lq;
            if (s0 + j < nquad) {   // uniform
                const float aw = cW[l][lm];
#pragma unroll
                for (int t = 0; t < CT; ++t)
                    add(j, t, aw, l < f ? u4[j].x[t] : 0.0f);
            }
        }
    }
    // (the blocks above end the sums, and a branch may skip any of them)
    if constexpr (!CHAINS) {
        settle<SETTLE_FP32>(acc[0], acc[CT - 1]);
    } else {
#pragma unroll
        for (int t = 0; t < CT; ++t)
            settle<SETTLE_FP32>(part[0][t], part[NACC - 1][t]);
        add_chains();
    }
    // acc[t][v] = row m = 4 lq + v, column col2 + t
    if (wave < NWC)   // uniform
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (CT == 2)
                *reinterpret_cast<float2 *>(&fin[4 * lq + v][col2]) = make_float2(acc[0][v], acc[CT - 1][v]);
            else
                fin[4 * lq + v][col2] = acc[0][v];
        }
    __builtin_amdgcn_wave_barrier();   // (a wave finishes its own columns)

    // ---- 5. the T new rows among themselves; results ---------------------------
    // (all loads are consumed before the first store: the memory counter also counts stores,
    // and a wait for a late load inside the loop would wait for the stores of earlier drafts)
    float vf[TMX];
#pragma unroll
    for (int i = 0; i < TMX; ++i) {
        vf[i] = to_f32(v_raw[i]);
        asm volatile("" : "+v"(vf[i]));
    }
    if (lane < WC && wave < NWC) {
        // (every LDS value of the substitution is fetched up front: one round trip for all)
        float fu[TMX], fo[TMX];
#pragma unroll
        for (int i = 0; i < TMX; ++i) {
            fu[i] = fin[i][colf];
            fo[i] = fin[8 + i][colf];
        }
#pragma unroll
        for (int i = 0; i < TMX; ++i)
            asm volatile("" : "+v"(fu[i]), "+v"(fo[i]));
        float uprev[TMX];
#pragma unroll
        for (int i = 0; i < TMX; ++i) {
            if (i < T) {   // uniform
                float acc = vf[i] + fu[i];   // (the weights of k rows are negated)
                float ao = fo[i];
#pragma unroll
                for (int j = 0; j < i; ++j) {
                    acc = fmaf(scalar_of(pair_w[i % 4], 16 * (i / 4) + j), uprev[j], acc);
                    ao = fmaf(scalar_of(pair_w[i % 4], 16 * (2 + i / 4) + j), uprev[j], ao);
                }
                // the record as it will be stored is what every later use reads
                const float ui = rounded_to<TRec>(scalar_of(beta_mine, i) * acc);
                ao = fmaf(scalar_of(pair_w[i % 4], 16 * (2 + i / 4) + i), ui, ao);
                uprev[i] = ui;
                fin[i][colf] = ui;                 // a lane overwrites only what it has read itself
                fin[8 + i][colf] = a.scale * ao;
            }
        }
    }
    // results leave by rows, 16 bytes per lane, T rows of u, then T rows of out: the wave's own columns where its part of a
    // record is a 128-byte line, else whole rows
    constexpr bool WHOLE = sizeof(TRec) == 2 || D < 128;
    constexpr int PR = WHOLE ? D / 4 : WC / 4;   // pieces of a row
    if constexpr (WHOLE)
        __syncthreads();
    else
        __builtin_amdgcn_wave_barrier();
    for (int idx = WHOLE ? tid : lane; idx < 2 * T * PR; idx += WHOLE ? NT : 64) {
        const int rr = idx / PR, col = 4 * (idx % PR) + (WHOLE ? 0 : WC * wave);
        const bool is_u = rr < T;
        const int i = is_u ? rr : rr - T;
        const float4 val = *reinterpret_cast<const float4 *>(&fin[is_u ? i : 8 + i][col]);
        if (is_u)   // (already rounded to the record type: the conversion is exact)
            store4<STREAM>(urec.at(f + i, col), val);
        else
            out.template put4<STREAM>((((size_t)b * T + i) * a.Hv + h) * D + col, val);
    }
    if (tid < T)
        put<STREAM>(Grec.at(f + tid, 0), G_prev + rel);   // (lane = draft)
    if (h % r == 0 && wave == 0 && lm < T) {   // lanes holding k rows store them
        TIn *kw = krec.at(f + lm, EW * lq);
#pragma unroll
        for (int st = 0; st < NWA; ++st)
            put<STREAM>(reinterpret_cast<uint4 *>(kw + 4 * EW * st), wa[st]);
    }
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
template <int D, typename TIn, typename TRec, int WREC>
void launch_verify_w(const StepArgs &a, int blocks, hipStream_t stream)
{
    const int deal = unit_deal(blocks, a.r, deals_from(DEAL_SPEC, a.st.apart()));
    if (!a.st.state) {
        LAUNCH_LEAD(blocks, deal, stream, a, kvb_verify_mfma_kernel<D, TIn, TRec, WREC, false, false);
        return;
    }
    if constexpr (D == 128) {   // (the small head sizes are not tuned: no streaming variant)
        if (a.stream_state) {
            LAUNCH_LEAD(blocks, deal, stream, a, kvb_verify_mfma_kernel<D, TIn, TRec, WREC, true, true);
            return;
        }
    }
    LAUNCH_LEAD(blocks, deal, stream, a, kvb_verify_mfma_kernel<D, TIn, TRec, WREC, true, false);
}

template <int D, typename TIn, typename TRec>
void launch_verify_d(const StepArgs &a, int blocks, hipStream_t stream)
{
    // record window: a request that fits has fill <= cap - T
    if constexpr (D == 128) {
        if (a.cap - a.T <= 16) {
            launch_verify_w<D, TIn, TRec, 16>(a, blocks, stream);
            return;
        }
    }
    if (a.cap - a.T <= 32)
        launch_verify_w<D, TIn, TRec, 32>(a, blocks, stream);
    else
        launch_verify_w<D, TIn, TRec, 64>(a, blocks, stream);
}

template <typename TIn, typename TRec>
void launch_verify_typed(int dk, const StepArgs &a, int blocks, hipStream_t stream)
{
    switch (dk) {   // (checked by the caller)
    case 32:
        launch_verify_d<32, TIn, TRec>(a, blocks, stream);
        break;
    case 64:
        launch_verify_d<64, TIn, TRec>(a, blocks, stream);
        break;
    case 128:
        launch_verify_d<128, TIn, TRec>(a, blocks, stream);
        break;
    }
}

}  // namespace kvb_impl
#endif  // KVB_VERIFY_KERNEL_H
