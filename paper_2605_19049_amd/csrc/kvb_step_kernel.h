// kvb_step_kernel and kvb_buffer_step_kernel: kvb_decode and kvb_decode_flush (and kvb_verify of a single draft), with their launch
// helpers.  Template code only; kvb_step_*.hip instantiate it per (input type, record type), so that they
// compile side by side.
#ifndef KVB_STEP_KERNEL_H
#define KVB_STEP_KERNEL_H

#include "kvb_device.h"

namespace kvb_impl {

// ---------------------------------------------------------------------------
// kvb_decode: row f of the chunkwise form, Eq. 16.  Per (b,h):
//   accU = -gamma k S0 - sum_{l<f} Gamma_l (k.k_l) u_l
//   accO =  gamma q S0 + sum_{l<f} Gamma_l (q.k_l) u_l
// are accumulated over state rows and buffered records alike (both are "rows"
// weighted by a per-row scalar) and reduced across the workgroup.
//
// Load order is the point of this kernel.  The memory counter retires loads
// in issue order, so the few small loads whose values are needed first (the new
// q/k rows, v; with the 64-record window also the buffered records) are issued
// before the 64 KB state tile; the dot products and the LDS exchange then run
// while the state is still in flight.
// ---------------------------------------------------------------------------
// The sum over groups of N adjacent lanes, in every lane: permutations inside a row of 16 lanes ride on the additions,
// where shuffles through LDS are a chain of round trips.  16 steps of kvb_decode_flush: one request 71.6 -> 67.5 us, 13
// of 8 heads, fp16, 97.6 -> 92.4; 4 steps of 500 requests with 64-record buffers 1062 -> 948.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x)
{
    const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true);
    return x + __builtin_bit_cast(float, y);
}
template <int N>
__device__ __forceinline__ float group_sum(float x)
{
    static_assert(N == 4 || N == 8 || N == 16);
    x = dpp_add<0xB1>(x);        // quad_perm 1 0 3 2
    x = dpp_add<0x4E>(x);        // quad_perm 2 3 0 1
    if constexpr (N > 4)
        x = dpp_add<0x141>(x);   // mirrored in 8 lanes: the other four
    if constexpr (N > 8)
        x = dpp_add<0x140>(x);   // mirrored in 16: the other eight
    return x;
}

// x + x of the lane whose index differs in bit OFF, for whole rows of 16 lanes and halves of the wave too.
// (through LDS, as shuffles, 16 steps of one request took 63.5 us instead of 62.6, the pass of kvb_decode without a state
// 437.8 instead of 435.7)
template <int OFF>
__device__ __forceinline__ float add_across(float x)
{
    static_assert(OFF == 8 || OFF == 16 || OFF == 32);
    if constexpr (OFF == 8) {
        return dpp_add<0x128>(x);   // rotated by 8 in its row of 16 lanes
    } else {
        const uint32_t u = __float_as_uint(x);
        const auto both = OFF == 16 ? __builtin_amdgcn_permlane16_swap(u, u, false, false) : __builtin_amdgcn_permlane32_swap(u, u, false, false);
        return __uint_as_float(both[0]) + __uint_as_float(both[1]);
    }
}
// The sum over lanes c4 + LPR i of a wave.
template <int LPR>
__device__ __forceinline__ float column_sum(float x)
{
    if constexpr (LPR <= 8)
        x = add_across<8>(x);
    if constexpr (LPR <= 16)
        x = add_across<16>(x);
    return add_across<32>(x);
}
template <int LPR>
__device__ __forceinline__ float4 column_sum(const float4 &x)
{
    return make_float4(column_sum<LPR>(x.x), column_sum<LPR>(x.y), column_sum<LPR>(x.z), column_sum<LPR>(x.w));
}

//
// FUSE (decode only): when the append brings the buffer to `threshold` records the same
// workgroup applies the deferred update S <- gamma_f S0 + sum_{l<=f} Gamma_fl k_l^T u_l to
// the state tile it already holds in registers and writes it back, which saves the second
// kernel's re-read of the state.
template <int D, typename TIn, typename TRec, int WREC, bool FUSE, bool STREAM, bool PAGED>
// (register budget: the 64-record decode variants sit at the edge of three workgroups per CU; hold them there,
// and those with the matrix-core update, which would spread the state over accumulation registers)
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WREC == 64 || (FUSE && D == 128 && sizeof(TIn) == 2) ? 3 : 1)))
void kvb_step_kernel(const int32_t *slot_arg, int32_t Hv_arg, int32_t deal_arg,
                                                      const StepArgs a)
{
    // The three leading arguments are a.slot, a.Hv and the dealing of the units (unit_deal): as plain leading kernel
    // arguments they are preloaded into scalar registers at wave launch (the build asks for it), so
    // the load of slot[b] -- the head of the dependent chain to the first state byte -- goes out at
    // once instead of after the round trip that fetches the argument block.
    constexpr int LPR = D / 4;       // lanes covering one state row with float4
    constexpr int RPP = NT / LPR;    // rows covered by the workgroup per pass
    constexpr int NPASS = D / RPP;   // state rows per thread
    constexpr int GL = D / 8;        // lanes sharing one key dot product (8 elements each)
    constexpr int NG = NT / GL;      // records handled per pass of the dot-product phase
    constexpr int KP = (WREC + NG - 1) / NG;    // key passes held in registers
    constexpr int UP = (WREC + RPP - 1) / RPP;  // delta-value passes held in registers
    constexpr int NC = KVB_MAX_CAP + 1;
    // the two smaller window tiers are only launched when the whole buffer fits the window
    constexpr bool TAIL = WREC >= 64;
    constexpr int LT = 16;                 // records per LDS tile of the fused state update
    constexpr int EPT = LT * D / NT;
    // the fused state update runs on the matrix cores (see fold_tile)
    constexpr bool MFOLD = FUSE && D == 128 && sizeof(TIn) == 2;
    constexpr int KPC = __is_same(TIn, f16_t) ? 2 : 1;   // bf16 pieces of a key
    constexpr int UPC = 3;                               // bf16 pieces of a weighted delta value
    constexpr int FS = 24;                               // halves per staged row: 16 records + padding (16-byte reads)
    // state loads issued before the fill is known (the 64-record window keeps the records first:
    // holding it across the state pass costs a workgroup per CU)
    constexpr bool EARLY = WREC <= 32;

    __shared__ __attribute__((aligned(16))) float sKs[D];  // -gamma k (state-row weights for accU)
    __shared__ __attribute__((aligned(16))) float sQs[D];  //  gamma q
    __shared__ float cK[NC];     // Gamma_l (k.k_l) of record l
    __shared__ float cQ[NC];     // Gamma_l (q.k_l), and q.k of the token itself at l = f
    __shared__ __attribute__((aligned(16))) float red[NW][2][D];
    __shared__ __attribute__((aligned(16))) float kh[FUSE && !MFOLD ? LT : 1][D];  // Gamma_fl k_l tile
    __shared__ int sBlk[NW][MAX_BLOCKS];
    __shared__ __attribute__((aligned(16))) float uu[FUSE && !MFOLD ? LT : 1][D];  // u_l tile
    __shared__ float wF[MFOLD ? NC : 1];                                           // Gamma_fl
    __shared__ __attribute__((aligned(16))) uint16_t kT[MFOLD ? KPC : 1][MFOLD ? D : 1][FS];  // pieces of k_l, by state row
    __shared__ __attribute__((aligned(16))) uint16_t uT[MFOLD ? UPC : 1][MFOLD ? D : 1][FS];  // of Gamma_fl u_l, by column

    const int tid = threadIdx.x;
    const int lb = unit_of(blockIdx.x, deal_arg);
    const int b = quotient(lb, Hv_arg);
    const int32_t slot = slot_arg[b];
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    const int s = with_registers(slot, a.q, a.k, a.v, a.st.state, a.st.fill, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.g, a.beta, a.st.n_slots, a.st.fill_lg, a.r, a.cap);
    const int h = lb - b * Hv_arg;
    const int r = a.r;
    const int hk = quotient(h, r);
    const int cap = a.cap;
    if (s < 0 || s >= a.st.n_slots)
        return;

    const int rg = tid / LPR, c4 = tid % LPR;
    const int grp = tid / GL, sub = tid % GL;
    const size_t unit = (size_t)s * a.Hv + h;
    const TIn *qin = static_cast<const TIn *>(a.q);
    const TIn *kin = static_cast<const TIn *>(a.k);
    const TIn *vin = static_cast<const TIn *>(a.v);
    const Out<TIn> out{a.out, a.out_wide != 0};
    const int blk_id = load_block_id<PAGED>(a.st, s, tid % 64);

    // ---- 1. loads that need only the request index --------------------------
    // All vector loads of this kernel are issued as raw bits from always-valid addresses (an
    // index past the fill is clamped to record 0 and its value ignored), with no branch and
    // no conversion in between, so nothing waits before the state tile is in flight.
    // the new rows: each thread's 8-element slice of q, k
    const size_t nr_o = ((size_t)b * a.Hk + hk) * D + 8 * sub;
    const Raw8<TIn> q_raw = load_raw8(qin + nr_o);
    const Raw8<TIn> k_raw = load_raw8(kin + nr_o);
    const TIn v_raw = vin[((size_t)b * a.Hv + h) * D + tid % D];

    const int word = *a.st.fill_of(s);
    // ---- 2. the state tile goes in flight ------------------------------------
    // Decoding one token (EARLY): the state's address needs the slot only, so its loads go out
    // before the fill count is known.  Each dependent scalar load costs microseconds while the
    // chip is streaming, and this takes one of them off the path to the first state byte.  The
    // buffered records, whose addresses do need the fill, follow the state and are consumed
    // after it.  The 64-record window keeps them ahead of the state.
    // (scheduling fences: the instruction scheduler must not reorder loads across them; the
    // memory counter retires loads in issue order)
    float4 sreg[NPASS];
    auto issue_state = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        const float4 *sp = reinterpret_cast<const float4 *>(a.st.state + unit * D * D);
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
            sreg[p] = load_state4<STREAM>(sp + (size_t)(rg + RPP * p) * LPR + c4);
            __builtin_amdgcn_sched_barrier(0);   // issue in the order they are consumed
        }
    };
    if constexpr (EARLY)
        issue_state();

    // scalars of the token (uniform); requested together with the fill, after the state loads,
    // so that no scalar wait stands between the slot and the first state byte
    const float gnew = a.g[(size_t)b * a.Hv + h], bet = a.beta[(size_t)b * a.Hv + h];
    // while the fill is on its way: the new rows as weights of the state rows (EARLY applies gamma after the sum over
    // state rows; Gc comes back behind the state)
    float q8[8], k8[8], dqk = 0.0f;
    auto stage_rows = [&](float gw) {
        unpack8(q_raw, q8);
        unpack8(k_raw, k8);
        if (grp == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                sKs[8 * sub + e] = -gw * k8[e];
                sQs[8 * sub + e] = gw * q8[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            dqk = fmaf(q8[e], k8[e], dqk);
        dqk = group_sum<GL>(dqk);
    };
    if constexpr (EARLY) {
        __builtin_amdgcn_sched_barrier(0);
        stage_rows(1.0f);
        __builtin_amdgcn_sched_barrier(0);
    }
    const int f = fill_before(word, a.threshold - 1);
    if (f + 1 > cap) {
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
        return;
    }
    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, cap, sBlk[__builtin_amdgcn_readfirstlane(tid / 64)], tid % 64, blk_id);
    const auto krec = make_rows<D>(static_cast<TIn *>(a.st.buf_k), pg, a.Hk, hk);
    const auto urec = make_rows<D>(static_cast<TRec *>(a.st.buf_u), pg, a.Hv, h);
    const auto Grec = make_rows<1>(a.st.buf_G, pg, a.Hv, h);
    // cumulative log decay of the new row (uniform)
    float Gc;
    float G_prev = f > 0 ? *Grec.at(f - 1, 0) : 0.0f;
    if constexpr (!EARLY)
        Gc = G_prev + gnew;
    // window of buffered records
    Raw8<TIn> kl_raw[KP];
    float Gl[KP];
#pragma unroll
    for (int p = 0; p < KP; ++p) {
        const int l = grp + NG * p;
        const int lc = l < f ? l : 0;
        kl_raw[p] = load_raw8(krec.at(lc, 8 * sub));
        Gl[p] = *Grec.at(lc, 0);
    }
    Raw4<TRec> ur_raw[UP];
#pragma unroll
    for (int j = 0; j < UP; ++j) {
        const int l = rg + RPP * j;
        ur_raw[j] = load_raw4(urec.at(l < f ? l : 0, 4 * c4));
    }
    if constexpr (!EARLY)
        issue_state();
    __builtin_amdgcn_sched_barrier(0);
    // (uniform over the workgroup, and over the request.  A buffer that was due earlier: its fill does not follow from 0)
    const bool fold = FUSE && f + 1 >= a.threshold, overdue = FUSE && f + 1 > a.threshold;
    // youngest memory operation of the wave (EARLY: behind the barrier that it needs anyway, below)
    if (!EARLY && a.advance && !overdue)
        advance_fill(a.st.fill_of(s), h == 0, a.Hv, fold ? -f : 1);

    // ---- 3. decayed dot products of the new rows with every earlier key ----
    float4 accU = make_float4(0.f, 0.f, 0.f, 0.f), accO = make_float4(0.f, 0.f, 0.f, 0.f);
    {
        if constexpr (!EARLY)
            stage_rows(expf(Gc));
        if (tid == 0) {
            cK[f] = 0.0f;
            cQ[f] = dqk;
        }
        if constexpr (EARLY) {
            // the state rows are consumed first, in the order they were issued; the records
            // (younger loads) are not touched before the last state row has been used
            __syncthreads();
            if (a.advance && !overdue)
                advance_fill_read(a.st.fill_of(s), h == 0, a.Hv, fold ? -f : 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < NPASS; ++p) {
                const int row = rg + RPP * p;
                fma4(accU, sKs[row], sreg[p]);
                fma4(accO, sQs[row], sreg[p]);
            }
            // pins the sums (and everything derived from G_prev, a load younger than the
            // state) to this point: pure arithmetic is otherwise free to drift across the fences
            asm volatile("" : "+v"(accU.x), "+v"(accU.y), "+v"(accU.z), "+v"(accU.w),
                              "+v"(accO.x), "+v"(accO.y), "+v"(accO.z), "+v"(accO.w),
                              "+v"(G_prev));
            __builtin_amdgcn_sched_barrier(0);
            Gc = G_prev + gnew;
            const float gam = expf(Gc);
            accU.x *= gam; accU.y *= gam; accU.z *= gam; accU.w *= gam;
            accO.x *= gam; accO.y *= gam; accO.z *= gam; accO.w *= gam;
        }
#pragma unroll
        for (int p = 0; p < KP; ++p) {
            const int l = grp + NG * p;
            float kx[8];
            unpack8(kl_raw[p], kx);
            float dkk = 0.0f, dq = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                dkk = fmaf(kx[e], k8[e], dkk);
                dq = fmaf(kx[e], q8[e], dq);
            }
            dkk = group_sum<GL>(dkk);
            dq = group_sum<GL>(dq);
            if (sub == 0 && l < f) {
                const float w = expf(Gc - Gl[p]);
                cK[l] = w * dkk;
                cQ[l] = w * dq;
                if constexpr (MFOLD)
                    wF[l] = w;
            }
        }
        if constexpr (TAIL) {
            // records beyond the register window: all their passes are requested together (clamped,
            // no branch around the loads), so a long buffer costs one more round trip, not one per pass
            constexpr int KT = (KVB_MAX_CAP - KP * NG + NG - 1) / NG;
            if (f > KP * NG) {   // uniform
                Raw8<TIn> kt_raw[KT];
                float Gt[KT];
#pragma unroll
                for (int x = 0; x < KT; ++x) {
                    const int l = (KP + x) * NG + grp;
                    const int lc = l < f ? l : 0;
                    kt_raw[x] = load_raw8(krec.at(lc, 8 * sub));
                    Gt[x] = *Grec.at(lc, 0);
                }
#pragma unroll
                for (int x = 0; x < KT; ++x) {
                    const int l = (KP + x) * NG + grp;
                    if ((KP + x) * NG < f) {   // uniform
                        float kx[8];
                        unpack8(kt_raw[x], kx);
                        float dkk = 0.0f, dq = 0.0f;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            dkk = fmaf(kx[e], k8[e], dkk);
                            dq = fmaf(kx[e], q8[e], dq);
                        }
                        dkk = group_sum<GL>(dkk);
                        dq = group_sum<GL>(dq);
                        if (sub == 0 && l < f) {
                            const float w = expf(Gc - Gt[x]);
                            cK[l] = w * dkk;
                            cQ[l] = w * dq;
                            if constexpr (MFOLD)
                                wF[l] = w;
                        }
                    }
                }
            }
        }
    }
    __syncthreads();

    // ---- 4. accumulate over buffered records and state rows ----------------
    float4 ur[UP];
#pragma unroll
    for (int j = 0; j < UP; ++j) {
        const int l = rg + RPP * j;
        ur[j] = unpack4(ur_raw[j]);
        if (l < f) {
            fma4(accU, -cK[l], ur[j]);
            fma4(accO, cQ[l], ur[j]);
        }
    }
    if constexpr (TAIL) {
        // delta values beyond the register window, four passes to a round trip
        constexpr int UT = (KVB_MAX_CAP - UP * RPP + RPP - 1) / RPP;
#pragma unroll
        for (int x0 = 0; x0 < UT; x0 += 4) {
            if ((UP + x0) * RPP < f) {   // uniform
                Raw4<TRec> ut_raw[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int l = (UP + x0 + j) * RPP + rg;
                    ut_raw[j] = load_raw4(urec.at(l < f ? l : 0, 4 * c4));
                }
                float4 ut[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    ut[j] = unpack4(ut_raw[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int l = (UP + x0 + j) * RPP + rg;
                    if (x0 + j < UT && l < f) {
                        fma4(accU, -cK[l], ut[j]);
                        fma4(accO, cQ[l], ut[j]);
                    }
                }
            }
        }
    }
    if constexpr (!EARLY) {
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
            const int row = rg + RPP * p;
            fma4(accU, sKs[row], sreg[p]);
            fma4(accO, sQs[row], sreg[p]);
        }
    }

    // ---- 5. reduce over the row groups: lane permutations inside the wave, LDS across waves
    accU = column_sum<LPR>(accU);
    accO = column_sum<LPR>(accO);
    {
        const int wave = tid / 64, lane = tid % 64;
        if (lane < LPR) {
            *reinterpret_cast<float4 *>(&red[wave][0][4 * lane]) = accU;
            *reinterpret_cast<float4 *>(&red[wave][1][4 * lane]) = accO;
        }
    }
    __syncthreads();

    // ---- 6. finish the new row, write results --------------------------------
    float u_new = 0.0f;
    auto write_row = [&](auto plain) __attribute__((always_inline)) {
        constexpr bool PLAIN = decltype(plain)::value;
        if (tid < D) {
            float au = 0.0f, ao = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                au += red[w][0][tid];
                ao += red[w][1][tid];
            }
            // the record as it is stored is what every later use reads, this token's output included
            const TRec ur_new = from_f32<TRec>(bet * (to_f32(v_raw) + au));
            u_new = to_f32(ur_new);
            ao = fmaf(cQ[f], u_new, ao);
            out.template put1<STREAM, PLAIN>(((size_t)b * a.Hv + h) * D + tid, a.scale * ao);
            put<STREAM, PLAIN>(urec.at(f, tid), ur_new);
        }
        if (tid == 0)
            put<STREAM, PLAIN>(Grec.at(f, 0), Gc);
        if (h == hk * r && tid < D / 8)   // the threads that loaded the new k row store it
            store_raw8<STREAM, PLAIN>(krec.at(f, 8 * sub), k_raw);
    };
    // Where at least every fourth step folds (threshold up to 4; 1 is recurrent decoding), what a step leaves is read back by the
    // next few, mostly on the same XCD, and stays in its L2; with fewer folds it goes through to memory.  us a step, plain /
    // through, with a plain state: threshold 1, 128 requests of 32 heads 81.9 / 86.6, one 5.14 / 5.35; threshold 2, 128
    // requests 59.8 / 60.9.  By the workgroup's own fold instead of the threshold: 83.0 at threshold 1, and 16 steps of 13
    // requests of 8 heads with 32 fp16 records 78.8 instead of 78.0.
    // Also where buffers grow past the 64 records that are loaded ahead: the rest is read late, from the L2 sooner.  Threshold 128, through / plain:
    // 4 requests of 8 heads, 8 steps 53.8 / 52.2, 11 of 16 heads of 32 39.4 / 37.1, 4 of 9 heads of 64, 16 steps 82.9 / 81.0; 64 of 32
    // 575 / 576, 333 of 9 894 / 892.
    if constexpr (FUSE && !STREAM) {
        if (a.threshold <= 4 || a.threshold > 64)
            write_row(std::true_type{});
        else
            write_row(std::false_type{});
    } else {
        write_row(std::false_type{});
    }
    const int m = f + 1;
    if (overdue)
        publish_fill(a.st.fill_of(s), a.Hv, 0);
    if constexpr (FUSE) {
        if (fold) {
            const float gam = expf(Gc);
            if constexpr (MFOLD) {
                // The rank-m update on the matrix cores, 16 records a step.  A thread holds rows
                // rg + 8 p (p = 0..15, rg = 2 wave + lane / 32) of columns 4 c4 + e: for each e that is
                // the accumulator of a 32 x 32 tile, its column index c4 = lane % 32 and its row index
                // 8 (p / 4) + 4 (lane / 32) + p % 4, so the state is updated where it already lies and
                // nothing crosses waves but the two staged factors.  The factors are exact: Gamma u is cut
                // into three bf16 pieces (24 bits), a key is one bf16 value or, from fp16, two (11 bits;
                // bf16 also has the exponent range that a large delta value needs), products are summed in
                // fp32.  The vector ALU took 4096 cycles a wave for 16 records, the chain that ended every launch
                // in which some request folds.  13 requests of 8 heads, C = 32, fp16, 16 steps: 120 -> 99 us;
                // 64 of 32 heads, C = 16, bf16: 483 -> 475 us; 1 of 32: 76.1 -> 74.9 us.  (500 of 32 at C = 64:
                // the same 1072 us, its launches wait for memory.)
                // (With fp16 records two fp16 pieces of Gamma u and a key as it is, two products instead of six, took 78.6 us for the
                // first of these instead of 85.6, but what lies below 6e-8 is lost: of values of 1e-4 half the bits.  Scaling the
                // columns first takes the maximum over all waves and 64 products a lane, as much as it saves.)
                // Pieces of an infinity are NaN: a wave whose result is not finite folds again on the vector ALU.
                // The records of a tile go to contraction slots 2 (r % 8) + r / 8, so that the two a thread
                // stages share a word.
                f32x16_t acc[4];
#pragma unroll
                for (int p = 0; p < NPASS; ++p) {
                    acc[0][p] = gam * sreg[p].x;
                    acc[1][p] = gam * sreg[p].y;
                    acc[2][p] = gam * sreg[p].z;
                    acc[3][p] = gam * sreg[p].w;
                }
                if (tid < D)
                    sKs[tid] = u_new;   // (the state rows were weighted long ago)
                const int lane = tid % 64, wv = tid / 64;
                // kx: elements 8 sub .. + 7 of key l0 + grp; u0, u1: columns 4 c4 .. + 3 of records l0 + rg, + 8
                auto fold_tile = [&](int l0, const Raw8<TIn> &kx, const float4 &u0, const float4 &u1) {
                    __syncthreads();
                    {
                        const int l = l0 + grp, at = 2 * (grp % 8) + grp / 8;
                        float kf[8];
                        unpack8(kx, kf);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float x = l < f ? kf[e] : l == f ? k8[e] : 0.0f;
                            const int row = 32 * (e / 2) + 8 * (sub / 4) + 4 * (e % 2) + sub % 4;
                            const uint32_t top = __float_as_uint(x) & 0xFFFF0000u;
                            kT[0][row][at] = (uint16_t)(top >> 16);
                            if constexpr (KPC == 2)
                                kT[KPC - 1][row][at] = (uint16_t)(__float_as_uint(x - __uint_as_float(top)) >> 16);
                        }
                        const float *un = &sKs[4 * c4];
                        const int la = l0 + rg, lb8 = la + 8;
                        const float wa = la < f ? wF[la] : 0.0f, wb = lb8 < f ? wF[lb8] : 0.0f;
                        const float xa[4] = {u0.x, u0.y, u0.z, u0.w}, xb[4] = {u1.x, u1.y, u1.z, u1.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float nw = un[e];
                            float ra = la < f ? wa * xa[e] : la == f ? nw : 0.0f;
                            float rb = lb8 < f ? wb * xb[e] : lb8 == f ? nw : 0.0f;
#pragma unroll
                            for (int q = 0; q < UPC; ++q) {   // the leading 8 bits of what is left; the rest is exact
                                const uint32_t ta = __float_as_uint(ra) & 0xFFFF0000u, tb = __float_as_uint(rb) & 0xFFFF0000u;
                                *reinterpret_cast<uint32_t *>(&uT[q][32 * e + c4][2 * rg]) = (ta >> 16) | tb;
                                ra -= __uint_as_float(ta);
                                rb -= __uint_as_float(tb);
                            }
                        }
                    }
                    __syncthreads();
                    bf16x8_t ka[KPC];
#pragma unroll
                    for (int x = 0; x < KPC; ++x)
                        ka[x] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(&kT[x][32 * wv + lane % 32][8 * (lane / 32)]));
#pragma unroll
                    for (int q = UPC - 1; q >= 0; --q)   // smallest pieces first
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const bf16x8_t ub8 = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(&uT[q][32 * e + lane % 32][8 * (lane / 32)]));
#pragma unroll
                            for (int x = KPC - 1; x >= 0; --x)
                                acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[x], ub8, acc[e], 0, 0, 0);
                        }
                };
                if constexpr (WREC <= 32) {   // the whole buffer is in registers: a key pass is one tile, two passes of u fill it
#pragma unroll
                    for (int p = 0; p < KP; ++p)
                        if (LT * p < m)   // uniform
                            fold_tile(LT * p, kl_raw[p], ur[2 * p], ur[2 * p + 1]);
                } else {
                    // (holding the 64-record window this long costs a workgroup per CU: its records come back
                    // from memory, the next tile requested before this one is applied.  Requests are clamped;
                    // rows >= f are not used)
                    const int lmax = f > 0 ? f - 1 : 0;
                    Raw8<TIn> kq;
                    Raw4<TRec> ua, ub4;
                    auto request = [&](int l0) {
                        kq = load_raw8(krec.at(min(l0 + grp, lmax), 8 * sub));
                        ua = load_raw4(urec.at(min(l0 + rg, lmax), 4 * c4));
                        ub4 = load_raw4(urec.at(min(l0 + rg + 8, lmax), 4 * c4));
                    };
                    request(0);
                    for (int l0 = 0; l0 < m; l0 += LT) {
                        const Raw8<TIn> kc = kq;
                        const float4 u0 = unpack4(ua), u1 = unpack4(ub4);
                        request(l0 + LT);   // (past the last tile: a valid record, dropped)
                        fold_tile(l0, kc, u0, u1);
                    }
                }
                float big = 0.0f;
#pragma unroll
                for (int p = 0; p < NPASS; ++p) {
                    big = largest(largest(big, acc[0][p], acc[1][p]), acc[2][p], acc[3][p]);
                    sreg[p] = make_float4(acc[0][p], acc[1][p], acc[2][p], acc[3][p]);
                }
                if (__builtin_expect(!all_finite(big), 0)) {   // (the state, the records and the new token as the formula has them)
                    // (everything from an opaque thread index: nothing is kept in a register for this)
                    int t = tid;
                    asm volatile("" : "+v"(t));
                    const int row0 = t / LPR, col0 = t % LPR * 4;
                    Pages<PAGED> pq = pg;
                    pq.tab = sBlk[t / 64];
                    const float gs = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, gam)));
                    const float *sp = a.st.state + unit * D * D + (size_t)row0 * D + col0;
#pragma unroll
                    for (int p = 0; p < NPASS; ++p) {
                        sreg[p] = *reinterpret_cast<const float4 *>(sp + (size_t)RPP * p * D);
                        sreg[p].x *= gs; sreg[p].y *= gs; sreg[p].z *= gs; sreg[p].w *= gs;
                    }
#pragma unroll 1
                    for (int l = 0; l < m; ++l) {
                        const TIn *kp = (l < f ? static_cast<const TIn *>(a.st.buf_k) + pq.row(l, a.Hk, hk) * D : kin + ((size_t)b * a.Hk + hk) * D) + row0;
                        float4 u = *reinterpret_cast<const float4 *>(&sKs[col0]);
                        float w = 1.0f;
                        if (l < f) {   // uniform
                            u = unpack4(load_raw4(static_cast<const TRec *>(a.st.buf_u) + pq.row(l, a.Hv, h) * D + col0));
                            w = wF[l];
                        }
#pragma unroll
                        for (int p = 0; p < NPASS; ++p)
                            fma4(sreg[p], w * to_f32(kp[RPP * p]), u);
                    }
                }
            } else {
#pragma unroll
                for (int p = 0; p < NPASS; ++p) {
                    sreg[p].x *= gam; sreg[p].y *= gam; sreg[p].z *= gam; sreg[p].w *= gam;
                }
                // one LDS tile of LT records: record f itself comes from this workgroup's registers
                auto inject_new = [&](int l0) {
                    if (f >= l0 && f < l0 + LT) {
                        if (grp == 0) {
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                kh[f - l0][8 * sub + e] = k8[e];
                        }
                        if (tid < D)
                            uu[f - l0][tid] = u_new;
                    }
                };
                auto apply_tile = [&](int l0) {
                    const int nl = min(LT, m - l0);
                    for (int l = 0; l < nl; ++l) {
                        const float4 u = *reinterpret_cast<const float4 *>(&uu[l][4 * c4]);
#pragma unroll
                        for (int p = 0; p < NPASS; ++p)
                            fma4(sreg[p], kh[l][rg + RPP * p], u);
                    }
                };
                int l_done = 0;
                if constexpr (NG == LT && 2 * RPP == LT && WREC <= 32) {
                    // d = 128: a window pass of keys is exactly one tile, two passes of delta values
                    // fill it, so the tiles inside the register window need no second trip to memory
                    // (not for the 64-record window: keeping it alive this long costs a workgroup per CU)
#pragma unroll
                    for (int p = 0; p < KP; ++p) {
                        if (LT * p < m) {   // uniform
                            __syncthreads();
                            const int l = LT * p + grp;
                            float kx[8];
                            unpack8(kl_raw[p], kx);
                            const float w = l < f ? expf(Gc - Gl[p]) : 0.0f;
                            if (l != f) {   // row f of the tile belongs to inject_new
#pragma unroll
                                for (int e = 0; e < 8; ++e)
                                    kh[grp][8 * sub + e] = l < f ? w * kx[e] : 0.0f;
                            }
#pragma unroll
                            for (int jj = 0; jj < 2; ++jj) {
                                const int lu = LT * p + RPP * jj + rg;
                                const float4 u = ur[2 * p + jj];
                                if (lu != f)
                                    *reinterpret_cast<float4 *>(&uu[RPP * jj + rg][4 * c4]) =
                                        lu < f ? u : make_float4(0.f, 0.f, 0.f, 0.f);
                            }
                            inject_new(LT * p);
                            __syncthreads();
                            apply_tile(LT * p);
                        }
                    }
                    l_done = LT * KP;
                }
                if constexpr (NG == LT) {
                  if (l_done < m) {   // uniform
                    // records before f come back from memory (written by earlier calls): thread (grp, sub)
                    // brings 8 elements of record l0 + grp, and the next tile is requested before this
                    // one is applied, so its round trip hides under the multiply-adds
                    const int lmax = f > 0 ? f - 1 : 0;   // requests are clamped; rows >= f are not used
                    int lr = min(l_done + grp, lmax);
                    Raw8<TIn> kq = load_raw8(krec.at(lr, 8 * sub));
                    Raw8<TRec> uq = load_raw8(urec.at(lr, 8 * sub));
                    float Gq = *Grec.at(lr, 0);
                    for (int l0 = l_done; l0 < m; l0 += LT) {
                        __syncthreads();
                        const int l = l0 + grp;
                        if (l != f) {   // row f of the tile belongs to inject_new
                            float kx[8];
                            unpack8(kq, kx);
                            const float w = l < f ? expf(Gc - Gq) : 0.0f;
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                kh[grp][8 * sub + e] = l < f ? w * kx[e] : 0.0f;
                            // (component by component: a select between two float4 objects is compiled
                            // as a select between their addresses, which puts them in scratch memory)
                            const bool in = l < f;
                            float ux[8];
                            unpack8(uq, ux);
                            *reinterpret_cast<float4 *>(&uu[grp][8 * sub]) = make_float4(
                                in ? ux[0] : 0.0f, in ? ux[1] : 0.0f, in ? ux[2] : 0.0f, in ? ux[3] : 0.0f);
                            *reinterpret_cast<float4 *>(&uu[grp][8 * sub + 4]) = make_float4(
                                in ? ux[4] : 0.0f, in ? ux[5] : 0.0f, in ? ux[6] : 0.0f, in ? ux[7] : 0.0f);
                        }
                        inject_new(l0);
                        // (the request past the last tile re-reads a valid record and is dropped)
                        lr = min(l0 + LT + grp, lmax);
                        kq = load_raw8(krec.at(lr, 8 * sub));
                        uq = load_raw8(urec.at(lr, 8 * sub));
                        Gq = *Grec.at(lr, 0);
                        __syncthreads();
                        apply_tile(l0);
                    }
                  }
                } else {
                    for (int l0 = l_done; l0 < m; l0 += LT) {
                        __syncthreads();
                        // records before f come back from memory (written by earlier calls)
#pragma unroll
                        for (int x = 0; x < EPT; ++x) {
                            const int idx = tid + NT * x, l = l0 + idx / D, e = idx % D;
                            if (l < f) {
                                kh[idx / D][e] = expf(Gc - *Grec.at(l, 0)) * to_f32(*krec.at(l, e));
                                uu[idx / D][e] = to_f32(*urec.at(l, e));
                            } else if (l > f) {
                                kh[idx / D][e] = 0.0f;
                                uu[idx / D][e] = 0.0f;
                            }
                        }
                        inject_new(l0);
                        __syncthreads();
                        apply_tile(l0);
                    }
                }
            }
            float *sw = a.st.state + unit * D * D;
            const uint32_t lane_at = (uint32_t)(rg * LPR + c4) * 16;
#pragma unroll
            for (int p = 0; p < NPASS; ++p)   // (a state that is streamed in is streamed out again: +1 % on 1 GiB of state;
                                              // otherwise it stays in the L2: threshold 1, through / plain, us a step: 16
                                              // requests 11.8 / 10.1, one 5.73 / 5.29; 64, with the rest through, 40.7 / 41.4)
                put_at<STREAM>(sw + RPP * p * D, lane_at, sreg[p]);
        }
    }
}

// ---------------------------------------------------------------------------
// kvb_decode without a state (Sec. 3.4, Eq. 14): the buffer is all there is to read, so a workgroup of a single
// v-head moves a few KB and lives on its chain of loads (slot, fill, records) and exchanges.  HB v-heads of a key
// head share a workgroup: the keys are read and multiplied once for them, and their chains run side by side.
// The records go in blocks of 64: keys, decays and delta values of a block are requested together, one round
// trip for each block that the fill reaches.  With 16-bit inputs the dot products of 16 records with the new key and
// query are one product on the matrix cores per 32 dimensions, rows k and q of which every lane group holds, so that a
// lane ends up with both of its record for the head whose weights it makes.  128 contexts of up to 100 tokens, 32 heads,
// fp16, 16 steps: 476 us with the dots on the vector ALU, sums by shuffles through LDS and 64-bit record addresses, 447
// without the three.
// Rule (buffer_step_heads): two heads a workgroup from as many units on as leave the CUs busy; below, the halves of
// the chip that would stay idle are worth more.  What two heads save are the keys and half of the workgroups.
// Passes beyond the fill load a valid record and compute nothing.
// One head a workgroup / two, a line to each fill word, us a call, each request at its own fill, 0..60 records unless said:
//   requests of 32 heads       2            4            8            16           32           64            128           16, 0..10    128, 0..10    32, 0..119    128, 0..119
//   units                      64           128          256          512          1024         2048          4096          512          4096          1024          4096
//   d = 128, bf16 / fp32       4.6 / 5.2    4.9 / 5.6    5.1 / 5.8    5.9 / 5.9    7.9 / 7.1    11.9 / 11.6   19.3 / 18.4   5.0 / 4.8    15.1 / 12.1   10.1 / 10.8   27.6 / 28.6
//   d = 128, fp16 / fp16       4.5 / 5.0    4.9 / 5.4    5.0 / 5.6    5.8 / 5.7    7.8 / 6.7    11.5 /  8.9   18.5 / 14.7   5.0 / 4.7    15.0 / 11.2    9.5 /  8.3   24.2 / 20.7
//   d = 128, fp32              4.7 / 5.3    5.0 / 5.7    5.3 / 6.1    6.0 / 6.2    7.8 / 8.4    12.7 / 13.3   20.7 / 21.4   4.9 / 4.8    14.5 / 12.3   10.8 / 12.1   32.2 / 34.2
//   d = 64,  bf16 / fp32       4.2 / 4.6    4.2 / 4.6    4.4 / 4.8    5.0 / 4.8    6.0 / 5.5     8.1 /  7.0   12.3 / 11.8   4.6 / 4.3    10.5 /  9.0    7.3 /  6.5   17.5 / 17.8
//   d = 64,  fp32              4.1 / 4.6    4.2 / 4.6    4.3 / 4.8    4.9 / 4.8    5.9 / 5.7     8.0 /  7.4   13.1 / 13.1   4.6 / 4.3    10.6 /  9.1    7.4 /  8.2   19.4 / 20.2
//   d = 32,  fp16 / fp16       4.2 / 4.4    4.1 / 4.4    4.2 / 4.5    4.7 / 4.6    5.4 / 5.0     6.6 /  6.1    9.2 /  7.8   4.5 / 4.3     8.8 /  7.3    5.9 /  5.6   10.9 /  9.7
//   d = 32,  fp32              4.1 / 4.3    4.1 / 4.3    4.1 / 4.3    4.7 / 4.5    5.4 / 5.1     6.8 /  6.4    9.5 /  8.5   4.4 / 4.2     8.9 /  7.8    6.0 /  5.6   12.8 / 12.8
// Three v-heads to a key head, where the second workgroup of a key head has one of them, and heads of 8:
//   requests                   16 of 9      45 of 9      120 of 9     240 of 9      13 of 8      30 of 8      100 of 8
//   units                      144          405          1080         2160          104          240          800
//   d = 128, bf16 / fp32       5.2 / 5.8    6.3 / 6.6    8.7 / 8.3    12.4 / 12.8   4.8 / 5.5    5.1 / 5.8    7.4 / 7.0
//   d = 128, fp16 / fp16       5.1 / 5.6    6.2 / 6.2    8.5 / 8.0    12.0 / 11.5   4.8 / 5.3    5.1 / 5.6    7.4 / 6.7
//   d = 128, fp32              5.3 / 6.0    6.2 / 6.6    8.1 / 8.5    12.4 / 13.6   4.9 / 5.7    5.3 / 6.1    7.1 / 7.4
//   d = 64,  bf16 / fp32       4.4 / 4.7    5.3 / 5.4    6.4 / 6.3     8.4 /  8.8   4.4 / 4.8    4.6 / 5.0    5.7 / 5.5
//   d = 32,  fp16 / fp16       4.2 / 4.5    4.9 / 5.0    5.5 / 5.6     7.1 /  7.0   4.1 / 4.5    4.2 / 4.5    5.1 / 5.1
// The line: 320 units (12 contexts of 32 heads, d = 128, bf16, up to 48 tokens and 16 steps, 384 units, 90.1 / 86.7 a pass; 8
// contexts, fp16, 72.6 / 79.3).  fp32 inputs at d = 128 keep one head unless the buffers are short (cap <= 64: 100 contexts of up to
// 40 tokens, 8 steps, 187.6 / 184.7), or one head has more workgroups a request than a fill word counts.
// Packed fill words (32 slots to a line): two heads also halve the additions that queue for a line, and win earlier, from 256
// units on at d = 128 and 96 below, with fp32 inputs too.  One / two: 8 requests of 32 heads, up to 48 records, d = 128, bf16 6.2 / 5.3,
// fp32, cap 128, 6.8 / 5.8; 6 of d = 64 5.9 / 5.1; 128 of up to 108 records, fp32 33.5 / 30.5; 13 of 8 heads, d = 128, 4.9 / 5.6.
// ---------------------------------------------------------------------------
template <int D, typename TIn, typename TRec, int HB, bool PAGED>
__global__ __launch_bounds__(NT) void kvb_buffer_step_kernel(const int32_t *slot_arg, int32_t nu_arg, int32_t deal_arg,
                                                             const StepArgs a)
{
    // (leading arguments: as in kvb_step_kernel, with the workgroups of a request in the place of its heads)
    constexpr int LPR = D / 4;       // lanes covering one record with 4 elements each
    constexpr int RPP = NT / LPR;    // delta-value rows per pass
    constexpr int GL = D / 8;        // lanes sharing one key dot product (8 elements each)
    constexpr int NG = NT / GL;      // keys per pass
    constexpr int WREC = 64;
    constexpr bool MDOT = sizeof(TIn) == 2;      // dot products on the matrix instruction: a wave takes 16 records of a block
    constexpr int NST = D / 32;                  // its steps
    constexpr int KP = MDOT ? 1 : (WREC + NG - 1) / NG, UP = WREC / RPP;
    constexpr int NC = (KVB_MAX_CAP + WREC) / WREC * WREC;
    static_assert(GL >= HB && HB <= 4 && HB * D <= NT, "a lane of each key group and a column of each head to a thread");

    __shared__ float2 cW[HB][NC];    // -Gamma_l (k.k_l) and Gamma_l (q.k_l) of record l
    __shared__ float sQK;            // q.k of the token itself
    __shared__ __attribute__((aligned(16))) float red[NW][HB][2][D];
    __shared__ int sBlk[NW][MAX_BLOCKS];

    const int tid = threadIdx.x;
    const int lb = unit_of(blockIdx.x, deal_arg);
    const int b = quotient(lb, nu_arg);
    const int32_t slot = slot_arg[b];
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    const int s = with_registers(slot, a.q, a.k, a.v, a.Hv, a.st.fill, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.g, a.beta, a.st.n_slots, a.st.fill_lg, a.r, a.cap);
    const int r = a.r;
    const int per = (r + HB - 1) / HB;   // workgroups of a key head
    const int of_b = lb - b * nu_arg, hk = quotient(of_b, per);
    const int h0 = hk * r + (of_b - hk * per) * HB, hlast = hk * r + r - 1;
    const int nh = min(HB, hlast - h0 + 1);
    const int cap = a.cap;
    if (s < 0 || s >= a.st.n_slots)
        return;

    const int rg = tid / LPR, c4 = tid % LPR;
    const int grp = tid / GL, sub = tid % GL;
    const int lm = tid % 16, lq = tid % 64 / 16, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int own = MDOT ? lq : sub;         // lanes own < nh make the weights of head own
    const int jw = min(own, nh - 1);
    const int jc = min(tid / D, nh - 1);     // head whose column tid % D this thread finishes
    const Out<TIn> out{a.out, a.out_wide != 0};
    const int blk_id = load_block_id<PAGED>(a.st, s, tid % 64);

    // loads that need only the request
    const size_t nr_o = ((size_t)b * a.Hk + hk) * D + 8 * sub;
    const Raw8<TIn> q_raw = load_raw8(static_cast<const TIn *>(a.q) + nr_o);
    const Raw8<TIn> k_raw = load_raw8(static_cast<const TIn *>(a.k) + nr_o);
    // the rows k, q, k, q, .. as an operand of the matrix instruction
    uint4 kq_op[MDOT ? NST : 1];
    if constexpr (MDOT) {
        const TIn *row = static_cast<const TIn *>(lm % 2 ? a.q : a.k) + ((size_t)b * a.Hk + hk) * D + 8 * lq;
#pragma unroll
        for (int st = 0; st < NST; ++st)
            kq_op[st] = *reinterpret_cast<const uint4 *>(row + 32 * st);
    }
    const TIn v_raw = static_cast<const TIn *>(a.v)[((size_t)b * a.Hv + h0 + jc) * D + tid % D];
    const float bet = a.beta[(size_t)b * a.Hv + h0 + jc];
    const float g_w = a.g[(size_t)b * a.Hv + h0 + jw];
    const int f = fill_before(*a.st.fill_of(s), 0);
    if (f + 1 > cap) {
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
        return;
    }
    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, cap, sBlk[__builtin_amdgcn_readfirstlane(tid / 64)], tid % 64, blk_id);
    const auto krec = make_rows<D>(static_cast<TIn *>(a.st.buf_k), pg, a.Hk, hk);
    // (of head h0; the next heads' records follow a block of cap or block_size records further on)
    const auto urec = make_rows<D>(static_cast<TRec *>(a.st.buf_u), pg, a.Hv, h0);
    const auto Grec = make_rows<1>(a.st.buf_G, pg, a.Hv, h0);
    // cumulative log decay of the new row, of head h0 + jw
    const float Gc = (f > 0 ? *Grec.at(f - 1, jw * pg.bs) : 0.0f) + g_w;

    float q8[8], k8[8];
    float4 accU[HB], accO[HB];
#pragma unroll
    for (int j = 0; j < HB; ++j)
        accU[j] = accO[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    unpack8(q_raw, q8);
    unpack8(k_raw, k8);
    for (int l0 = 0; l0 == 0 || l0 < f; l0 += WREC) {   // uniform
        // raw bits from always-valid addresses: an index past the fill is clamped to record 0, its value ignored
        Raw8<TIn> kl_raw[MDOT ? 1 : KP];
        uint4 k_op[MDOT ? NST : 1];
        float Gl[KP];
        Raw4<TRec> ur_raw[HB][UP];
        if constexpr (MDOT) {   // key row lm of the wave's 16 as the other operand
            const int l = l0 + 16 * wave + lm, lc = l < f ? l : 0;
#pragma unroll
            for (int st = 0; st < NST; ++st)
                k_op[st] = *reinterpret_cast<const uint4 *>(krec.at(lc, 8 * lq + 32 * st));
            Gl[0] = *Grec.at(lc, jw * pg.bs);
        } else {
#pragma unroll
            for (int p = 0; p < KP; ++p) {
                const int l = l0 + grp + NG * p, lc = l < f ? l : 0;
                kl_raw[p] = load_raw8(static_cast<const TIn *>(krec.at(lc, 8 * sub)));
                Gl[p] = *Grec.at(lc, jw * pg.bs);
            }
        }
#pragma unroll
        for (int p = 0; p < UP; ++p) {
            const int l = l0 + rg + RPP * p, lc = l < f ? l : 0;
#pragma unroll
            for (int j = 0; j < HB; ++j)
                ur_raw[j][p] = load_raw4(static_cast<const TRec *>(urec.at(lc, min(j, nh - 1) * pg.bs * D + 4 * c4)));
        }
        __builtin_amdgcn_sched_barrier(0);
        if (l0 == 0 && a.advance)
            advance_fill(a.st.fill_of(s), of_b == 0, nu_arg, 1);
        if constexpr (MDOT) {
            if (l0 + 16 * wave < f) {   // uniform
                // rows 4 lq + v of the product are k (v = 0) and q (v = 1) for every lq, its columns the records
                // 32 dimensions a product, their sums added in pairs: in one chain, whose roundings are each of the whole sum, dots of
                // positive terms were 6.3e-8 off 64 bits (root mean square) instead of 4.0e-8 as on the vector ALU and so, and the
                // outputs of short contexts 2 % further off.  (fp16 below its normal range keeps fewer bits in these products:
                // contexts of such keys alone 1.9e-7 off at 2^-18, 2.8e-6 at 2^-22, on the vector ALU 7e-8.)
                float dk = 0.0f, dq = 0.0f;
#pragma unroll
                for (int st = 0; st < NST; st += 2) {
                    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
                    const f32x4_t x = mfma16x32<TIn>(kq_op[st], k_op[st], zero);
                    float xk = x[0], xq = x[1];
                    if constexpr (NST > 1) {
                        const f32x4_t y = mfma16x32<TIn>(kq_op[st + 1], k_op[st + 1], zero);
                        xk += y[0];
                        xq += y[1];
                    }
                    dk = st == 0 ? xk : dk + xk;
                    dq = st == 0 ? xq : dq + xq;
                    asm volatile("" : "+v"(dk), "+v"(dq));
                }
                // (opaque: the compiler otherwise puts its address for the next WREC records ahead of the branch that leaves the
                // loop, into a register with a load in flight, and wave 0 waits for its addition to the fill there: 0.5 us a
                // step.  6 contexts of 32 heads, 20 records, eight steps: 46.7 us with it, 42.9 so; blocks of 8 52.1 and 47.1)
                int row = lm;
                asm volatile("" : "+v"(row));
                const int l = l0 + 16 * wave + row;
                const float w = expf(Gc - Gl[0]);
                if (own < nh && l < f)
                    cW[own][l] = make_float2(-w * dk, w * dq);
            }
        } else {
#pragma unroll
            for (int p = 0; p < KP; ++p) {
                const int l = l0 + grp + NG * p;
                if (l0 + NG * p >= f)   // uniform: nothing of this pass is live
                    break;
                float kx[8];
                unpack8(kl_raw[p], kx);
                float dkk = 0.0f, dq = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    dkk = fmaf(kx[e], k8[e], dkk);
                    dq = fmaf(kx[e], q8[e], dq);
                }
                dkk = group_sum<GL>(dkk);
                dq = group_sum<GL>(dq);
                if (own < nh && l < f) {
                    const float w = expf(Gc - Gl[p]);
                    cW[own][l] = make_float2(-w * dkk, w * dq);
                }
            }
        }
        __syncthreads();   // (blocks write disjoint parts of cW)
#pragma unroll
        for (int p = 0; p < UP; ++p) {
            const int l = l0 + rg + RPP * p;
            if (l0 + RPP * p >= f)   // uniform
                break;
#pragma unroll
            for (int j = 0; j < HB; ++j) {
                const float4 u = unpack4(ur_raw[j][p]);
                if (l < f) {
                    const float2 c = cW[j][l];
                    fma4(accU[j], c.x, u);
                    fma4(accO[j], c.y, u);
                }
            }
        }
    }
    float dqk = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        dqk = fmaf(q8[e], k8[e], dqk);
    dqk = group_sum<GL>(dqk);
    if (tid == 0)
        sQK = dqk;

    // reduce over the row groups: lane permutations inside the wave, LDS across waves
#pragma unroll
    for (int j = 0; j < HB; ++j) {
        accU[j] = column_sum<LPR>(accU[j]);
        accO[j] = column_sum<LPR>(accO[j]);
        if (tid % 64 < LPR) {
            *reinterpret_cast<float4 *>(&red[tid / 64][j][0][4 * (tid % 64)]) = accU[j];
            *reinterpret_cast<float4 *>(&red[tid / 64][j][1][4 * (tid % 64)]) = accO[j];
        }
    }
    __syncthreads();
    if (tid < nh * D) {
        const int col = tid % D;
        float au = 0.0f, ao = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            au += red[w][jc][0][col];
            ao += red[w][jc][1][col];
        }
        // the record as it is stored is what every later use reads, this token's output included
        const TRec ur_new = from_f32<TRec>(bet * (to_f32(v_raw) + au));
        ao = fmaf(sQK, to_f32(ur_new), ao);
        out.put1(((size_t)b * a.Hv + h0 + jc) * D + col, a.scale * ao);
        put<false>(urec.at(f, jc * pg.bs * D + col), ur_new);
    }
    if (own < nh && (MDOT ? tid < 64 && lm == 0 : grp == 0))
        put<false>(Grec.at(f, jw * pg.bs), Gc);
    if (h0 == hk * r && tid < D / 8)   // the threads that loaded the new k row store it
        store_raw8(krec.at(f, 8 * sub), k_raw);
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
template <int D, typename TIn, typename TRec, int WREC>
void launch_step_s(const StepArgs &a, int blocks, hipStream_t stream)
{
    // (a branch inside the kernel around the state loads would make the compiler's wait
    // counters conservative at the join, so these are compile-time variants)
    const bool st = a.stream_state != 0 && D == 128;   // the small head sizes are not tuned: no streaming variant
    const int deal = unit_deal(blocks, a.r, step_deals_from(D, blocks, a.threshold, st, a.advance != 0, a.st.apart()));
    if (a.threshold > 0) {
        if constexpr (D == 128) {
            if (st) {
                LAUNCH_LEAD(blocks, deal, stream, a, kvb_step_kernel<D, TIn, TRec, WREC, true, true);
                return;
            }
        }
        LAUNCH_LEAD(blocks, deal, stream, a, kvb_step_kernel<D, TIn, TRec, WREC, true, false);
        return;
    }
    if constexpr (D == 128) {
        if (st) {
            LAUNCH_LEAD(blocks, deal, stream, a, kvb_step_kernel<D, TIn, TRec, WREC, false, true);
            return;
        }
    }
    LAUNCH_LEAD(blocks, deal, stream, a, kvb_step_kernel<D, TIn, TRec, WREC, false, false);
}

template <int D, typename TIn, typename TRec, int HB>
void launch_buffer_step_h(const StepArgs &a, int B, hipStream_t stream)
{
    const int32_t per = (a.r + HB - 1) / HB, nu = a.Hk * per;   // workgroups of a key head and of a request
    const int deal = unit_deal(B * nu, per, deals_from(DEAL_BUFFER_STEP, a.st.apart()));
    if (a.st.block_table)
        launch(kvb_buffer_step_kernel<D, TIn, TRec, HB, true>, B * nu, stream, a.slot, nu, deal, a);
    else
        launch(kvb_buffer_step_kernel<D, TIn, TRec, HB, false>, B * nu, stream, a.slot, nu, deal, a);
}

template <int D, typename TIn, typename TRec>
void launch_buffer_step(const StepArgs &a, int blocks, hipStream_t stream)
{
    const int B = blocks / a.Hv;
    if (buffer_step_heads(D, sizeof(TIn) == 4, a.Hk, a.Hv, a.cap, blocks, a.st.apart()) == 2)
        launch_buffer_step_h<D, TIn, TRec, 2>(a, B, stream);
    else
        launch_buffer_step_h<D, TIn, TRec, 1>(a, B, stream);
}

template <int D, typename TIn, typename TRec>
void launch_step_w(const StepArgs &a, int blocks, hipStream_t stream)
{
    if (!a.st.state) {
        launch_buffer_step<D, TIn, TRec>(a, blocks, stream);
        return;
    }
    // Register window of buffered records.  For d = 128 the smallest tier that holds the
    // whole buffer is used; the smaller head sizes only carry the general (64 + tail) tier.
    if constexpr (D == 128) {
        if (a.cap <= 16) {
            launch_step_s<D, TIn, TRec, 16>(a, blocks, stream);
            return;
        }
        if (a.cap <= 32) {
            launch_step_s<D, TIn, TRec, 32>(a, blocks, stream);
            return;
        }
    }
    launch_step_s<D, TIn, TRec, 64>(a, blocks, stream);
}

// All head sizes of one (input type, record type) pair.
template <typename TIn, typename TRec>
int launch_step_typed(int dk, const StepArgs &a, int blocks, hipStream_t stream)
{
    switch (dk) {
    case 32:
        launch_step_w<32, TIn, TRec>(a, blocks, stream);
        return KVB_OK;
    case 64:
        launch_step_w<64, TIn, TRec>(a, blocks, stream);
        return KVB_OK;
    case 128:
        launch_step_w<128, TIn, TRec>(a, blocks, stream);
        return KVB_OK;
    }
    return KVB_EUNSUPPORTED;
}

}  // namespace kvb_impl
#endif  // KVB_STEP_KERNEL_H
