// kvb_direct: kvb_direct_mfma_kernel (16-bit inputs, d = 128) and kvb_direct_rows_kernel (fp32 inputs and the
// other head sizes).
#include "kvb_device.h"

namespace kvb_impl {

// (HIP's uint4 is a struct: arrays of it can end up in scratch memory)
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// kvb_direct for 16-bit inputs (bf16 or fp16) and d = 128, on the matrix cores throughout.
//
// The context is cut into blocks of 16 rows.  With N_il = beta_i Gamma_il (k_i.k_l) (l < i)
// and M_il = Gamma_il (q_i.k_l) (l <= i) the parallel form (Eq. 13) is
//     (I + N) U = Diag(beta) V,      O = M U.
// The diagonal blocks T_d = (I + N_dd)^-1 come from a blocked inversion (unit_lower_inverse16 below; N_dd is
// strictly lower) with fp32 operands on v_mfma_f32_16x16x4_f32 (exact products); the kernel then forms the
// whole inverse and multiplies (see its own header).
//   * Gram tiles (k.k, q.k over dk = 128, 16-bit operands): v_mfma_f32_16x16x32_{bf16,f16}.
//
// Register chaining.  Call "A-form" of a 16x16 matrix X the register layout in which lane l
// holds X[l%16][4*(l/16)+v], v = 0..3, and "B-form" the one with X[4*(l/16)+v][l%16].  An
// MFMA result is in B-form; feeding four k-steps with (a = xa[v], b = yb[v]) gives the
// B-form of X Y, and swapping the operands, (a = yb[v], b = xa[v]), gives the A-form of X Y.
// A Gram tile computed as (rows of block e) x (rows of block d) lands directly in A-form of
// the (d, e) tile, so no value ever needs to move between lanes: tiles shared between waves
// go through LDS as whole per-lane float4s.  Each wave owns 32 dv columns (two column tiles).
// ---------------------------------------------------------------------------

// B-form of X Y from X in A-form and Y in B-form (swap the arguments for the A-form of X Y).
__device__ __forceinline__ f32x4_t mm16(const f32x4_t &xa, const f32x4_t &yb, f32x4_t acc)
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[v], yb[v], acc, 0, 0, 0);
    return acc;
}

// A-form of (I + N)^-1 for a strictly lower triangular 16 x 16 block N given in both forms
// (ia: the identity, which reads the same in both).  Blocked inversion, exact: with the
// diagonal blocks of a 2 x 2 block partition already inverted (T), [[A,0],[C,B]]^-1 =
// T - T C T.  Three levels: 4 x 4 diagonal blocks D0, where (I + D0)^-1 = (I - D0)(I + D0^2)
// since D0^4 = 0; then the 4 x 4 blocks C1 under them inside each 8 x 8; then the lower left
// 8 x 8 block C2.  Every intermediate stays of the size of the inverse itself.  (The plain
// Neumann product (I - N)(I + N^2)(I + N^4)(I + N^8) is also exact in exact arithmetic, but its
// powers grow like binomial coefficients when the keys of a block are strongly correlated, and
// the cancellation then costs four digits.)
__device__ __forceinline__ f32x4_t unit_lower_inverse16(const f32x4_t &na, const f32x4_t &nb, const f32x4_t &ia,
                                                        int c16, int lq)
{
    f32x4_t d0a, d0b, c1a, c2a;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int ai = c16, al = 4 * lq + v;   // A-form: row, column inside the block
        const int bi = al, bl = ai;            // B-form
        d0a[v] = ai / 4 == al / 4 ? na[v] : 0.0f;
        d0b[v] = bi / 4 == bl / 4 ? nb[v] : 0.0f;
        c1a[v] = (ai / 8 == al / 8 && ai / 4 == al / 4 + 1) ? na[v] : 0.0f;
        c2a[v] = (ai >= 8 && al < 8) ? na[v] : 0.0f;
    }
    const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
    const f32x4_t d2b = mm16(d0a, d0b, z);                 // D0^2
    const f32x4_t t0a = mm16(ia + d2b, ia - d0a, z);       // (I - D0)(I + D0^2), A-form
    const f32x4_t t0b = mm16(ia - d0a, ia + d2b, z);       //                     B-form
    const f32x4_t p1b = mm16(c1a, t0b, z);                 // C1 T0
    const f32x4_t t1a = t0a - mm16(p1b, t0a, z);           // T0 - T0 C1 T0
    const f32x4_t t1b = t0b - mm16(t0a, p1b, z);
    const f32x4_t p2b = mm16(c2a, t1b, z);                 // C2 T1
    return t1a - mm16(p2b, t1a, z);                        // T1 - T1 C2 T1
}

// exp for arguments that are differences of cumulative log decays (<= 0, a few tens at
// most): one multiply and the hardware exp2; relative error about |x| * 2^-23, far inside
// the 2e-3 bound of the bf16 paths that use it.
__device__ __forceinline__ float fast_exp(float x) { return __expf(x); }

template <typename... Ts>
constexpr uint32_t pack2(Ts... xs)
{
    uint32_t r = 0;
    int sh = 0;
    ((r |= (uint32_t)xs << sh, sh += 2), ...);
    return r;
}

// Raw Gram tile from rows staged in LDS (row stride GS bf16 elements): lane l reads row l%16
// of the A-side block and of the B-side block at k = 8*(l/16) + 32*step.  acc[v] =
// (A-side row 4*(l/16)+v) . (B-side row l%16), i.e. the A-form of the (B-block, A-block) tile.
template <typename TIn, int GS>
__device__ __forceinline__ f32x4_t gram16(const TIn *arow, const TIn *brow, int lq)
{
    f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const uint4 av = *reinterpret_cast<const uint4 *>(arow + 8 * lq + 32 * st);
        const uint4 bv = *reinterpret_cast<const uint4 *>(brow + 8 * lq + 32 * st);
        c = mfma16x32<TIn>(av, bv, c);
    }
    return c;
}

// One step of a 16 x 16 Gram tile in A-form (rows of block d against rows of block e): 16 bytes of row 16 e + c16 and of
// row 16 d + c16; fp32: contraction slot lq of instruction v stands for element 4 lq + v on both sides.
template <typename TIn>
__device__ __forceinline__ f32x4_t gram_step(const u32x4_t &row, const u32x4_t &own, f32x4_t c)
{
    if constexpr (sizeof(TIn) == 2) {
        c = mfma16x32<TIn>(__builtin_bit_cast(uint4, row), __builtin_bit_cast(uint4, own), c);
    } else {
        const f32x4_t x = __builtin_bit_cast(f32x4_t, row), y = __builtin_bit_cast(f32x4_t, own);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[v], y[v], c, 0, 0, 0);
    }
    return c;
}

// ---------------------------------------------------------------------------
// Contexts whose result is not finite.
//
// The kernels below multiply whole 16 x 16 tiles, zeros above the diagonal included, and those for 16-bit inputs
// cut fp32 values into 16-bit pieces.  For finite values in range that changes nothing.  But 0 * Inf and the second
// piece of Inf are NaN, so an infinity or a NaN in one token's key or value would reach earlier tokens, an infinite
// value would become NaN, and a fp16 piece has no value beyond 65504 (queries and keys need not be normalised, and a
// fp32 delta value may be larger).  All of these end in an output that is not finite: an output tile sums over the
// whole diagonal tile of delta values, and whatever an infinity meets stays infinite or becomes NaN.  So a wave whose
// outputs are all finite is done, and one that has produced anything else solves its columns again with this
// function, where a row sees exactly the rows before it:
//     u_i = beta_i ( v_i - sum_{l<i} Gamma_il (k_i.k_l) u_l )     o_i = sum_{l<=i} Gamma_il (q_i.k_l) u_l
// with fp32 products: Gram tiles and the products with earlier blocks on the matrix cores (every entry of those tiles
// belongs to the sum), the 16 rows of a diagonal block one after the other.  Nothing is staged: keys and queries come
// from the inputs again, earlier delta values from the records, which the same lane has written.  A wave needs nothing
// from the others, so this is no barrier's business.
// col0: the first of the lane's NC adjacent columns; sG, sB: cumulative log decays and betas of the context; ru: row of
// a record in buf_u.
// ---------------------------------------------------------------------------
template <int D, int NC, typename TIn, typename TRec, typename RowOf>
__device__ __forceinline__ void solve_by_token(const DirectArgs &a, int b, int h, int L, int col0, const float *sG, const float *sB,
                                               const RowOf &ru, int lane)
{
    constexpr int EPC = 16 / sizeof(TIn);   // elements of 16 bytes
    // (opaque: nothing computed for the kernel's own work stays in a register for this)
    asm volatile("" : "+v"(lane), "+v"(col0), "+s"(b), "+s"(h), "+s"(L));
    const int c16 = lane % 16, lq = lane / 16;
    const int hk = h / a.r;
    const TIn *kbase = static_cast<const TIn *>(a.k) + ((size_t)b * a.Lmax * a.Hk + hk) * D;
    const TIn *qbase = static_cast<const TIn *>(a.q) + ((size_t)b * a.Lmax * a.Hk + hk) * D;
    const TIn *vbase = static_cast<const TIn *>(a.v) + ((size_t)b * a.Lmax * a.Hv + h) * D + col0;
    const uint32_t qk_stride = (uint32_t)a.Hk * D, v_stride = (uint32_t)a.Hv * D;
    const Out<TIn> out{a.out, a.out_wide != 0};
    const size_t outp = (((size_t)b * a.Lmax) * a.Hv + h) * D + col0;
    TRec *up = static_cast<TRec *>(a.st.buf_u) + col0;
#pragma unroll 1
    for (int d = 0; 16 * d < L; ++d) {
        const int i = 16 * d + c16;   // this lane's row of the tiles in A-form
        const float gi = sG[i];
        const uint32_t own = (uint32_t)min(i, L - 1) * qk_stride + EPC * lq;
        f32x4_t acc[NC], o[NC];   // B-form: rows 16 d + 4 lq + v
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            o[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc[c][v] = to_f32(vbase[(uint32_t)min(16 * d + 4 * lq + v, L - 1) * v_stride + c]);
        }
        auto tiles = [&](int e, f32x4_t &n, f32x4_t &m) {   // -Gamma (k.k) below the diagonal, Gamma (q.k) up to it
            const uint32_t row = (uint32_t)min(16 * e + c16, L - 1) * qk_stride + EPC * lq;
            n = m = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1   // (few registers: this must not cost the kernel anything)
            for (int o = 0; o < D; o += 4 * EPC) {
                const u32x4_t kr = *reinterpret_cast<const u32x4_t *>(kbase + row + o);
                n = gram_step<TIn>(kr, *reinterpret_cast<const u32x4_t *>(kbase + own + o), n);
                m = gram_step<TIn>(kr, *reinterpret_cast<const u32x4_t *>(qbase + own + o), m);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int l = 16 * e + 4 * lq + v;
                const float w = expf(gi - sG[l]);
                n[v] = i < L && l < i ? -w * n[v] : 0.0f;
                m[v] = i < L && l <= i ? w * m[v] : 0.0f;
            }
        };
        f32x4_t n, m;
#pragma unroll 1
        for (int e = 0; e < d; ++e) {
            tiles(e, n, m);
            f32x4_t u[NC];
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    u[c][v] = to_f32(up[ru(16 * e + 4 * lq + v) * D + c]);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                acc[c] = mm16(n, u[c], acc[c]);
                o[c] = mm16(m, u[c], o[c]);
            }
        }
        tiles(d, n, m);
        // the rows of the block: row 4 g + x is held by the lanes lq = g, entry (row, 4 g + x) of a tile in A-form by
        // lane 16 g + row
        f32x4_t ub[NC];
#pragma unroll 1
        for (int g = 0; g < 4; ++g) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                float nc[4], mc[4];   // column 4 g + x, of the lane's own rows
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    nc[v] = __shfl(n[x], 16 * g + 4 * lq + v);
                    mc[v] = __shfl(m[x], 16 * g + 4 * lq + v);
                }
                const float beta = sB[16 * d + 4 * g + x];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    // the record as it is stored is what every later use reads
                    const float u = __shfl(rounded_to<TRec>(beta * acc[c][x]), 16 * g + c16);
                    if (lq == g)
                        ub[c][x] = u;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (4 * lq + v > 4 * g + x)
                            acc[c][v] = fmaf(nc[v], u, acc[c][v]);
                        if (4 * lq + v >= 4 * g + x)
                            o[c][v] = fmaf(mc[v], u, o[c][v]);
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * d + 4 * lq + v;
            if (row < L) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    out.put1(outp + (uint32_t)row * v_stride + c, a.scale * o[c][v]);
                    store1(up + ru(row) * D + c, ub[c][v]);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Pieces.  A fp32 value x is cut into NP values of the 16-bit input type, x = x_1 + ... + x_NP
// (+ a remainder below 2^-24 |x| for three bf16 pieces, 2^-22 |x| for two fp16 pieces), each
// what is left rounded to nearest, so that a product of two fp32 tiles becomes a few products
// of 16-bit tiles on v_mfma_f32_16x16x32, which runs at 16 times the rate of the fp32 matrix
// instruction.  take_piece handles two values at once and returns their pieces packed in one
// word (first value in the low half); the two arguments become the remainders.
// ---------------------------------------------------------------------------
template <typename T>
constexpr int pieces_of_f32() { return __is_same(T, bf16_t) ? 3 : 2; }

template <typename T>
__device__ __forceinline__ uint32_t take_piece(float &a, float &b)
{
    if constexpr (__is_same(T, bf16_t)) {
        typedef float f32x2_t __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
        a -= __uint_as_float(p << 16);   // exact
        b -= __uint_as_float(p & 0xFFFF0000u);
        return p;
    } else {
        const f16_t ha = from_f32<f16_t>(a), hb = from_f32<f16_t>(b);
        a -= to_f32(ha);   // exact
        b -= to_f32(hb);
        return (uint32_t)ha.bits | ((uint32_t)hb.bits << 16);
    }
}

// The four values a lane holds of a 16 x 16 tile (either form), cut into NP pieces; piece p is
// two words: values (0, 1) and (2, 3), which is how an operand of the 16-bit matrix instruction
// holds four consecutive contraction indices.
template <typename T, int NP>
__device__ __forceinline__ void split_tile(const f32x4_t &x, uint2 (&p)[NP])
{
    float x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        p[i].x = take_piece<T>(x0, x1);
        p[i].y = take_piece<T>(x2, x3);
    }
}

// acc += X Y for a 16 x 16 fp32 tile X given as NPX pieces in A-form and a tile Y given as NPY
// pieces in B-form (NPY = 1: Y is exactly representable in the 16-bit type).  One instruction
// contracts over 32 slots; a lane's 8 slots are its 4 contraction indices taken twice, so an
// instruction adds two piece products X_a Y_b + X_c Y_d.  Three instructions give the six
// products down to 2^-16 of the leading one.  The three that are left out, X2 Y3 + X3 Y2 + X3 Y3, are at most
// 5.4e-8 of the product and 6e-9 rms, without a bias (4 million pairs of normal values; the rounding of a fp32
// product is up to 6e-8, 2.5e-8 rms): that needs the pieces rounded to nearest.  Cut off instead, every piece has the
// sign of its value and they add up: 4.3e-7, 6e-8 rms, 4e-8 on the average.
template <typename T, int NPX, int NPY>
__device__ __forceinline__ f32x4_t mm16_pieces(const uint2 (&x)[NPX], const uint2 (&y)[NPY], f32x4_t acc)
{
    auto ins = [&](const uint2 &xa, const uint2 &xc, const uint2 &yb, const uint2 &yd) {
        acc = mfma16x32<T>(uint4{xa.x, xa.y, xc.x, xc.y}, uint4{yb.x, yb.y, yd.x, yd.y}, acc);
    };
    const uint2 zero = {0u, 0u};
    if constexpr (NPX == 3 && NPY == 3) {   // smallest terms first
        ins(x[2], x[0], y[0], y[2]);        // X3 Y1 + X1 Y3
        ins(x[1], x[1], y[1], y[0]);        // X2 Y2 + X2 Y1
        ins(x[0], x[0], y[0], y[1]);        // X1 Y1 + X1 Y2
    } else if constexpr (NPX == 3 && NPY == 1) {
        ins(x[2], zero, y[0], y[0]);        // X3 Y
        ins(x[0], x[1], y[0], y[0]);        // X1 Y + X2 Y
    } else if constexpr (NPX == 3 && NPY == 2) {
        ins(x[2], x[2], y[0], y[1]);        // X3 Y1 + X3 Y2
        ins(x[1], x[1], y[0], y[1]);        // X2 Y1 + X2 Y2
        ins(x[0], x[0], y[0], y[1]);        // X1 Y1 + X1 Y2
    } else if constexpr (NPX == 2 && NPY == 2) {
        ins(x[1], x[1], y[0], y[1]);        // X2 Y1 + X2 Y2
        ins(x[0], x[0], y[0], y[1]);        // X1 Y1 + X1 Y2
    } else {
        static_assert(NPX == 2 && NPY == 1, "piece counts");
        ins(x[0], x[1], y[0], y[0]);        // X1 Y + X2 Y
    }
    return acc;
}

// ---------------------------------------------------------------------------
// Longest contexts first.  The work of a launch grows with the contexts faster than linearly, and in the order of the
// batch a launch ends with whatever long contexts have come last.  Every workgroup therefore sorts the lengths of the
// batch, by counting, into classes of 16 tokens (the blocks that the kernels work in; the order of the batch inside a
// class) and takes the p-th request of that order: one vector load of lengths in the place of the scalar one, a barrier
// and a scan over 64 counts, 0.3 to 0.6 us.
// (The rule, longest_first, and the leading kernel argument, rank_lead, are in kvb_device.h.)

// inclusive sum over the wave
__device__ __forceinline__ int wave_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast 15 to rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast 31 to rows 2 and 3
    return x;
}
// The request at place p, and its length as it stands in len.
__device__ __forceinline__ int ranked_request(const int32_t *len, int B, int Lmax, int p, int wave, int lane, int &L,
                                              int *sLen /* [MAX_RANKED] */, int *sCount /* [64] */)
{
    auto class_of = [&](int l) {   // 0: the longest
        const int n = l < 0 || l > Lmax ? Lmax : l;
        return 7 - min(max(n - 1, 0) / 16, 7);
    };
    int l[2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
        l[x] = len[min(NT * x + 64 * wave + lane, B - 1)];
    int count = 0;   // lane 2 k + x: requests of class k among the 64 of this wave and half
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int i = NT * x + 64 * wave + lane, c = i < B ? class_of(l[x]) : -1;
        sLen[i] = l[x];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int n = __popcll(__ballot(c == k));
            count = lane == 2 * k + x ? n : count;
        }
    }
    if (lane < 16)
        sCount[8 * (lane / 2) + 4 * (lane % 2) + wave] = count;   // by class, then in the order of the batch
    __syncthreads();
    const int n = sCount[lane], upto = wave_sum(n);
    const int e = __builtin_ctzll(__ballot(upto > p));
    const int nth = p - __builtin_amdgcn_readlane(upto - n, e);
    const int first = NT * (e % 8 / 4) + 64 * (e % 4);
    const int mine = sLen[first + lane];
    const uint64_t in_class = __ballot(first + lane < B && class_of(mine) == e / 8);
    const bool hit = (in_class >> lane & 1) && (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(in_class >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in_class, 0)) == nth;
    const int at = __builtin_ctzll(__ballot(hit));
    L = __builtin_amdgcn_readlane(mine, at);
    return first + at;
}

// ---------------------------------------------------------------------------
// kvb_direct for 16-bit inputs, d = 128 and contexts of up to 64 tokens.
//
// With N_il = beta_i Gamma_il (k_i.k_l) (l < i) and M_il = Gamma_il (q_i.k_l) (l <= i) the
// parallel form (Eq. 13) is U = (I + N)^-1 Diag(beta) V, O = M U.  The kernel forms the inverse
// itself, A^ = (I + N)^-1 Diag(beta) (64 x 64, lower triangular, in 16 x 16 tiles), because then
//   * U = A^ V has the values -- exact 16-bit operands -- as its right factor: with A^ cut into
//     pieces the product runs on the 16-bit matrix instruction, one instruction per piece and per
//     two tiles of A^, and no block row waits for another (there is no substitution chain through
//     the 128 columns, which is where the time of a row-by-row solve goes);
//   * O = M U uses M in pieces (cut once, when the tile is weighted) and U in pieces.
// What is left in fp32 (v_mfma_f32_16x16x4_f32, exact products) is the small triangular
// work that produces A^: the four diagonal blocks T_d = (I + N_dd)^-1 (unit_lower_inverse16), and
// two levels of blocked inversion  [[P, 0], [C, R]]^-1 = [[P^-1, 0], [-R^-1 C P^-1, R^-1]]:
//     A_10 = -T_1 N_10 T_0                     A_32 = -T_3 N_32 T_2
//     W = C P^-1:  W_20 = (N_20 - N_21 T_1 N_10) T_0    W_21 = N_21 T_1      (same for row 3)
//     A_20 = -T_2 W_20   A_21 = -T_2 W_21   A_30 = -(A_32 W_20 + T_3 W_30)   A_31 = -(A_32 W_21 + T_3 W_31)
// Every entry of A is a key-to-key product through a chain of factors (I - beta k^T k); where these
// contract (beta |k|^2 <= 2, so for normalised keys, however they are correlated) it is bounded by
// |k|^2: forming the inverse loses nothing here.  The four waves
// share this work tile by tile; tiles cross LDS row-major, so that a reader takes them in
// A-form (one 16-byte read) or in B-form (four 4-byte reads, the transposed access).
//
// LDS, one region X used three times -- the staged keys; then the fp32 tiles N_de (d > e), T_d,
// A_32, W_20, W_21; then the pieces of A^ -- and the pieces of M next to it: 36 KB for bf16,
// four workgroups per CU (28 KB and five for fp16).  A wave owns 32 dv columns: column tile c of wave w holds columns
// 32 w + 2 n + c (n = 0..15), so a lane's two tiles are adjacent columns.
//
// LONG: contexts of up to 128 tokens, in two panels of 64 rows.  The first is the method above; its
// U_0 stays in registers, in pieces.  The second sees the first through N' = Gamma K_1 K_0^T (no beta)
// and M' = Gamma Q_1 K_0^T, 4 x 4 tiles each:
//     X = V_1 - N' U_0        U_1 = A^_1 X        O_1 = M' U_0 + M_1 U_1
// with A^_1 formed like A^_0.  X is fp32, so it goes through the 16-bit instruction in pieces as U
// does.  A context of up to 64 tokens in a LONG launch leaves after the first panel.  The line to LONG
// lies at Lmax = 64 because the 64-row kernel is the faster one there (four or five workgroups per CU
// instead of three).  Bound by the issue of vector and matrix instructions at three long-lived waves per
// SIMD.  96 contexts of ~U(1,128), 32 heads, bf16 with fp32 records: 192 -> 130 us (without the fold) against the kernel
// before it (8 block rows solved one after the other with fp32 matrix instructions); 128 of ~U(1,100),
// fp16 throughout: 193 -> 127 us.  Two workgroups per CU without any spill were 5 % slower than three that spill.  Token rows
// are a scalar address and the lane's own row, whose offsets the second panel works out again: 64-bit addresses lane by
// lane, kept from the first panel, made three workgroups spill 15 to 24 words (now one with contiguous fp32 records, else
// none): 96 contexts 100 -> 95 us (both sorted by length);
// pieces of U_0 kept in registers instead of cut again: two fit.
// ---------------------------------------------------------------------------
// Workgroups per CU: the two fp16 pieces need 28 KB of LDS and 95 registers, which leaves room for
// five (6 % faster than four on ragged lengths); the three bf16 pieces need 36 KB and 118.
// LONG: 53 KB and 168 registers, three.
template <typename T, bool LONG>
constexpr int DIRECT_WG_PER_CU = LONG ? 3 : __is_same(T, f16_t) ? 5 : 4;
template <typename TIn, typename TRec, bool LONG, bool PAGED>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(DIRECT_WG_PER_CU<TIn, LONG>, DIRECT_WG_PER_CU<TIn, LONG>))) void kvb_direct_mfma_kernel(
    const int32_t *len_arg, int32_t lead_arg, int32_t deal_arg, const DirectArgs a)
{
    // The three leading arguments hold a.len, rank_lead() and deal_of(): as plain leading kernel arguments
    // they are preloaded into scalar registers at wave launch (the build asks for it), so the load of
    // len[b] -- the head of the dependent chain to the first key byte -- goes out at once instead of after
    // the round trip that fetches the argument block.
    constexpr int D = 128;
    constexpr int LM = 64;   // rows of a panel
    constexpr int NB = LM / 16;                 // blocks of 16 rows (4)
    constexpr int NLOW = NB * (NB + 1) / 2;     // lower-triangular block pairs (10)
    constexpr int GS = D + 8;                   // LDS row stride of the staged keys (272 B:
                                                // consecutive rows start 4 banks apart)
    // Type of the pieces: the input type, whose values are then exact operands, but bf16 in every LONG kernel.
    // fp16 has not the range there: products beyond 65504 (queries and keys need not be normalised) have no
    // piece, and the second piece of a value below 0.25 is subnormal, in steps of 6e-8, which over two panels
    // adds up to twice the error of fp32 products (8.9e-7 of the outputs at 128 tokens).  A fp16 value of V or
    // of a record is then two bf16 pieces, exactly.
    using TP = std::conditional_t<LONG, bf16_t, TIn>;
    constexpr bool SAME = __is_same(TP, TIn);   // an input value is its own single piece
    constexpr int NP = pieces_of_f32<TP>();     // pieces of a fp32 tile
    constexpr int NPU = sizeof(TRec) == 4 ? NP : SAME ? 1 : 2;   // a 16-bit record is one piece as it stands
    static_assert(NB == NW, "one diagonal block per wave");
    constexpr int STAGE_BYTES = LM * GS * 2;
    constexpr int PIECE_BYTES = NLOW * NP * 512;        // pieces of A^ (and as much again for M)
    constexpr int F32_TILE = 1024;
    constexpr int OFF_N = 0;                            // N_de, d > e: 6 tiles, slot d (d - 1) / 2 + e
    constexpr int OFF_T01 = 6 * F32_TILE;               // T_0, T_1 (read before the pieces are written)
    constexpr int OFF_LATE = PIECE_BYTES;               // T_2, T_3, A_32, W_20, W_21 (read while they are)
    constexpr int X_BYTES = STAGE_BYTES > OFF_LATE + 5 * F32_TILE ? STAGE_BYTES : OFF_LATE + 5 * F32_TILE;
    static_assert(OFF_T01 + 2 * F32_TILE <= OFF_LATE, "the early tiles lie under the pieces only");
    // second panel (LONG): the keys of both panels staged, then the pieces of the 4 x 4 tiles N' (later M')
    // in the place of the pieces of M
    constexpr int CROSS_BYTES = NB * NB * NP * 512;
    constexpr int REGION_BYTES = !LONG                                     ? X_BYTES + PIECE_BYTES
                                 : X_BYTES + CROSS_BYTES > 2 * STAGE_BYTES ? X_BYTES + CROSS_BYTES
                                                                           : 2 * STAGE_BYTES;
    static_assert(CROSS_BYTES >= PIECE_BYTES, "the pieces of M fit where those of N' were");
    __shared__ __attribute__((aligned(16))) unsigned char region[REGION_BYTES];
    __shared__ __attribute__((aligned(16))) float sG[LONG ? 2 * LM : LM];
    __shared__ __attribute__((aligned(16))) float sB[LONG ? 2 * LM : LM];
    __shared__ int sBlk[NW][MAX_BLOCKS];
    // LONG: the first two weighted query tiles of each block row of the second panel, kept for its end (a lane's values
    // together, written and read by the same lane; 160 KB hold three workgroups with them)
    __shared__ float4 sM[LONG ? 7 : 1][64];
    TIn *sK = reinterpret_cast<TIn *>(region);
    auto pieceA = [&](int tile, int p) { return reinterpret_cast<uint2 *>(region + (tile * NP + p) * 512); };
    auto pieceM = [&](int tile, int p) { return reinterpret_cast<uint2 *>(region + X_BYTES + (tile * NP + p) * 512); };

    // (the wave index as a scalar: conditions and tile numbers derived from it are then uniform for
    // the compiler, scalar branches instead of masked ones)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int c16 = lane % 16, lq = lane / 16;
    const int lb = dealt_unit(blockIdx.x, deal_arg);
    const int Hv = lead_arg < 0 ? lead_arg & 0xFFFF : lead_arg;
    const int place = quotient(lb, Hv);   // of the request in the order of the launch
    int b = place, L;
    if (__builtin_expect(lead_arg < 0, LONG)) {   // uniform
        // (its tables lie where nothing is written before the barrier behind the staged keys)
        static_assert(REGION_BYTES >= STAGE_BYTES + 4 * (MAX_RANKED + 64), "room for the lengths");
        int *tables = reinterpret_cast<int *>(region + STAGE_BYTES);
        b = ranked_request(len_arg, lead_arg >> 16 & 0x7FFF, a.Lmax, place, wave, lane, L, tables, tables + MAX_RANKED);
    } else {
        L = len_arg[b];
    }
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    L = with_registers(L, a.slot, a.q, a.k, a.v, a.g, a.beta, a.st.fill, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.st.n_slots, a.Lmax, a.Hk, a.Hv);
    const int h = lb - place * Hv;
    const int r = a.r;
    const int hk = quotient(h, r);
    const int Lmax = a.Lmax;

    const int s = a.slot[b];
    if (s < 0 || s >= a.st.n_slots)
        return;
    if (L < 0 || L > Lmax) {
        L = Lmax;
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
    }
    if (L == 0) {
        if (h == 0 && tid == 0)
            put<false, true>(a.st.fill_of(s), 0);
        return;
    }
    // ---- every input of the workgroup is requested at once ------------------------
    // (no branch around a load: at a join the compiler waits for every load in flight, which would
    // make the passes take their round trips one after the other; a row past the context re-reads
    // the context's last row from the cache and is never used.  Reading the rows up to Lmax as they
    // are instead would cost a short context the traffic of a long one.)
    u32x4_t kst[NB];
    const int srow = tid / 16, sc8 = tid % 16;
    const int col2 = 32 * wave + 2 * c16;
    // (uniform 64-bit base + 32-bit per-lane offset keeps the address arithmetic out of the VGPRs)
    const TIn *kbase = static_cast<const TIn *>(a.k) + ((size_t)b * Lmax * a.Hk + hk) * D;
    const TIn *qbase = static_cast<const TIn *>(a.q) + ((size_t)b * Lmax * a.Hk + hk) * D;
    const TIn *vbase = static_cast<const TIn *>(a.v) + ((size_t)b * Lmax * a.Hv + h) * D;
    const uint32_t qk_stride = (uint32_t)a.Hk * (2 * D), v_stride = (uint32_t)a.Hv * (2 * D);   // bytes
    // 16 rows from i0 on as a scalar address; a lane adds its own row (times the stride), cut off at the last row
    auto row_at = [&](const TIn *base, uint32_t stride, int i0, uint32_t own, uint32_t in_row) {
        const int r0 = min(i0, L - 1);   // (scalars)
        return reinterpret_cast<const char *>(base) + (size_t)r0 * stride + (row_of_16(own, L - 1 - r0, stride) + in_row);
    };
    const uint32_t own_s = (uint32_t)srow * qk_stride, own_c = (uint32_t)c16 * qk_stride;
    uint32_t own_v[4];
#pragma unroll
    for (int v = 0; v < 4; ++v)
        own_v[v] = (uint32_t)(4 * lq + v) * v_stride;
#pragma unroll
    for (int p = 0; p < NB; ++p)   // pass p = rows 16 p .. 16 p + 15, 16 bytes per thread
        kst[p] = *reinterpret_cast<const u32x4_t *>(row_at(kbase, qk_stride, 16 * p, own_s, 16 * sc8));
    // Q is not staged: the waves read the rows of their q.k tiles straight from memory in the
    // operand layout of the matrix instruction (row 16 d + c16, k = 8 lq + 32 step); a block of
    // 16 query rows is 4 KB and is shared by at most 4 tiles, so the repeats hit in the caches.
    // Tiles are dealt round-robin: t = wave + 4 n; t < 6 are k.k pairs, the rest q.k pairs.
    constexpr uint32_t PDB = pack2(1, 2, 2, 3, 3, 3, 0, 1, 1, 2, 2, 2, 3, 3, 3, 3);
    constexpr uint32_t PEB = pack2(0, 0, 1, 0, 1, 2, 0, 0, 1, 0, 1, 2, 0, 1, 2, 3);
    auto PD = [](int t) { return (int)((PDB >> (2 * t)) & 3u); };
    auto PE = [](int t) { return (int)((PEB >> (2 * t)) & 3u); };
    u32x4_t qop[3][4];   // n = 1 (waves 2, 3 only), 2, 3
#pragma unroll
    for (int n = 1; n < 4; ++n) {
        const char *qrow = row_at(qbase, qk_stride, 16 * PD(wave + NW * n), own_c, 16 * lq);
#pragma unroll
        for (int st = 0; st < 4; ++st)
            qop[n - 1][st] = *reinterpret_cast<const u32x4_t *>(qrow + 64 * st);
    }
    const size_t gb_o = (size_t)b * Lmax * a.Hv + h;
    const uint32_t gb_l = (uint32_t)min(lane, L - 1) * a.Hv;
    float g_raw = (a.g + gb_o)[gb_l], beta_raw = (a.beta + gb_o)[gb_l];   // (every wave: a branch around a load costs more)
    float g_raw1 = 0.0f, beta_raw1 = 0.0f;
    if constexpr (LONG) {
        const uint32_t gb_l1 = (uint32_t)min(LM + lane, L - 1) * a.Hv;
        g_raw1 = (a.g + gb_o)[gb_l1];
        beta_raw1 = (a.beta + gb_o)[gb_l1];
    }

    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, a.cap, sBlk[wave], lane, load_block_id<PAGED>(a.st, s, lane));
    auto ru = [&](int l) { return pg.row(l, a.Hv, h); };
    const auto krec = make_rows<D>(static_cast<TIn *>(a.st.buf_k), pg, a.Hk, hk);
    const auto urec = make_rows<D>(static_cast<TRec *>(a.st.buf_u), pg, a.Hv, h);
    const auto Grec = make_rows<1>(a.st.buf_G, pg, a.Hv, h);
    const Out<TIn> out{a.out, a.out_wide != 0};
    const int nb = ((LONG ? min(L, LM) : L) + 15) / 16;
    auto tri = [](int d, int e) { return d * (d + 1) / 2 + e; };    // slot of pair d >= e
    auto trn = [](int d, int e) { return d * (d - 1) / 2 + e; };    // slot of pair d > e
    // fp32 tiles in LDS are row-major 16 x 16: A-form is one 16-byte access, B-form four 4-byte ones
    auto lds_a = [&](int off) {
        const float4 t = *reinterpret_cast<const float4 *>(region + off + c16 * 64 + lq * 16);
        return f32x4_t{t.x, t.y, t.z, t.w};
    };
    auto lds_b = [&](int off) {
        const float *t = reinterpret_cast<const float *>(region + off) + 64 * lq + c16;
        return f32x4_t{t[0], t[16], t[32], t[48]};
    };
    auto put_a = [&](int off, const f32x4_t &x) {
        *reinterpret_cast<float4 *>(region + off + c16 * 64 + lq * 16) = make_float4(x[0], x[1], x[2], x[3]);
    };
    // (tiles that only ever travel in B-form keep their per-lane layout)
    auto put_lane = [&](int off, const f32x4_t &x) {
        *reinterpret_cast<float4 *>(region + off + lane * 16) = make_float4(x[0], x[1], x[2], x[3]);
    };
    auto lds_lane = [&](int off) {
        const float4 t = *reinterpret_cast<const float4 *>(region + off + lane * 16);
        return f32x4_t{t.x, t.y, t.z, t.w};
    };
    constexpr int OFF_T2 = OFF_LATE, OFF_T3 = OFF_LATE + F32_TILE, OFF_A32 = OFF_LATE + 2 * F32_TILE,
                  OFF_W20 = OFF_LATE + 3 * F32_TILE, OFF_W21 = OFF_LATE + 4 * F32_TILE;
    auto off_n = [&](int d, int e) { return OFF_N + trn(d, e) * F32_TILE; };
    auto off_t = [&](int d) { return d < 2 ? OFF_T01 + d * F32_TILE : OFF_LATE + (d - 2) * F32_TILE; };

    // cumulative log decay (inclusive scan over the wave) and beta; wave 1 takes the second panel's and
    // scans the first one's again for the sum it starts from
    auto wave_scan = [&](float gv) {
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const float t = __shfl_up(gv, off);
            if (lane >= off)
                gv += t;
        }
        return gv;
    };
    if (wave == 0 || (LONG && wave == 1)) {
        float gv = wave_scan(lane < L ? g_raw : 0.0f);
        float bv = lane < L ? beta_raw : 0.0f;
        int row = lane;
        if (LONG && wave == 1) {
            row = LM + lane;
            gv = __shfl(gv, 63) + wave_scan(row < L ? g_raw1 : 0.0f);
            bv = row < L ? beta_raw1 : 0.0f;
        }
        sG[row] = gv;
        sB[row] = bv;
        // Decays and the fill, parts of a line, are plain stores: through the L2 each waits for memory, which short contexts do not
        // hide.  Through / plain, paged bf16 contexts of up to 15 tokens: 37 of 8 heads 6.57 / 6.34 us, 121 9.12 / 8.87; of up to 34,
        // 13 of 32 heads 9.88 / 9.75; kvb_direct and fold, 70 to 500 us, the same.  Keys, whole lines, go through (plain: 48 of 16
        // heads up to 57 tokens 12.9 / 13.3, 8 paged blocks 12.7 / 13.0).
        if (row < L)
            put<false, true>(Grec.at(row, 0), gv);
    }
    // stage K; the thread that loaded a piece of K also appends it to the buffer
#pragma unroll
    for (int p = 0; p < NB; ++p) {
        if (p < nb) {   // uniform
            *reinterpret_cast<u32x4_t *>(sK + (16 * p + srow) * GS + 8 * sc8) = kst[p];
            if (h == hk * r && 16 * p + srow < L)
                put<false>(reinterpret_cast<u32x4_t *>(krec.at(16 * p, srow, 8 * sc8)), kst[p]);
        }
    }
    __syncthreads();

    // ---- raw Gram tiles: this wave's diagonal k.k tile and its share of the others ----
    // off-diagonal k.k pairs (d > e): 6; q.k pairs (d >= e): 10
    // (two bits per entry, packed: a table indexed by the wave number would live in scratch)
    f32x4_t gdiag = {0.f, 0.f, 0.f, 0.f};
    if (wave < nb)
        gdiag = gram16<TIn, GS>(sK + (16 * wave + c16) * GS, sK + (16 * wave + c16) * GS, lq);
    f32x4_t gsh[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int t = wave + NW * n, d = PD(t), e = PE(t);
        gsh[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (d < nb) {   // uniform
            if (t < 6) {
                gsh[n] = gram16<TIn, GS>(sK + (16 * e + c16) * GS, sK + (16 * d + c16) * GS, lq);
            } else if (n > 0) {   // t >= 6 implies n >= 1
                const TIn *arow = sK + (16 * e + c16) * GS;
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const uint4 av = *reinterpret_cast<const uint4 *>(arow + 8 * lq + 32 * st);
                    gsh[n] = mfma16x32<TIn>(av, __builtin_bit_cast(uint4, qop[n > 0 ? n - 1 : 0][st]), gsh[n]);
                }
            }
        }
    }
    __syncthreads();   // every wave is done with the staged rows: the region now takes the tiles

    // v in B-form: rows 16 d + 4 lq + v, this lane's two adjacent columns 32 wave + 2 c16, + 1.
    // Requested only now, when the registers of the staged rows are free again; the values are not
    // needed before the last phase.
    uint32_t v_raw[NB][4];
#pragma unroll
    for (int d = 0; d < NB; ++d)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            v_raw[d][v] = *reinterpret_cast<const uint32_t *>(row_at(vbase, v_stride, 16 * d, own_v[v], 2 * col2));
    // ---- weights and masks.  A-form element of tile (d, e): row i = 16 d + c16, column l = 16 e + 4 lq + v.
    // N tiles go to LDS in fp32 (they enter the inverse), M tiles are cut into pieces at once.
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int t = wave + NW * n, d = PD(t), e = PE(t);
        if (d < nb) {
            const int i = 16 * d + c16;
            const bool isq = t >= 6;
            // (LDS reads without a condition, then selects: a read under a condition becomes a
            // branch with a wait of its own, one round trip per element)
            const float gi = sG[i];
            const float si = isq ? 1.0f : sB[i];
            const float4 gl4 = *reinterpret_cast<const float4 *>(&sG[16 * e + 4 * lq]);
            const float gl[4] = {gl4.x, gl4.y, gl4.z, gl4.w};
            f32x4_t o;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int l = 16 * e + 4 * lq + v;
                const bool ok = i < L && (isq ? l <= i : l < i);
                o[v] = ok ? si * fast_exp(gi - gl[v]) * gsh[n][v] : 0.0f;
            }
            if (isq) {
                uint2 pc[NP];
                split_tile<TP, NP>(o, pc);
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    pieceM(tri(d, e), p)[lane] = pc[p];
            } else {
                put_a(off_n(d, e), o);
            }
        }
    }
    // T_d = (I + N_dd)^-1 of the 16 rows from row0 on.  The raw diagonal tile is symmetric, so the same
    // registers give the A-form (row row0 + c16, column row0 + 4 lq + v) and the B-form (row and column swapped).
    const f32x4_t z4 = {0.f, 0.f, 0.f, 0.f};
    auto diagonal_inverse = [&](int row0, const f32x4_t &gdiag) {
        f32x4_t na, nbm, ia;   // N in both forms; identity mask (the same in both forms)
        const float gc = sG[row0 + c16], bc = sB[row0 + c16];
        const float4 gq4 = *reinterpret_cast<const float4 *>(&sG[row0 + 4 * lq]);
        const float4 bq4 = *reinterpret_cast<const float4 *>(&sB[row0 + 4 * lq]);
        const float gq[4] = {gq4.x, gq4.y, gq4.z, gq4.w}, bq[4] = {bq4.x, bq4.y, bq4.z, bq4.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int ia_i = row0 + c16, ia_l = row0 + 4 * lq + v;    // A-form indices
            const int ib_i = ia_l, ib_l = ia_i;                        // B-form indices
            na[v] = (ia_i < L && ia_l < ia_i) ? bc * fast_exp(gc - gq[v]) * gdiag[v] : 0.0f;
            nbm[v] = (ib_i < L && ib_l < ib_i) ? bq[v] * fast_exp(gq[v] - gc) * gdiag[v] : 0.0f;
            ia[v] = ia_i == ia_l ? 1.0f : 0.0f;
        }
        return unit_lower_inverse16(na, nbm, ia, c16, lq);
    };
    f32x4_t w_own = z4;    // W_2w (waves 0, 1) or W_3,w-2 (waves 2, 3), B-form
    f32x4_t a_lvl2 = z4;   // A_10 (wave 1) or A_32 (wave 3), A-form
    // ---- the off-diagonal tiles of A = (I + N)^-1, first half: A_10, A_32 and W = C P^-1, for the nb
    // row blocks of a panel (uniform; mm16(x_a, y_b) = B-form of X Y, mm16(y_b, x_a) = its A-form)
    auto inverse_first_half = [&](int nb, const f32x4_t &t_own) {
        if (nb > 1) {
            if (wave == 0 || wave == 2) {
                const int dr = wave == 0 ? 2 : 3;        // block row of C
                if (dr < nb) {
                    const f32x4_t y1a = mm16(lds_b(off_t(1)), lds_a(off_n(dr, 1)), z4);   // N_d1 T_1
                    const f32x4_t y2a = mm16(lds_b(off_n(1, 0)), y1a, z4);                // N_d1 T_1 N_10
                    w_own = mm16(lds_a(off_n(dr, 0)) - y2a, lds_b(off_t(0)), z4);         // (N_d0 - ...) T_0
                    if (wave == 0)
                        put_lane(OFF_W20, w_own);
                }
            } else if (wave == 1) {
                const f32x4_t pb = mm16(lds_a(off_n(1, 0)), lds_b(off_t(0)), z4);          // N_10 T_0
                a_lvl2 = -mm16(pb, t_own, z4);                                             // -T_1 (N_10 T_0)
                if (nb > 2) {
                    w_own = mm16(lds_a(off_n(2, 1)), lds_b(off_t(1)), z4);                 // N_21 T_1
                    put_lane(OFF_W21, w_own);
                }
            } else if (nb == 4) {   // wave 3
                w_own = mm16(lds_a(off_n(3, 1)), lds_b(off_t(1)), z4);                     // N_31 T_1
                const f32x4_t pb = mm16(lds_a(off_n(3, 2)), lds_b(off_t(2)), z4);          // N_32 T_2
                a_lvl2 = -mm16(pb, t_own, z4);                                             // -T_3 (N_32 T_2)
                put_a(OFF_A32, a_lvl2);
            }
        }
    };
    // ---- second half: A_2e = -T_2 W_2e, A_3e = -(A_32 W_2e + T_3 W_3e); then every tile of A,
    // its columns scaled by beta (A^ = A Diag(beta)), goes to LDS in pieces.  The pieces take the
    // place of the N tiles, T_0 and T_1, which nobody reads any more.
    auto inverse_second_half = [&](int row0, int nb, const f32x4_t &t_own) {
        auto put_pieces = [&](int d, int e, const f32x4_t &xa) {
            const float4 b4 = *reinterpret_cast<const float4 *>(&sB[row0 + 16 * e + 4 * lq]);
            uint2 pc[NP];
            split_tile<TP, NP>(f32x4_t{xa[0] * b4.x, xa[1] * b4.y, xa[2] * b4.z, xa[3] * b4.w}, pc);
#pragma unroll
            for (int p = 0; p < NP; ++p)
                pieceA(tri(d, e), p)[lane] = pc[p];
        };
        if (wave < nb)
            put_pieces(wave, wave, t_own);
        if (wave == 1 && nb > 1)
            put_pieces(1, 0, a_lvl2);
        if (wave == 3 && nb == 4)
            put_pieces(3, 2, a_lvl2);
        if (wave < 2) {
            if (nb > 2)
                put_pieces(2, wave, -mm16(w_own, lds_a(OFF_T2), z4));
        } else if (nb == 4) {
            const f32x4_t w2b = lds_lane(wave == 2 ? OFF_W20 : OFF_W21);
            f32x4_t x = mm16(w2b, lds_a(OFF_A32), z4);
            x = mm16(w_own, lds_a(OFF_T3), x);
            put_pieces(3, wave - 2, -x);
        }
    };
    f32x4_t t_own = z4;   // T_wave, A-form
    if (wave < nb) {
        t_own = diagonal_inverse(16 * wave, gdiag);
        if (nb > 1)
            put_a(off_t(wave), t_own);
    }
    __syncthreads();
    inverse_first_half(nb, t_own);
    __syncthreads();
    inverse_second_half(0, nb, t_own);
    __syncthreads();

    // ---- U = A^ V and O = M U on the 16-bit matrix instruction, this wave's 32 columns ----------
    // Operand of the values for two row blocks (e, e + 1) and column tile c: the lane's 8 slots are
    // rows 16 e + 4 lq + 0..3 and 16 (e + 1) + 4 lq + 0..3; a word of v_raw holds both column tiles.
    // (LONG takes the blocks one by one: a pair of tiles of which one lies above the diagonal multiplies its
    // values by zero, which a NaN among them would pass on to earlier rows.)
    constexpr int NPV = SAME ? 1 : 2;
    uint4 vop[LONG ? 1 : NB / 2][2];
    uint2 vpc[LONG ? NB : 1][2][NPV];   // pieces of V_e, column tile c
    if constexpr (!LONG) {
#pragma unroll
        for (int e2 = 0; e2 < NB / 2; ++e2) {
            const uint32_t *w0 = v_raw[2 * e2], *w1 = v_raw[2 * e2 + 1];
            vop[e2][0] = uint4{__builtin_amdgcn_perm(w0[1], w0[0], 0x05040100u), __builtin_amdgcn_perm(w0[3], w0[2], 0x05040100u),
                               __builtin_amdgcn_perm(w1[1], w1[0], 0x05040100u), __builtin_amdgcn_perm(w1[3], w1[2], 0x05040100u)};
            vop[e2][1] = uint4{__builtin_amdgcn_perm(w0[1], w0[0], 0x07060302u), __builtin_amdgcn_perm(w0[3], w0[2], 0x07060302u),
                               __builtin_amdgcn_perm(w1[1], w1[0], 0x07060302u), __builtin_amdgcn_perm(w1[3], w1[2], 0x07060302u)};
        }
    } else {
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const uint32_t *w = v_raw[e];
            if constexpr (SAME) {
                vpc[e][0][0] = uint2{__builtin_amdgcn_perm(w[1], w[0], 0x05040100u), __builtin_amdgcn_perm(w[3], w[2], 0x05040100u)};
                vpc[e][1][0] = uint2{__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u)};
            } else {
                float2 vv[4];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    vv[v] = unpack_pair<TIn>(w[v]);
                split_tile<TP, NPV>(f32x4_t{vv[0].x, vv[1].x, vv[2].x, vv[3].x}, vpc[e][0]);
                split_tile<TP, NPV>(f32x4_t{vv[0].y, vv[1].y, vv[2].y, vv[3].y}, vpc[e][1]);
            }
        }
    }
    uint2 upc[NB][2][NPU];   // the pieces of U_e, column tile c (B-form)
    auto cut_u = [](const f32x4_t &u, uint2(&p)[NPU]) {   // (16-bit records: already rounded)
        if constexpr (NPU == 1)
            p[0] = uint2{pack_pair<TRec>(u[0], u[1]), pack_pair<TRec>(u[2], u[3])};
        else
            split_tile<TP, NPU>(u, p);
    };
    // what the second panel keeps of U_0: one or two pieces as they are, but the fp32 values instead of
    // three (16 registers less; they are cut again where they are used)
    constexpr bool RECUT = NPU > 2;
    f32x4_t ukeep[LONG && RECUT ? NB : 1][2];
    // outputs: a scalar row 16 d + v, and the lane's rows 4 lq below it
    const size_t outp = (((size_t)b * Lmax) * a.Hv + h) * D;
    const uint32_t out_l = (uint32_t)(4 * lq) * a.Hv * D + col2;
    auto out_row = [&](int i) { return outp + (size_t)i * a.Hv * D; };
    float big = 0.0f;   // largest output
#pragma unroll
    for (int d = 0; d < NB; ++d) {
        if (d < nb) {   // uniform
            f32x4_t U[2] = {z4, z4}, o[2] = {z4, z4};
            if constexpr (!LONG) {
#pragma unroll
                for (int p = NP - 1; p >= 0; --p) {   // smallest pieces first
#pragma unroll
                    for (int e2 = 0; e2 <= d / 2; ++e2) {
                        const uint2 lo = pieceA(tri(d, 2 * e2), p)[lane];
                        uint2 hi = {0u, 0u};
                        if (2 * e2 + 1 <= d)
                            hi = pieceA(tri(d, 2 * e2 + 1), p)[lane];
                        const uint4 aop = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
                        for (int c = 0; c < 2; ++c)
                            U[c] = mfma16x32<TP>(aop, vop[e2][c], U[c]);
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e <= d; ++e) {
                    uint2 ap[NP];
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        ap[p] = pieceA(tri(d, e), p)[lane];
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        U[c] = mm16_pieces<TP, NP, NPV>(ap, vpc[e][c], U[c]);
                }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if constexpr (sizeof(TRec) == 2) {
                    // the outputs read the records as stored
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        U[c][v] = rounded_to<TRec>(U[c][v]);
                }
                cut_u(U[c], upc[d][c]);
                if constexpr (LONG && RECUT)
                    ukeep[d][c] = U[c];
            }
#pragma unroll
            for (int e = 0; e <= d; ++e) {
                uint2 mp[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    mp[p] = pieceM(tri(d, e), p)[lane];
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    o[c] = mm16_pieces<TP, NP, NPU>(mp, upc[e][c], o[c]);
            }
            big = largest(largest(big, o[0]), o[1]);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * d + 4 * lq + v;
                if (i < L) {
                    // (streaming stores: neither array is read again by this kernel, and lines that do not
                    // linger in the L2 leave it to the keys, queries and values that the heads of a request share)
                    out.put2_nt(out_row(16 * d + v), out_l, a.scale * o[0][v], a.scale * o[1][v]);
                    store2_nt(urec.at(16 * d + v, 4 * lq, col2), U[0][v], U[1][v]);
                }
            }
        }
    }
    if constexpr (LONG) {
        if (L > LM) {   // uniform
            const int nb1 = (L - LM + 15) / 16;
            // keys of both panels for staging (the first panel's again: their place in LDS was needed), and
            // this wave's 16 query rows in operand layout
            u32x4_t ks[2 * NB], qo[4];
            // (the lane's row offsets again, opaque: kept from the first panel they cost registers all the way)
            int row_s = srow, row_c = c16, row_q = lq;
            asm volatile("" : "+v"(row_s), "+v"(row_c), "+v"(row_q));
#pragma unroll
            for (int p = 0; p < 2 * NB; ++p)
                ks[p] = *reinterpret_cast<const u32x4_t *>(row_at(kbase, qk_stride, 16 * p, (uint32_t)row_s * qk_stride, 16 * sc8));
            {
                const char *qrow = row_at(qbase, qk_stride, LM + 16 * wave, (uint32_t)row_c * qk_stride, 16 * lq);
#pragma unroll
                for (int st = 0; st < 4; ++st)
                    qo[st] = *reinterpret_cast<const u32x4_t *>(qrow + 64 * st);
            }
            __syncthreads();   // the first panel's pieces are no longer read
            TIn *sK1 = reinterpret_cast<TIn *>(region + STAGE_BYTES);
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                *reinterpret_cast<u32x4_t *>(sK + (16 * p + srow) * GS + 8 * sc8) = ks[p];
                *reinterpret_cast<u32x4_t *>(sK1 + (16 * p + srow) * GS + 8 * sc8) = ks[NB + p];
                if (h == hk * r && LM + 16 * p + srow < L)
                    put<false>(reinterpret_cast<u32x4_t *>(krec.at(LM + 16 * p, srow, 8 * sc8)), ks[NB + p]);
            }
            __syncthreads();

            // ---- Gram tiles of block row `wave` of this panel, keys and queries against the keys of the first
            // panel (4 tiles) and of this one (up to the diagonal), weighted as they are (A-form: row LM + 16 wave +
            // c16, columns 4 lq + v of the block)
            f32x4_t n0[NB], m0[NB], n1[NB], m1[NB], gd1 = z4;
            const int i1 = LM + 16 * wave + c16;
            {
                u32x4_t ko[4];
#pragma unroll
                for (int st = 0; st < 4; ++st)
                    ko[st] = *reinterpret_cast<const u32x4_t *>(sK1 + (16 * wave + c16) * GS + 8 * lq + 32 * st);
                auto pair = [&](const TIn *arow, f32x4_t &n, f32x4_t &m) {
                    n = m = z4;
#pragma unroll
                    for (int st = 0; st < 4; ++st) {
                        const uint4 av = *reinterpret_cast<const uint4 *>(arow + 8 * lq + 32 * st);
                        n = mfma16x32<TIn>(av, __builtin_bit_cast(uint4, ko[st]), n);
                        m = mfma16x32<TIn>(av, __builtin_bit_cast(uint4, qo[st]), m);
                    }
                    settle<SETTLE_16BIT>(n, m);
                };
                const float gi = sG[i1], bi = sB[i1];
                auto weigh = [&](int l0, const f32x4_t &x, float si, bool strict) {
                    const float4 gl4 = *reinterpret_cast<const float4 *>(&sG[l0]);
                    const float gl[4] = {gl4.x, gl4.y, gl4.z, gl4.w};
                    f32x4_t o;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int l = l0 + v;
                        const bool ok = i1 < L && (strict ? l < i1 : l <= i1);
                        o[v] = ok ? si * fast_exp(gi - gl[v]) * x[v] : 0.0f;
                    }
                    return o;
                };
#pragma unroll
                for (int e = 0; e < NB; ++e) {
                    n0[e] = m0[e] = n1[e] = m1[e] = z4;
                    if (wave < nb1) {
                        pair(sK + (16 * e + c16) * GS, n0[e], m0[e]);
                        n0[e] = weigh(16 * e + 4 * lq, n0[e], 1.0f, true);
                        m0[e] = weigh(16 * e + 4 * lq, m0[e], 1.0f, true);
                        if (e <= wave) {
                            pair(sK1 + (16 * e + c16) * GS, n1[e], m1[e]);
                            if (e < wave)
                                n1[e] = weigh(LM + 16 * e + 4 * lq, n1[e], bi, true);
                            else   // (the diagonal tile stays raw: diagonal_inverse weighs it in both forms)
                                gd1 = n1[e];
                            m1[e] = weigh(LM + 16 * e + 4 * lq, m1[e], 1.0f, false);
                            if (e < 2)
                                sM[4 * e + wave - e][lane] = make_float4(m1[e][0], m1[e][1], m1[e][2], m1[e][3]);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __syncthreads();   // the staged keys are no longer read
            auto pieceX = [&](int d, int e, int p) {   // of the 4 x 4 tiles N', later M'
                return reinterpret_cast<uint2 *>(region + X_BYTES + ((NB * d + e) * NP + p) * 512);
            };
            auto put_cross = [&](int e, const f32x4_t &x) {
                uint2 pc[NP];
                split_tile<TP, NP>(x, pc);
#pragma unroll
                for (int p = 0; p < NP; ++p)
                    pieceX(wave, e, p)[lane] = pc[p];
            };
            t_own = z4;
            if (wave < nb1) {
#pragma unroll
                for (int e = 0; e < NB; ++e) {
                    put_cross(e, -n0[e]);
                    if (e < wave)
                        put_a(off_n(wave, e), n1[e]);
                }
                t_own = diagonal_inverse(LM + 16 * wave, gd1);
                if (nb1 > 1)
                    put_a(off_t(wave), t_own);
            }
            __syncthreads();

            // The products below go through the right factor block by block: its pieces are cut once and meet
            // every row block, whose eight sums are independent chains.
            auto first_panel_pieces = [&](int e, uint2(&up0)[2][NPU]) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if constexpr (RECUT) {
                        // (opaque, or the compiler keeps the pieces of an earlier cut in registers instead)
                        asm volatile("" : "+v"(ukeep[e][c]));
                        split_tile<TP, NPU>(ukeep[e][c], up0[c]);
                    } else {
#pragma unroll
                        for (int p = 0; p < NPU; ++p)
                            up0[c][p] = upc[e][c][p];
                    }
                }
            };
            auto cross_product = [&](f32x4_t(&acc)[NB][2]) {   // acc_d += sum_e (tile d, e in LDS) U_0e
#pragma unroll
                for (int e = 0; e < NB; ++e) {
                    uint2 up0[2][NPU];
                    first_panel_pieces(e, up0);
#pragma unroll
                    for (int d = 0; d < NB; ++d) {
                        if (d < nb1) {   // uniform
                            uint2 tp[NP];
#pragma unroll
                            for (int p = 0; p < NP; ++p)
                                tp[p] = pieceX(d, e, p)[lane];
#pragma unroll
                            for (int c = 0; c < 2; ++c)
                                acc[d][c] = mm16_pieces<TP, NP, NPU>(tp, up0[c], acc[d][c]);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);   // (one step's operands in registers at a time)
                }
            };
            // ---- X = V_1 - N' U_0 beside the first half of the inverse
            // (v in B-form: rows LM + 16 d + 4 lq + v, this lane's two columns; needed at the end only)
            uint32_t v1_raw[NB][4];
            auto request_v1 = [&]() {
#pragma unroll
                for (int d = 0; d < NB; ++d)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        v1_raw[d][v] = *reinterpret_cast<const uint32_t *>(row_at(vbase, v_stride, LM + 16 * d, (uint32_t)(4 * row_q + v) * v_stride, 2 * col2));
            };
            inverse_first_half(nb1, t_own);
            __builtin_amdgcn_sched_barrier(0);
            request_v1();
            f32x4_t x[NB][2];
#pragma unroll
            for (int d = 0; d < NB; ++d)
                x[d][0] = x[d][1] = z4;
            cross_product(x);   // (N' is stored negated)
            settle<SETTLE_16BIT>(x);
#pragma unroll
            for (int d = 0; d < NB; ++d)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float2 vv = unpack_pair<TIn>(v1_raw[d][v]);
                    x[d][0][v] += vv.x;
                    x[d][1][v] += vv.y;
                }
            __syncthreads();
            inverse_second_half(LM, nb1, t_own);
            if (wave < nb1) {
#pragma unroll
                for (int e = 0; e < NB; ++e)
                    put_cross(e, m0[e]);   // M' in the place of N'
            }
            __syncthreads();

            // ---- M' U_0, then U_1 = A^_1 X: row block e is complete with step e
            f32x4_t o1[NB][2], u1[NB][2];
#pragma unroll
            for (int d = 0; d < NB; ++d)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    o1[d][c] = u1[d][c] = z4;
            cross_product(o1);
            settle<SETTLE_16BIT>(o1);
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                if (e < nb1) {   // uniform
                    uint2 xp[2][NP];
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        split_tile<TP, NP>(x[e][c], xp[c]);
#pragma unroll
                    for (int d = e; d < NB; ++d) {
                        if (d < nb1) {   // uniform
                            uint2 ap[NP];
#pragma unroll
                            for (int p = 0; p < NP; ++p)
                                ap[p] = pieceA(tri(d, e), p)[lane];
#pragma unroll
                            for (int c = 0; c < 2; ++c)
                                u1[d][c] = mm16_pieces<TP, NP, NP>(ap, xp[c], u1[d][c]);
                        }
                    }
                    settle<SETTLE_16BIT>(u1[e][0], u1[e][1]);
                    if constexpr (sizeof(TRec) == 2) {
#pragma unroll
                        for (int c = 0; c < 2; ++c)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                u1[e][c][v] = rounded_to<TRec>(u1[e][c][v]);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = LM + 16 * e + 4 * lq + v;
                        if (i < L)
                            store2_nt(urec.at(LM + 16 * e + v, 4 * lq, col2), u1[e][0][v], u1[e][1][v]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();   // M' is no longer read: the pieces of M_1 take its place
            if (wave < nb1) {
#pragma unroll
                for (int e = 0; e < NB; ++e) {
                    if (e <= wave) {
                        uint2 pc[NP];
                        if (e < 2) {
                            const float4 t = sM[4 * e + wave - e][lane];
                            m1[e] = f32x4_t{t.x, t.y, t.z, t.w};
                        }
                        split_tile<TP, NP>(m1[e], pc);
#pragma unroll
                        for (int p = 0; p < NP; ++p)
                            pieceM(tri(wave, e), p)[lane] = pc[p];
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                if (e < nb1) {   // uniform
                    uint2 up1[2][NPU];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        cut_u(u1[e][c], up1[c]);
                    }
#pragma unroll
                    for (int d = e; d < NB; ++d) {
                        if (d < nb1) {   // uniform
                            uint2 mp[NP];
#pragma unroll
                            for (int p = 0; p < NP; ++p)
                                mp[p] = pieceM(tri(d, e), p)[lane];
#pragma unroll
                            for (int c = 0; c < 2; ++c)
                                o1[d][c] = mm16_pieces<TP, NP, NPU>(mp, up1[c], o1[d][c]);
                        }
                    }
                    settle<SETTLE_16BIT>(o1[e][0], o1[e][1]);
                    big = largest(largest(big, o1[e][0]), o1[e][1]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = LM + 16 * e + 4 * lq + v;
                        if (i < L)
                            out.put2_nt(out_row(LM + 16 * e + v), out_l, a.scale * o1[e][0][v], a.scale * o1[e][1][v]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if (__builtin_expect(!all_finite(big), 0))
        solve_by_token<D, 2, TIn, TRec>(a, b, h, L, col2, sG, sB, ru, lane);
    if (h == 0 && tid == 0)
        put<false, true>(a.st.fill_of(s), L);
}

// ---------------------------------------------------------------------------
// kvb_direct for fp32 inputs at any head size and for 16-bit inputs at d = 32 and 64 (contexts of up to 64
// tokens): block row by block row,
//     U_d = T_d ( beta V_d - sum_{e<d} N_de U_e ),      O_d = sum_{e<=d} M_de U_e,
// all products with fp32 values on v_mfma_f32_16x16x4_f32 (exact products), T_d by unit_lower_inverse16, the
// Gram tiles of 16-bit inputs on the 16-bit instruction.  With heads this small (or inputs this wide) a unit
// is a chain of waits rather than of products, so the pieces of the kernel above would shorten nothing and
// cost registers; what counts is that every input is requested at once and that no step is taken row by row.
// 48 contexts of ~U(1,64), 8/16 heads of 64, bf16, with the fold (17 us of it): 204 -> 32 us a pass against the
// kernel before it, which kept everything in LDS and solved row by row on the vector ALU.
// ---------------------------------------------------------------------------
// The 16 x 16 tile (rows of block d against rows of block e) in A-form: `rows` are the staged keys of block e,
// `own` this lane's part of row 16 d + c16, 16 bytes a step.
template <typename TIn, int D, int NST>
__device__ __forceinline__ f32x4_t gram_rows(const TIn *rows, const u32x4_t (&own)[NST], int lq)
{
    f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < NST; ++st)
        c = gram_step<TIn>(*reinterpret_cast<const u32x4_t *>(rows + (D / NST) * st + (D / NST / 4) * lq), own[st], c);
    if constexpr (sizeof(TIn) == 4)
        settle<SETTLE_FP32>(c);
    return c;
}

template <int D, typename TIn, typename TRec, bool PAGED>
// (register budgets: 4 workgroups per CU; fp32 rows of 128 take 55 KB of LDS, two; 16-bit rows of 32 with fp32 records
// 26 KB, and six were 6 % faster than five at 500 requests of 32 heads)
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(
    D == 128 ? 2 : D == 32 && sizeof(TIn) == 2 && sizeof(TRec) == 4 ? 6 : 4))) void kvb_direct_rows_kernel(
    const int32_t *len_arg, int32_t lead_arg, int32_t deal_arg, const DirectArgs a)
{
    // (leading arguments: see kvb_direct_mfma_kernel)
    constexpr int LM = 64;   // longest context
    constexpr int NB = LM / 16;
    constexpr int NLOW = NB * (NB + 1) / 2, NKK = NB * (NB - 1) / 2;
    constexpr int NC = D == 128 ? 2 : 1;          // column tiles per wave (d = 32: the last two waves have none)
    constexpr int EPC = 16 / sizeof(TIn);         // elements per 16-byte chunk
    constexpr int CPR = D / EPC;                  // chunks per row
    constexpr int NPS = LM * CPR / NT;            // chunks of K per thread
    constexpr int NST = D / (4 * EPC);            // steps of a Gram tile
    constexpr int GS = D + EPC;                   // LDS row stride: consecutive rows start 4 banks apart
    static_assert(NB == NW, "one diagonal block per wave");
    __shared__ __attribute__((aligned(16))) TIn sK[LM * GS];
    __shared__ float4 tN[NKK][64], tM[NLOW][64], tT[NB][64];   // -N_de (d > e), M_de, T_d in A-form, a lane's values together
    constexpr bool R16 = sizeof(TRec) == 2;
    __shared__ float4 tD[R16 ? NB : 1][64];                    // -N_dd
    __shared__ __attribute__((aligned(16))) float sG[LM], sB[LM];
    __shared__ int sBlk[NW][MAX_BLOCKS];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;   // (a scalar)
    const int c16 = lane % 16, lq = lane / 16;
    const int lb = dealt_unit(blockIdx.x, deal_arg);
    const int Hv = lead_arg < 0 ? lead_arg & 0xFFFF : lead_arg;
    const int place = quotient(lb, Hv);   // of the request in the order of the launch
    int b = place, L;
    if (__builtin_expect(lead_arg < 0, 0)) {   // uniform
        // (its tables lie where nothing is written before the barrier behind the staged keys)
        static_assert(sizeof(tM) >= 4 * (MAX_RANKED + 64), "room for the lengths");
        int *tables = reinterpret_cast<int *>(&tM[0][0]);
        b = ranked_request(len_arg, lead_arg >> 16 & 0x7FFF, a.Lmax, place, wave, lane, L, tables, tables + MAX_RANKED);
    } else {
        L = len_arg[b];
    }
    __builtin_amdgcn_sched_barrier(0);   // nothing that needs the argument block goes above this load
    L = with_registers(L, a.slot, a.q, a.k, a.v, a.g, a.beta, a.st.fill, a.st.buf_k, a.st.buf_u, a.st.buf_G, a.st.n_slots, a.Lmax, a.Hk, a.Hv);
    const int h = lb - place * Hv;
    const int r = a.r;
    const int hk = quotient(h, r);
    const int Lmax = a.Lmax;

    const int s = a.slot[b];
    if (s < 0 || s >= a.st.n_slots)
        return;
    if (L < 0 || L > Lmax) {
        L = Lmax;
        if (tid == 0 && a.st.status)
            atomicOr(&a.st.status[s], KVB_STATUS_OVERFLOW);
    }
    if (L == 0) {
        if (h == 0 && tid == 0)
            put<false>(a.st.fill_of(s), 0);
        return;
    }
    // ---- every input is requested at once (no branch around a load; a row past the context re-reads its last row)
    const TIn *kbase = static_cast<const TIn *>(a.k) + ((size_t)b * Lmax * a.Hk + hk) * D;
    const TIn *qbase = static_cast<const TIn *>(a.q) + ((size_t)b * Lmax * a.Hk + hk) * D;
    const TIn *vbase = static_cast<const TIn *>(a.v) + ((size_t)b * Lmax * a.Hv + h) * D;
    const uint32_t qk_stride = (uint32_t)a.Hk * D, v_stride = (uint32_t)a.Hv * D;
    u32x4_t kst[NPS];
    const int srow = tid / CPR, sch = tid % CPR;   // this thread's row within a pass of NT / CPR rows, and its chunk
#pragma unroll
    for (int p = 0; p < NPS; ++p)
        kst[p] = *reinterpret_cast<const u32x4_t *>(kbase + (uint32_t)min(NT / CPR * p + srow, L - 1) * qk_stride + EPC * sch);
    // pairs of blocks, dealt round-robin as in kvb_direct_mfma_kernel: t = wave + 4 n; t < 6 are k.k pairs, the rest q.k
    constexpr uint32_t PDB = pack2(1, 2, 2, 3, 3, 3, 0, 1, 1, 2, 2, 2, 3, 3, 3, 3);
    constexpr uint32_t PEB = pack2(0, 0, 1, 0, 1, 2, 0, 0, 1, 0, 1, 2, 0, 1, 2, 3);
    auto PD = [](int t) { return (int)((PDB >> (2 * t)) & 3u); };
    auto PE = [](int t) { return (int)((PEB >> (2 * t)) & 3u); };
    u32x4_t qop[3][NST];   // n = 1 (waves 2, 3 only), 2, 3
#pragma unroll
    for (int n = 1; n < 4; ++n) {
        const uint32_t o = (uint32_t)min(16 * PD(wave + NW * n) + c16, L - 1) * qk_stride + EPC * lq;
#pragma unroll
        for (int st = 0; st < NST; ++st)
            qop[n - 1][st] = *reinterpret_cast<const u32x4_t *>(qbase + o + 4 * EPC * st);
    }
    const size_t gb_o = ((size_t)b * Lmax + min(lane, L - 1)) * a.Hv + h;
    const float g_raw = a.g[gb_o], beta_raw = a.beta[gb_o];
    // v in B-form: rows 16 d + 4 lq + v, columns col0 .. col0 + NC - 1
    const bool has_cols = 16 * NC * wave < D;   // uniform
    const int col0 = has_cols ? 16 * NC * wave + NC * c16 : 0;
    struct VRow {
        TIn x[NC];
    } __attribute__((aligned(NC * sizeof(TIn))));
    VRow v_raw[NB][4];
#pragma unroll
    for (int d = 0; d < NB; ++d)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            v_raw[d][v] = *reinterpret_cast<const VRow *>(vbase + (uint32_t)min(16 * d + 4 * lq + v, L - 1) * v_stride + col0);

    const Pages<PAGED> pg = make_pages<PAGED>(a.st, s, a.cap, sBlk[wave], lane, load_block_id<PAGED>(a.st, s, lane));
    auto ru = [&](int l) { return pg.row(l, a.Hv, h); };
    auto rk = [&](int l) { return pg.row(l, a.Hk, hk); };
    const Out<TIn> out{a.out, a.out_wide != 0};
    const int nb = (L + 15) / 16;
    auto tri = [](int d, int e) { return d * (d + 1) / 2 + e; };    // slot of pair d >= e
    auto trn = [](int d, int e) { return d * (d - 1) / 2 + e; };    // slot of pair d > e

    // stage K; the thread that loaded a piece of K also appends it to the buffer
    TIn *kb = static_cast<TIn *>(a.st.buf_k);
#pragma unroll
    for (int p = 0; p < NPS; ++p) {
        const int row = NT / CPR * p + srow;
        *reinterpret_cast<u32x4_t *>(sK + row * GS + EPC * sch) = kst[p];
        if (h == hk * r && row < L)
            put<false>(reinterpret_cast<u32x4_t *>(kb + rk(row) * D + EPC * sch), kst[p]);
    }
    // Cumulative log decay and beta.  Token by token: only differences G_i - G_l are used, nearby ones above all,
    // and the roundings of a running sum cancel in them (a scan over the wave was 1.4 times further off in the
    // outputs and the state).  The lane's sum takes part up to its own token.
    if (wave == 0) {
        const float gv = lane < L ? g_raw : 0.0f;
        float run = 0.0f;
        for (int t0 = 0; t0 < 16 * nb; t0 += 16) {
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const float gt = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gv), t0 + t));
                run += t0 + t <= lane ? gt : 0.0f;
            }
        }
        sG[lane] = run;
        sB[lane] = lane < L ? beta_raw : 0.0f;
        if (lane < L)
            put<false>(a.st.buf_G + ru(lane), run);
    }
    __syncthreads();

    // ---- Gram tiles, weighted and masked at once (A-form: row i = 16 d + c16, column l = 16 e + 4 lq + v) ----
    auto own_keys = [&](int d, u32x4_t(&x)[NST]) {
#pragma unroll
        for (int st = 0; st < NST; ++st)
            x[st] = *reinterpret_cast<const u32x4_t *>(sK + (16 * d + c16) * GS + 4 * EPC * st + EPC * lq);
    };
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int t = wave + NW * n, d = PD(t), e = PE(t);
        if (d < nb) {   // uniform
            const bool isq = t >= 6;   // (implies n >= 1)
            f32x4_t raw;
            if (isq) {
                raw = gram_rows<TIn, D, NST>(sK + (16 * e + c16) * GS, qop[n > 0 ? n - 1 : 0], lq);
            } else {
                u32x4_t own[NST];
                own_keys(d, own);
                raw = gram_rows<TIn, D, NST>(sK + (16 * e + c16) * GS, own, lq);
            }
            const int i = 16 * d + c16;
            const float gi = sG[i];
            const float si = isq ? 1.0f : -sB[i];
            const float4 gl4 = *reinterpret_cast<const float4 *>(&sG[16 * e + 4 * lq]);
            const float gl[4] = {gl4.x, gl4.y, gl4.z, gl4.w};
            float o[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int l = 16 * e + 4 * lq + v;
                const bool ok = i < L && (isq ? l <= i : l < i);
                o[v] = ok ? si * expf(gi - gl[v]) * raw[v] : 0.0f;
            }
            if (isq)
                tM[tri(d, e)][lane] = make_float4(o[0], o[1], o[2], o[3]);
            else
                tN[trn(d, e)][lane] = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
    // T_d = (I + N_dd)^-1 for d = wave.  The raw diagonal tile is symmetric: the same registers give both forms.
    if (wave < nb) {
        const int d = wave;
        u32x4_t own[NST];
        own_keys(d, own);
        const f32x4_t gdiag = gram_rows<TIn, D, NST>(sK + (16 * d + c16) * GS, own, lq);
        f32x4_t na, nbm, ia;
        const float gc = sG[16 * d + c16], bc = sB[16 * d + c16];
        const float4 gq4 = *reinterpret_cast<const float4 *>(&sG[16 * d + 4 * lq]);
        const float4 bq4 = *reinterpret_cast<const float4 *>(&sB[16 * d + 4 * lq]);
        const float gq[4] = {gq4.x, gq4.y, gq4.z, gq4.w}, bq[4] = {bq4.x, bq4.y, bq4.z, bq4.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int ia_i = 16 * d + c16, ia_l = 16 * d + 4 * lq + v;    // A-form indices
            const int ib_i = ia_l, ib_l = ia_i;                            // B-form indices
            na[v] = (ia_i < L && ia_l < ia_i) ? bc * expf(gc - gq[v]) * gdiag[v] : 0.0f;
            nbm[v] = (ib_i < L && ib_l < ib_i) ? bq[v] * expf(gq[v] - gc) * gdiag[v] : 0.0f;
            ia[v] = ia_i == ia_l ? 1.0f : 0.0f;
        }
        const f32x4_t p = unit_lower_inverse16(na, nbm, ia, c16, lq);
        tT[d][lane] = make_float4(p[0], p[1], p[2], p[3]);
        if constexpr (R16)
            tD[d][lane] = make_float4(-na[0], -na[1], -na[2], -na[3]);
    }
    __syncthreads();

    // ---- block forward substitution and outputs, this wave's columns ----
    if (has_cols) {
        const f32x4_t z4 = {0.f, 0.f, 0.f, 0.f};
        auto tile = [&](const float4 &t) { return f32x4_t{t.x, t.y, t.z, t.w}; };
        f32x4_t U[NB][NC];
        const size_t outp = (((size_t)b * Lmax) * a.Hv + h) * D;
        TRec *up = static_cast<TRec *>(a.st.buf_u);
        float big = 0.0f;   // largest output
#pragma unroll
        for (int d = 0; d < NB; ++d) {
            if (d < nb) {   // uniform
                f32x4_t acc[NC], o[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    o[c] = z4;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[c][v] = sB[16 * d + 4 * lq + v] * to_f32(v_raw[d][v].x[c]);   // (beta is zero beyond the context)
                }
#pragma unroll
                for (int e = 0; e < d; ++e) {
                    const f32x4_t nn = tile(tN[trn(d, e)][lane]), mm = tile(tM[tri(d, e)][lane]);
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        acc[c] = mm16(nn, U[e][c], acc[c]);
                        o[c] = mm16(mm, U[e][c], o[c]);
                    }
                }
                const f32x4_t tt = tile(tT[d][lane]), mm = tile(tM[tri(d, d)][lane]);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    U[d][c] = mm16(tt, acc[c], z4);
                    if constexpr (R16) {
                        // Later blocks and this block's outputs read the records as stored, and so do the rows of
                        // the block themselves: once more, U = acc - N_dd U, from the rounded values (without it the
                        // outputs are 3 % further from 64 bits).
                        auto round_all = [&](f32x4_t x) {
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                x[v] = rounded_to<TRec>(x[v]);
                            return x;
                        };
                        U[d][c] = round_all(mm16(tile(tD[d][lane]), round_all(U[d][c]), acc[c]));
                    }
                    o[c] = mm16(mm, U[d][c], o[c]);
                    big = largest(big, o[c]);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * d + 4 * lq + v;
                    if (i < L) {
                        const size_t oo = outp + (uint32_t)i * v_stride + col0, uo = ru(i) * D + col0;
                        if constexpr (NC == 2) {
                            out.put2(oo, a.scale * o[0][v], a.scale * o[1][v]);
                            store2(up + uo, U[d][0][v], U[d][1][v]);
                        } else {
                            out.put1(oo, a.scale * o[0][v]);
                            store1(up + uo, U[d][0][v]);
                        }
                    }
                }
            }
        }
        if (!all_finite(big))
            solve_by_token<D, NC, TIn, TRec>(a, b, h, L, col0, sG, sB, ru, lane);
    }
    if (h == 0 && tid == 0)
        put<false>(a.st.fill_of(s), L);
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
int launch_direct(int dk, int in_dtype, int rec_dtype, const DirectArgs &a, int blocks, hipStream_t stream)
{
    const bool mfma = dk == 128 && in_dtype != KVB_F32;
    const int32_t lead = rank_lead(blocks / a.Hv, a.Hv, longest_first(blocks, a.Lmax, dk, in_dtype)), deal = deal_of(blocks, a.r);
    auto start = [&](auto paged, auto contiguous) {
        launch(a.st.block_table ? paged : contiguous, blocks, stream, a.len, lead, deal, a);
    };
    if (mfma)
        return dispatch_types16(in_dtype, rec_dtype, [&]<typename TIn, typename TRec>() {
            if (a.Lmax > 64)   // two panels of 64 rows
                start(kvb_direct_mfma_kernel<TIn, TRec, true, true>, kvb_direct_mfma_kernel<TIn, TRec, true, false>);
            else
                start(kvb_direct_mfma_kernel<TIn, TRec, false, true>, kvb_direct_mfma_kernel<TIn, TRec, false, false>);
        });
    if (a.Lmax > 64)   // the block-row kernel holds a 64-token context in LDS
        return KVB_EUNSUPPORTED;
    return dispatch(dk, in_dtype, rec_dtype, [&]<int D, typename TIn, typename TRec>() {
        if constexpr (!(D == 128 && sizeof(TIn) == 2))
            start(kvb_direct_rows_kernel<D, TIn, TRec, true>, kvb_direct_rows_kernel<D, TIn, TRec, false>);
    });
}

}  // namespace kvb_impl
