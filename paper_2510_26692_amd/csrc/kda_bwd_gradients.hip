// Last kernel of the backward pass, one workgroup of four waves per (chunk, head): from the state at the chunk's
// start S0, the gradient of the state at its end dS1, R = v - S^T k and Z = dV / beta (kda_f32_walk.hip) to the
// gradients of q, k, v, log alpha and beta.
//
//   X = beta Z = dV,   Vn = beta R,   dbeta_r = Z_r . R_r
//   dP = Tril(dO Vn^T)                      dA = -StrictTril(X Vn^T)
//   dQg = dO S0^T    dKg = -X S0^T          dKt = Vn dS1^T
//   dq_r = Gamma_r dQg_r + a2_r             a2_r = sum_{i<=r} dP[r,i] k_i e^(G_r - G_i)
//   up_r = Gamma_r dKg_r + a1_r             a1_r = sum_{i<r}  dA[r,i] k_i e^(G_r - G_i)
//   dn_t = e^(G_C - G_t) dKt_t + b1_t       b1_t = sum_{r>t} dA[r,t] k_r e^(G_r - G_t) + sum_{r>=t} dP[r,t] q_r e^(G_r - G_t)
//   dk = up + dn,   dG = q dq + k (up - dn)  (r = t taken out of a2 and b1, where it cancels),   dG_C = e^(G_C) rowsum(dS1 . S0) + sum_t k_t e^(G_C - G_t) dKt_t
//   dlog alpha_t = sum_{r>=t} dG_r + dG_C
//
// (dA needs no product with the inverse: with T = (I + Diag(beta) A)^-1 the chain rule through it,
// -T^T (dVn Y^T) T^T, is -(T^T dVn) (T Diag(beta) Y)^T Diag(beta)^-1 = -Z Vn^T Diag(beta)^-1.)
//
// A wave owns whole 16-channel tiles (all 64 tokens), so everything that is per channel -- the running sum of the
// decay, the decay factors, the sums over tokens that make dlog alpha -- stays in its registers, and S0 and dS1 are
// read as B operands straight from memory, once, a column tile ahead of their products.  Only dO, X and Vn (the operands
// all waves share) and the two C x C results go through LDS: the former 16 value columns at a time in two buffers, so
// that one barrier a part is enough and the next part's rows are on their way while this one is multiplied; the latter
// as fragments in both forms, so that every operand of the second half is one 16-byte read.  The registers (256) allow
// two workgroups a compute unit.
//
// The products with S0 and dS1 and the two C x C ones, three quarters of the kernel's, are formed from bf16 pieces (kda_f32_tile.h):
// a state's fragment meets four token tiles in one or two products and a row's eight channel tiles, so the splitting is spread
// over 192 to 384 cycles of products; dO, X and Vn are split once, by the wave that stages them.  The products of the second half,
// whose factors are formed for one or two uses, stay on the fp32 instruction.
//
// Bounds: at 4 x 4096 tokens x 16 heads 1.5 GB of traffic (0.29 ms at the rate of a large copy), and per wave 25 of the 40 thousand
// cycles of matrix products that the fp32 instruction takes for all of them: 0.49 -> 0.44 ms (two workgroups a compute unit overlap
// the two), 9 x 1 tokens x 32 heads 55 -> 45 us; 2-norm errors of dq 0.75, dk 0.80 and dlog alpha 0.95 of what they were (bf16 inputs and dO,
// mean log alpha -0.18; fp32 0.89, 0.91, 0.98).  32 columns a part leave 30 registers in scratch memory.
#include "kda_f32_tile.h"

namespace kda {
namespace f32 {

constexpr int kGradThreads = 256;
constexpr int kCols = 1;                                     // column tiles of a part
// One operand of a part, [token tile][column tile]: in pieces (X, Vn and an fp32 dO), or bf16 as it stands (a bf16 dO).
constexpr int kPart = 4 * kCols * kSplitFrag;
template <typename T> constexpr int kRowFrag = sizeof(T) == 2 ? kFrag / 2 : kSplitFrag;
template <typename T> constexpr int part_floats() { return 2 * kPart + 4 * kCols * kRowFrag<T>; }
constexpr int kBoth = 2 * kTri * kFrag;                      // dA or dP: its blocks in row form, then in column form
// Inputs of a channel tile on their way to column form, per wave: rows 16 bytes longer than they are, so that rows 4
// apart lie in different banks.
template <typename T> constexpr int turn_row() { return 16 * (int)sizeof(T) + 16; }
template <typename T, typename O> constexpr size_t grad_lds()
{
    const size_t first = (size_t)2 * part_floats<O>() * 4, second = (size_t)(2 * kBoth + kC) * 4 + 4 * kC * turn_row<T>();
    return first > second ? first : second;
}
static_assert(2 * grad_lds<float, float>() <= 160 * 1024, "two workgroups share a compute unit");

// dO: four values of a row as they lie in memory, what of them goes to LDS, and the left factor read from there.  fp32 rows carry
// the scale there; bf16 ones stay as they are, which spares a third of their products, and the scale comes behind the products.
template <typename T> struct RowsOfO;
template <> struct RowsOfO<float> {
    using Factor = Left;
    f32x4 x;
    __device__ __forceinline__ void load(const float *p) { x = ld4(p); }
    __device__ __forceinline__ void put(float *frag, bool live, float scale, int lane) const
    {
        put_pieces(frag, split(live ? x * scale : f32x4{0.f, 0.f, 0.f, 0.f}), lane);
    }
    static __device__ __forceinline__ Factor get(const float *frag, int lane) { Factor f; f.set(get_pieces(frag, lane)); return f; }
    static __device__ __forceinline__ f32x4 scaled(const f32x4 &x, float) { return x; }
};
template <> struct RowsOfO<__hip_bfloat16> {
    using Factor = LeftExact;
    u32x2 x;
    __device__ __forceinline__ void load(const __hip_bfloat16 *p) { x = *reinterpret_cast<const u32x2 *>(p); }
    __device__ __forceinline__ void put(float *frag, bool live, float, int lane) const
    {
        *reinterpret_cast<u32x2 *>(frag + 2 * lane) = live ? x : u32x2{0u, 0u};
    }
    static __device__ __forceinline__ Factor get(const float *frag, int lane) { Factor f; f.set(*reinterpret_cast<const u32x2 *>(frag + 2 * lane)); return f; }
    static __device__ __forceinline__ f32x4 scaled(const f32x4 &x, float scale) { return x * scale; }
};

// kHalves: two workgroups a chunk, each with half of the channel tiles (and the C x C results for itself).
template <typename Tin, typename Tdo, int D, bool kHalves>
__device__ __forceinline__ void gradients(const Tin *__restrict__ q, const Tin *__restrict__ k, const Tin *__restrict__ log_alpha,
                                          const Tin *__restrict__ beta, const Tdo *__restrict__ d_o, const float *__restrict__ S0,
                                          const float *__restrict__ Rw, const float *__restrict__ dS1, const float *__restrict__ Zw,
                                          float *__restrict__ dq, float *__restrict__ dk, float *__restrict__ dv,
                                          float *__restrict__ dla, float *__restrict__ dbeta, const Problem &p)
{
    constexpr int NT = D / 16, TW = NT / 4 / (kHalves ? 2 : 1), NP = NT / kCols;
    const int half = kHalves ? (int)(blockIdx.x & 1) : 0, tile0 = 4 * TW * half;   // its channel tiles: tile0 + 4 tt + w
    extern __shared__ __attribute__((aligned(16))) float smem[];
    Chunk c;
    if (!locate(p.cu, p.num_seqs, p.T, p.H, p.chunks_per_seq, kHalves ? blockIdx.x >> 1 : blockIdx.x, c)) return;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t stride = (int64_t)p.H * D, base = (c.tok0 * p.H + c.h) * (int64_t)D;
    const float *s0 = S0 + c.slot * (int64_t)(D * D) + 4 * lane, *ds1 = dS1 + c.slot * (int64_t)(D * D) + 4 * lane;

    // ---- the products with S0 and dS1, and the two C x C products ----
    f32x4 aq[TW][4] = {}, ak[TW][4] = {}, at[TW][4] = {}, tile[5] = {};      // tiles of dA (u < 10) and dP
    float gc[TW] = {};
    {
        const int tok = 16 * w + m;                                          // staging: this wave's token tile, token m
        const bool live = tok < c.nv;
        const int64_t row = base + (int64_t)(live ? tok : c.nv - 1) * stride;
        const float bt = load_as_float(beta + (c.tok0 + (live ? tok : c.nv - 1)) * p.H + c.h);
        const int64_t rows = token_rows(c.tok0, p.H, c.h, c.nv, D);
        const int n = tile_tokens(c.nv, w);
        const float *rw = Rw + rows + (live ? row_form(w, 0, g, m, n, D) : 0), *zw = Zw + rows + (live ? row_form(w, 0, g, m, n, D) : 0);
        const int step = live ? 16 * n : 0;                                  // floats from a column tile to the next
        using RowO = RowsOfO<Tdo>;
        using FactorO = typename RowO::Factor;
        constexpr int kRowO = kRowFrag<Tdo>, kParts = part_floats<Tdo>();
        RowO go[kCols];
        f32x4 gz[kCols], gr[kCols];
        float db = 0.f;
        auto fetch = [&](int pt) __attribute__((always_inline)) {
#pragma unroll
            for (int cg = 0; cg < kCols; ++cg) {
                go[cg].load(d_o + row + 16 * (kCols * pt + cg) + 4 * g);
                gz[cg] = ld4(zw + (kCols * pt + cg) * step);
                gr[cg] = ld4(rw + (kCols * pt + cg) * step);
            }
        };
        // (in a buffer: X, Vn, dO)
        auto commit = [&](int pt, float *buf) __attribute__((always_inline)) {
#pragma unroll
            for (int cg = 0; cg < kCols; ++cg) {
                const f32x4 x = bt * gz[cg], zero = {0.f, 0.f, 0.f, 0.f};
                float *f = buf + (kCols * w + cg) * kSplitFrag;
                put_pieces(f, split(live ? x : zero), lane);
                put_pieces(f + kPart, split(live ? bt * gr[cg] : zero), lane);
                go[cg].put(buf + 2 * kPart + (kCols * w + cg) * kRowO, live, p.scale, lane);
                if (live && half == 0) st4(dv + row + 16 * (kCols * pt + cg) + 4 * g, x);
                db += gz[cg][0] * gr[cg][0] + gz[cg][1] * gr[cg][1] + gz[cg][2] * gr[cg][2] + gz[cg][3] * gr[cg][3];
            }
        };
        f32x4 bs[TW], bd[TW];
        auto fetch_states = [&](f32x4 (&to)[TW], const float *from, int ct) __attribute__((always_inline)) {
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) to[tt] = ld4(from + ((tile0 + 4 * tt + w) * NT + ct) * kFrag);
        };
        fetch(0);
        fetch_states(bs, s0, 0);
        fetch_states(bd, ds1, 0);
        pin_memory_order();
        commit(0, smem);
        fetch(1);
        lds_barrier();
#pragma unroll 1
        for (int pt = 0; pt < NP; ++pt) {
            const float *buf = smem + (pt & 1) * kParts;
#pragma unroll
            for (int cg = 0; cg < kCols; ++cg) {
                const int next = kCols * pt + cg + 1 < NT ? kCols * pt + cg + 1 : NT - 1;    // (the last one fetches its own again)
                Right b[TW];
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) {
                    gc[tt] += bs[tt][0] * bd[tt][0] + bs[tt][1] * bd[tt][1] + bs[tt][2] * bd[tt][2] + bs[tt][3] * bd[tt][3];
                    b[tt].set(split(bs[tt]));
                }
                fetch_states(bs, s0, next);
                pin_memory_order();
#pragma unroll
                for (int R = 0; R < 4; ++R) {
                    pin_memory_order();
                    Left ax;
                    ax.set(get_pieces(buf + (kCols * R + cg) * kSplitFrag, lane));
                    const FactorO ao = RowO::get(buf + 2 * kPart + (kCols * R + cg) * kRowO, lane);
#pragma unroll
                    for (int k = 0; k < Left::kSteps; ++k) {
#pragma unroll
                        for (int tt = 0; tt < TW; ++tt) ak[tt][R] = ax.step(k, b[tt], ak[tt][R]);
                        if (k < FactorO::kSteps) {
#pragma unroll
                            for (int tt = 0; tt < TW; ++tt) aq[tt][R] = ao.step(k, b[tt], aq[tt][R]);
                        }
                    }
                }
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) b[tt].set(split(bd[tt]));
                fetch_states(bd, ds1, next);
                pin_memory_order();
#pragma unroll
                for (int R = 0; R < 4; ++R) {
                    pin_memory_order();
                    Left av;
                    av.set(get_pieces(buf + kPart + (kCols * R + cg) * kSplitFrag, lane));
#pragma unroll
                    for (int k = 0; k < Left::kSteps; ++k)
#pragma unroll
                        for (int tt = 0; tt < TW; ++tt) at[tt][R] = av.step(k, b[tt], at[tt][R]);
                }
            }
#pragma unroll
            for (int cg = 0; cg < kCols; ++cg)
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const bool inA = i < 2 || (i == 2 && w < 2);             // u < 10
                    const int u = w + 4 * i, bl = inA ? u : u - 10;
                    const int R = bl >= 6 ? 3 : bl >= 3 ? 2 : bl >= 1 ? 1 : 0, I = bl - tri(R, 0);
                    pin_memory_order();
                    Right bv;
                    bv.set(get_pieces(buf + kPart + (kCols * I + cg) * kSplitFrag, lane));
                    if (inA) {
                        Left ax;
                        ax.set(get_pieces(buf + (kCols * R + cg) * kSplitFrag, lane));
#pragma unroll
                        for (int k = 0; k < Left::kSteps; ++k) tile[i] = ax.step(k, bv, tile[i]);
                    } else {
                        const FactorO ao = RowO::get(buf + 2 * kPart + (kCols * R + cg) * kRowO, lane);
#pragma unroll
                        for (int k = 0; k < FactorO::kSteps; ++k) tile[i] = ao.step(k, bv, tile[i]);
                    }
                }
            if (pt + 1 < NP) {
                commit(pt + 1, smem + ((pt + 1) & 1) * kParts);              // (last read before the previous barrier)
                if (pt + 2 < NP) fetch(pt + 2);
                lds_barrier();
            }
        }
#pragma unroll
        for (int tt = 0; tt < TW; ++tt)
#pragma unroll
            for (int R = 0; R < 4; ++R) aq[tt][R] = RowO::scaled(aq[tt][R], p.scale);
#pragma unroll
        for (int i = 0; i < 5; ++i)
            if (i > 2 || (i == 2 && w >= 2)) tile[i] = RowO::scaled(tile[i], p.scale);
        db += __shfl_xor(db, 16);
        db += __shfl_xor(db, 32);
        if (g == 0 && live && half == 0) dbeta[(c.tok0 + tok) * p.H + c.h] = db;
    }
    TileFetch<Tin> fg, fk, fq;
    auto fetch_inputs = [&](int tt) __attribute__((always_inline)) {
        const int64_t at0 = base + 16 * (tile0 + 4 * tt + w);
        int l = lane;
        asm volatile("" : "+v"(l));                                          // (addresses formed here, not kept from the first tile)
        fg.fetch(log_alpha + at0, stride, c.nv, l);
        fk.fetch(k + at0, stride, c.nv, l);
        fq.fetch(q + at0, stride, c.nv, l);
    };
    fetch_inputs(0);
    lds_barrier();
    const int turned = 4 * turned_lane(lane);
    float *sA = smem, *sP = smem + kBoth, *sD = smem + 2 * kBoth;            // sD: the diagonal of dP
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int u = w + 4 * i, b = u < 10 ? u : u - 10;
        const int R = b >= 6 ? 3 : b >= 3 ? 2 : b >= 1 ? 1 : 0, I = b - tri(R, 0);
        f32x4 x = u < 10 ? -tile[i] : tile[i];
        if (R == I) {
            const float d01 = m & 1 ? x[1] : x[0], d23 = m & 1 ? x[3] : x[2];
            if (u >= 10 && m >> 2 == g) sD[16 * R + m] = m & 2 ? d23 : d01;
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = m >= 4 * g + j ? 0.f : x[j];
        }
        float *dst = (u < 10 ? sA : sP) + b * kFrag;
        st4(dst + turned, quad_transpose(x, lane));
        st4(dst + kTri * kFrag + 4 * lane, x);
    }
    lds_barrier();
    const float *rowA = sA + 4 * lane, *rowP = sP + 4 * lane, *colA = rowA + kTri * kFrag, *colP = rowP + kTri * kFrag;
    char *turn = reinterpret_cast<char *>(sD + kC) + w * (kC * turn_row<Tin>());

    // ---- decay terms and results, a 16-channel tile at a time ----
    auto finish = [&](int tt, f32x4 (&aq)[4], f32x4 (&ak)[4], f32x4 (&at)[4], float gc) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");                                       // (one tile's inputs in registers at a time)
        f32x4 kk[4], qq[4], pf[4], nf[4];
        Decay d;
        fg.turn(d.x, turn, turn_row<Tin>(), c.nv, lane);
        fk.turn(kk, turn, turn_row<Tin>(), c.nv, lane);
        fq.turn(qq, turn, turn_row<Tin>(), c.nv, lane);
        sum_decay(d, lane);
        float run = 0.f;
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            const Exponents x(d, R);
            const f32x4 gam = exp2_4(x.start);
            aq[R] *= gam;
            ak[R] *= -gam;
            at[R] *= exp2_4(x.end);
            pf[R] = exp2_4(x.row);
            nf[R] = exp2_4(x.column);
            const f32x4 kt = kk[R] * at[R];
            run += kt[0] + kt[1] + kt[2] + kt[3];
        }
        run = fmaf(gc, fast_exp2(d.whole()), run);
        run += __shfl_xor(run, 16);
        run += __shfl_xor(run, 32);                                          // dG_C
        float across[6];                                                     // decay between the blocks of a pair
#pragma unroll
        for (int R = 1; R < 4; ++R)
#pragma unroll
            for (int I = 0; I < R; ++I) across[R * (R - 1) / 2 + I] = fast_exp2(d.across(R, I));
#pragma unroll
        for (int i = 0; i < 6; ++i) asm volatile("" : "+v"(across[i]));          // (kept, not formed again from the sums at each use)
        const bool any_strong = __any(d.strong());
#pragma unroll
        for (int R = 3; R >= 0; --R) {
            // (the diagonal block's products apart: in one sum the others are rounded at its size, and the sums over tokens below,
            // in which most of a1 and b1 cancel, collect it: dlog alpha 6.7e-7 -> 5.3e-7)
            const f32x4 none = {0.f, 0.f, 0.f, 0.f};
            f32x4 a1 = none, a2 = none, b1 = none, a1d = none, a2d = none, b1d = none;
#pragma unroll
            for (int I = 0; I < R; ++I) {
                const f32x4 b = kk[I] * nf[I] * across[R * (R - 1) / 2 + I];
                a1 = mfma16(ld4(rowA + tri(R, I) * kFrag), b, a1);
                a2 = mfma16(ld4(rowP + tri(R, I) * kFrag), b, a2);
            }
            {
                const f32x4 b = d.weak[R] ? kk[R] * nf[R] : none, x = d.weak[R] ? pf[R] : none;
                a1d = mfma16(ld4(rowA + tri(R, R) * kFrag), b, a1d);
                a2d = mfma16(ld4(rowP + tri(R, R) * kFrag), b, a2d);
                b1d = mfma16(ld4(colA + tri(R, R) * kFrag), x * kk[R], b1d);
                b1d = mfma16(ld4(colP + tri(R, R) * kFrag), x * qq[R], b1d);
            }
#pragma unroll
            for (int B = R + 1; B < 4; ++B) {
                const f32x4 x = pf[B] * across[B * (B - 1) / 2 + R];
                b1 = mfma16(ld4(colA + tri(B, R) * kFrag), x * kk[B], b1);
                b1 = mfma16(ld4(colP + tri(B, R) * kFrag), x * qq[B], b1);
            }
            a1 = (a1 + a1d) * pf[R]; a2 = (a2 + a2d) * pf[R]; b1 = (b1 + b1d) * nf[R];
            if (any_strong) {
                // strong channels of this block, pair by pair (the products above left their diagonal block out); G again
                // from the input: kept, it would cost every chunk registers
                Decay e;
                load_tile(e.x, log_alpha + base + 16 * (tile0 + 4 * tt + w) + m, stride, c.nv, g);
                sum_decay(e, lane);
                const f32x4 eL = e.in_block(R);
                const bool mine = !d.weak[R];
#pragma unroll 1
                for (int gi = 0; gi < 4; ++gi)
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    const int i = 4 * gi + ii, src = 16 * gi + m;
                    const float Gi = __shfl(eL[ii], src), ki = __shfl(kk[R][ii], src), qi = __shfl(qq[R][ii], src);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int t = 4 * g + j;
                        const float x = mine ? fast_exp2(i <= t ? fminf(eL[j] - Gi, 0.f) : fminf(Gi - eL[j], 0.f)) : 0.f;
                        const float *row = sA + tri(R, R) * kFrag + 4 * (t + 16 * gi) + ii;      // dA[t][i], dA[i][t] in row form
                        const float *cl = sA + tri(R, R) * kFrag + 4 * (i + 16 * g) + j;
                        if (i <= t) {                                        // (the diagonals are zero)
                            a1[j] = fmaf(row[0] * ki, x, a1[j]);
                            a2[j] = fmaf(row[kBoth] * ki, x, a2[j]);
                        }
                        if (i >= t) b1[j] = fmaf(fmaf(cl[0], ki, cl[kBoth] * qi), x, b1[j]);
                    }
                }
            }
            // (dP's diagonal stays out of s: q_r (dP_rr k_r) - k_r (dP_rr q_r) is nothing, and its rounding is most of dlog alpha's
            // error where the decay is fast: 2.7e-6 -> 0.7e-6 at a mean log alpha of -2.1, 5.3e-7 -> 4.8e-7 at -0.18)
            f32x4 gq = aq[R] + a2;
            const f32x4 up = ak[R] + a1, dn = at[R] + b1;
            f32x4 s = qq[R] * gq + kk[R] * (up - dn), gk = up + dn;
            pin_memory_order();
            const f32x4 diag = ld4(sD + 16 * R + 4 * g);
            gq += diag * kk[R];
            gk += diag * qq[R];
            // dlog alpha: sums over the tokens behind, inside the lane, across the four lane groups, over the blocks
            s[2] += s[3]; s[1] += s[2]; s[0] += s[1];
            float tot = s[0], u = __shfl_down(tot, 16);
            if (g <= 2) tot += u;
            u = __shfl_down(tot, 32);
            if (g <= 1) tot += u;
            u = __shfl_down(tot, 16);
            const float behind = run + (g <= 2 ? u : 0.f);
            run += __shfl(tot, m);
            const f32x4 tq = quad_transpose(gq, lane), tk = quad_transpose(gk, lane), tg = quad_transpose(s + behind, lane);
            const int r = 16 * R + 4 * g + (lane & 3);
            if (r < c.nv) {
                const int64_t to = base + r * stride + 16 * (tile0 + 4 * tt + w) + (lane & 12);
                st4(dq + to, tq); st4(dk + to, tk); st4(dla + to, tg);
            }
            if (tt + 1 < TW && R == (sizeof(Tin) == 2 ? 2 : 1)) fetch_inputs(tt + 1);    // (into what this tile has freed)
        }
    };
    finish(0, aq[0], ak[0], at[0], gc[0]);
    if (TW > 1) finish(TW - 1, aq[TW - 1], ak[TW - 1], at[TW - 1], gc[TW - 1]);
}

template <typename Tin, typename Tdo, int D>
__global__ __launch_bounds__(kGradThreads, 2)
void kda_bwd_gradients_kernel(const Tin *__restrict__ q, const Tin *__restrict__ k, const Tin *__restrict__ log_alpha,
                              const Tin *__restrict__ beta, const Tdo *__restrict__ d_o, const float *__restrict__ S0,
                              const float *__restrict__ Rw, const float *__restrict__ dS1, const float *__restrict__ Zw,
                              float *__restrict__ dq, float *__restrict__ dk, float *__restrict__ dv,
                              float *__restrict__ dla, float *__restrict__ dbeta, const Problem p)
{
    gradients<Tin, Tdo, D, false>(q, k, log_alpha, beta, d_o, S0, Rw, dS1, Zw, dq, dk, dv, dla, dbeta, p);
}

template <typename Tin, typename Tdo, int D>
__global__ __launch_bounds__(kGradThreads, 2)
void kda_bwd_half_gradients_kernel(const Tin *__restrict__ q, const Tin *__restrict__ k, const Tin *__restrict__ log_alpha,
                                   const Tin *__restrict__ beta, const Tdo *__restrict__ d_o, const float *__restrict__ S0,
                                   const float *__restrict__ Rw, const float *__restrict__ dS1, const float *__restrict__ Zw,
                                   float *__restrict__ dq, float *__restrict__ dk, float *__restrict__ dv,
                                   float *__restrict__ dla, float *__restrict__ dbeta, const Problem p)
{
    gradients<Tin, Tdo, D, true>(q, k, log_alpha, beta, d_o, S0, Rw, dS1, Zw, dq, dk, dv, dla, dbeta, p);
}

template <typename Tin, typename Tdo, int D>
kda_status launch_gradients(const Problem &p, const Tin *q, const Tin *k, const Tin *log_alpha, const Tin *beta, const Tdo *d_o,
                            const float *S0, const float *R, const float *dS1, const float *Z, float *dq, float *dk, float *dv,
                            float *dla, float *dbeta, int compute_units, hipStream_t stream)
{
    const int64_t blocks = p.slots * p.H;
    if (blocks == 0) return KDA_OK;
    if (blocks > 0x7fffffffLL) return fail(KDA_ERR_UNSUPPORTED, "%lld chunks in one call", (long long)blocks);
    auto launch = [&](auto kern, int64_t workgroups) {
        hipLaunchKernelGGL(kern, dim3((unsigned)workgroups), dim3(kGradThreads), (grad_lds<Tin, Tdo>()), stream, q, k, log_alpha, beta,
                           d_o, S0, R, dS1, Z, dq, dk, dv, dla, dbeta, p);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? KDA_OK : fail(KDA_ERR_LAUNCH, "kda_bwd_gradients: %s", hipGetErrorString(e));
    };
    // Up to one chunk a compute unit the time is that of one workgroup, half of which is spent on its channel tiles one after the
    // other: two share them (whole pass, d 128, whole / halves: 8 chunks 51.7 / 43.2 us, 32 57.7 / 48.7, 64 64.6 / 54.1, 128 76.8 / 67.6, 256
    // 103.9 / 101.9; beyond, what both do twice counts: 384 149.9 / 150.9, 512 171.6 / 175.8).  At d 64 a wave has one tile as it is.
    if constexpr (D == 128)
        if (blocks <= compute_units) return launch(kda_bwd_half_gradients_kernel<Tin, Tdo, D>, 2 * blocks);
    return launch(kda_bwd_gradients_kernel<Tin, Tdo, D>, blocks);
}

#define KDA_GRAD(T, O, DD) template kda_status launch_gradients<T, O, DD>(const Problem &, const T *, const T *, const T *, const T *, \
    const O *, const float *, const float *, const float *, const float *, float *, float *, float *, float *, float *, int, hipStream_t)
KDA_GRAD(float, float, 64);
KDA_GRAD(float, float, 128);
KDA_GRAD(__hip_bfloat16, float, 64);
KDA_GRAD(__hip_bfloat16, float, 128);
KDA_GRAD(__hip_bfloat16, __hip_bfloat16, 64);
KDA_GRAD(__hip_bfloat16, __hip_bfloat16, 128);
#undef KDA_GRAD

}  // namespace f32
}  // namespace kda
