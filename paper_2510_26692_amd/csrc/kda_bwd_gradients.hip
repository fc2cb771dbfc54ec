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
//   dk = up + dn,   dG = q dq + k (up - dn),   dG_C = e^(G_C) rowsum(dS1 . S0) + sum_t k_t e^(G_C - G_t) dKt_t
//   dlog alpha_t = sum_{r>=t} dG_r + dG_C
//
// (dA needs no product with the inverse: with T = (I + Diag(beta) A)^-1 the chain rule through it,
// -T^T (dVn Y^T) T^T, is -(T^T dVn) (T Diag(beta) Y)^T Diag(beta)^-1 = -Z Vn^T Diag(beta)^-1.)
//
// A wave owns whole 16-channel tiles (all 64 tokens), so everything that is per channel -- the running sum of the
// decay, the decay factors, the sums over tokens that make dlog alpha -- stays in its registers, and S0 and dS1 are
// read as B operands straight from memory, once.  Only dO, X and Vn (the operands all waves share) and the two C x C
// results go through LDS: 48 KiB, half of the value columns at a time, so that two workgroups share a compute unit
// and one loads while the other multiplies.
#include "kda_f32_tile.h"

namespace kda {
namespace f32 {

constexpr int kGradThreads = 256;
constexpr int kPart = 16 * kFrag;                            // one operand, 64 value columns: [token tile][column tile]
constexpr size_t kGradLds = (size_t)(3 * kPart) * 4;
static_assert(2 * kC * kLdT <= 3 * kPart, "the C x C tiles take the operands' place");

__device__ __forceinline__ f32x4 load4(const float *p) { return ld4(p); }
__device__ __forceinline__ f32x4 load4(const __hip_bfloat16 *p)
{
    const uint2 u = *reinterpret_cast<const uint2 *>(p);
    f32x4 x;
    float a, b;
    unpack_bf16x2(u.x, a, b); x[0] = a; x[1] = b;
    unpack_bf16x2(u.y, a, b); x[2] = a; x[3] = b;
    return x;
}

template <typename Tin, typename Tdo, int D>
__global__ __launch_bounds__(kGradThreads, 2)
void kda_bwd_gradients_kernel(const Tin *__restrict__ q, const Tin *__restrict__ k, const Tin *__restrict__ log_alpha,
                              const Tin *__restrict__ beta, const Tdo *__restrict__ d_o, const float *__restrict__ S0,
                              const float *__restrict__ Rw, const float *__restrict__ dS1, const float *__restrict__ Zw,
                              float *__restrict__ dq, float *__restrict__ dk, float *__restrict__ dv,
                              float *__restrict__ dla, float *__restrict__ dbeta, const Problem p)
{
    constexpr int NT = D / 16, TW = NT / 4, NH = D / 64;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *sO = smem, *sX = sO + kPart, *sV = sX + kPart;    // later: dA and dP, [64][kLdT] each
    Chunk c;
    if (!locate(p.cu, p.num_seqs, p.T, p.H, p.chunks_per_seq, blockIdx.x, c)) return;
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
        f32x4 go[4], gz[4], gr[4];
        float db = 0.f;
        auto fetch = [&](int hf) __attribute__((always_inline)) {
#pragma unroll
            for (int cg = 0; cg < 4; ++cg) {
                go[cg] = load4(d_o + row + 64 * hf + 16 * cg + 4 * g);
                gz[cg] = ld4(zw + (4 * hf + cg) * step);
                gr[cg] = ld4(rw + (4 * hf + cg) * step);
            }
        };
        fetch(0);
#pragma unroll 1
        for (int hf = 0; hf < NH; ++hf) {
            if (hf) lds_barrier();                                           // the previous half is read
#pragma unroll
            for (int cg = 0; cg < 4; ++cg) {
                const f32x4 x = bt * gz[cg], zero = {0.f, 0.f, 0.f, 0.f};
                const int f = (4 * w + cg) * kFrag + 4 * lane;
                st4(sO + f, live ? go[cg] * p.scale : zero);
                st4(sX + f, live ? x : zero);
                st4(sV + f, live ? bt * gr[cg] : zero);
                if (live) st4(dv + row + 64 * hf + 16 * cg + 4 * g, x);
                db += gz[cg][0] * gr[cg][0] + gz[cg][1] * gr[cg][1] + gz[cg][2] * gr[cg][2] + gz[cg][3] * gr[cg][3];
            }
            lds_barrier();
            if (hf + 1 < NH) fetch(hf + 1);
#pragma unroll
            for (int cg = 0; cg < 4; ++cg) {
                f32x4 bs[TW], bd[TW];
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) {
                    const int f = ((4 * tt + w) * NT + 4 * hf + cg) * kFrag;
                    bs[tt] = ld4(s0 + f); bd[tt] = ld4(ds1 + f);
                }
#pragma unroll
                for (int R = 0; R < 4; ++R) {
                    const int f = (4 * R + cg) * kFrag + 4 * lane;
                    const f32x4 ao = ld4(sO + f), ax = ld4(sX + f), av = ld4(sV + f);
#pragma unroll
                    for (int tt = 0; tt < TW; ++tt) {
                        aq[tt][R] = mfma16(ao, bs[tt], aq[tt][R]);
                        ak[tt][R] = mfma16(ax, bs[tt], ak[tt][R]);
                        at[tt][R] = mfma16(av, bd[tt], at[tt][R]);
                    }
                }
#pragma unroll
                for (int tt = 0; tt < TW; ++tt)
                    gc[tt] += bs[tt][0] * bd[tt][0] + bs[tt][1] * bd[tt][1] + bs[tt][2] * bd[tt][2] + bs[tt][3] * bd[tt][3];
            }
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                const int u = w + 4 * i, b = u < 10 ? u : u - 10;
                const int R = b >= 6 ? 3 : b >= 3 ? 2 : b >= 1 ? 1 : 0, I = b - tri(R, 0);
                const float *pa = (u < 10 ? sX : sO) + 4 * R * kFrag + 4 * lane, *pb = sV + 4 * I * kFrag + 4 * lane;
#pragma unroll
                for (int cg = 0; cg < 4; ++cg) tile[i] = mfma16(ld4(pa + cg * kFrag), ld4(pb + cg * kFrag), tile[i]);
            }
        }
        db += __shfl_xor(db, 16);
        db += __shfl_xor(db, 32);
        if (g == 0 && live) dbeta[(c.tok0 + tok) * p.H + c.h] = db;
    }
    lds_barrier();
    float *sA = smem, *sP = smem + kC * kLdT;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int u = w + 4 * i, b = u < 10 ? u : u - 10;
        const int R = b >= 6 ? 3 : b >= 3 ? 2 : b >= 1 ? 1 : 0, I = b - tri(R, 0);
        float *dst = (u < 10 ? sA : sP) + (16 * R + 4 * g) * kLdT + 16 * I + m;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float x = u < 10 ? -tile[i][j] : tile[i][j];
            if (R == I && (m > 4 * g + j || (u < 10 && m == 4 * g + j))) x = 0.f;
            dst[j * kLdT] = x;
        }
    }
    lds_barrier();

    // ---- decay terms and results, a 16-channel tile at a time ----
    auto finish = [&](int tt, f32x4 (&aq)[4], f32x4 (&ak)[4], f32x4 (&at)[4], float gc) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");                                       // (one tile's inputs in registers at a time)
        const int64_t col = base + 16 * (4 * tt + w) + m;
        f32x4 kk[4], qq[4], pf[4], nf[4];
        Decay d;
        load_tile(d.G, log_alpha + col, stride, c.nv, g);
        load_tile(kk, k + col, stride, c.nv, g);
        load_tile(qq, q + col, stride, c.nv, g);
        running_decay(d, lane);
        float run = 0.f;
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            const f32x4 gam = exp2_4(d.G[R]);
            aq[R] *= gam;
            ak[R] *= -gam;
            at[R] *= exp2_4(d.E[3] - d.G[R]);
            pf[R] = exp2_4(d.G[R] - d.pref[R]);
            nf[R] = exp2_4(d.nref[R] - d.G[R]);
            const f32x4 kt = kk[R] * at[R];
            run += kt[0] + kt[1] + kt[2] + kt[3];
        }
        run = fmaf(gc, fast_exp2(d.E[3]), run);
        run += __shfl_xor(run, 16);
        run += __shfl_xor(run, 32);                                          // dG_C
        const bool any_strong = __any(d.strong);
#pragma unroll
        for (int R = 3; R >= 0; --R) {
            f32x4 a1 = {0.f, 0.f, 0.f, 0.f}, a2 = a1, b1 = a1;
#pragma unroll
            for (int I = 0; I <= R; ++I) {
                const f32x4 b = kk[I] * nf[I] * (I == R ? d.fdiag[R] : fast_exp2(d.pref[R] - d.nref[I]));
                const int f = (16 * R + m) * kLdT + 16 * I + 4 * g;
                a1 = mfma16(ld4(sA + f), b, a1);
                a2 = mfma16(ld4(sP + f), b, a2);
            }
#pragma unroll
            for (int B = R; B < 4; ++B) {
                const f32x4 x = pf[B] * (B == R ? d.fdiag[R] : fast_exp2(d.pref[B] - d.nref[R]));
                const int f = (16 * B + 4 * g) * kLdT + 16 * R + m;
                b1 = mfma16(f32x4{sA[f], sA[f + kLdT], sA[f + 2 * kLdT], sA[f + 3 * kLdT]}, x * kk[B], b1);
                b1 = mfma16(f32x4{sP[f], sP[f + kLdT], sP[f + 2 * kLdT], sP[f + 3 * kLdT]}, x * qq[B], b1);
            }
            a1 *= pf[R]; a2 *= pf[R]; b1 *= nf[R];
            if (any_strong) {
                // strong channels of this block, pair by pair (the products above left their diagonal block out)
                const bool mine = d.fdiag[R] == 0.f;
#pragma unroll 1
                for (int gi = 0; gi < 4; ++gi)
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    const int i = 4 * gi + ii, src = 16 * gi + m;
                    const float Gi = __shfl(d.G[R][ii], src), ki = __shfl(kk[R][ii], src), qi = __shfl(qq[R][ii], src);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int t = 4 * g + j;
                        const float e = mine ? fast_exp2(i <= t ? fminf(d.G[R][j] - Gi, 0.f) : fminf(Gi - d.G[R][j], 0.f)) : 0.f;
                        const float *row = sA + (16 * R + t) * kLdT + 16 * R + i, *cl = sA + (16 * R + i) * kLdT + 16 * R + t;
                        if (i <= t) {                                        // (dA's diagonal is zero)
                            a1[j] = fmaf(row[0] * ki, e, a1[j]);
                            a2[j] = fmaf(row[kC * kLdT] * ki, e, a2[j]);
                        }
                        if (i >= t) b1[j] = fmaf(fmaf(cl[0], ki, cl[kC * kLdT] * qi), e, b1[j]);
                    }
                }
            }
            const f32x4 gq = aq[R] + a2, up = ak[R] + a1, dn = at[R] + b1, gk = up + dn;
            f32x4 s = qq[R] * gq + kk[R] * (up - dn);
            // dlog alpha: sums over the tokens behind, inside the lane, across the four lane groups, over the blocks
            s[2] += s[3]; s[1] += s[2]; s[0] += s[1];
            float tot = s[0], u = __shfl_down(tot, 16);
            if (g <= 2) tot += u;
            u = __shfl_down(tot, 32);
            if (g <= 1) tot += u;
            u = __shfl_down(tot, 16);
            const float behind = run + (g <= 2 ? u : 0.f);
            run += __shfl(tot, m);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * R + 4 * g + j;
                if (r < c.nv) {
                    const int64_t at_ = col + r * stride;
                    dq[at_] = gq[j]; dk[at_] = gk[j]; dla[at_] = s[j] + behind;
                }
            }
        }
    };
    finish(0, aq[0], ak[0], at[0], gc[0]);
    if (TW > 1) finish(TW - 1, aq[TW - 1], ak[TW - 1], at[TW - 1], gc[TW - 1]);
}

template <typename Tin, typename Tdo, int D>
kda_status launch_gradients(const Problem &p, const Tin *q, const Tin *k, const Tin *log_alpha, const Tin *beta, const Tdo *d_o,
                            const float *S0, const float *R, const float *dS1, const float *Z, float *dq, float *dk, float *dv,
                            float *dla, float *dbeta, hipStream_t stream)
{
    const int64_t blocks = p.slots * p.H;
    if (blocks == 0) return KDA_OK;
    if (blocks > 0x7fffffffLL) return fail(KDA_ERR_UNSUPPORTED, "%lld chunks in one call", (long long)blocks);
    hipLaunchKernelGGL((kda_bwd_gradients_kernel<Tin, Tdo, D>), dim3((unsigned)blocks), dim3(kGradThreads), kGradLds, stream, q, k,
                       log_alpha, beta, d_o, S0, R, dS1, Z, dq, dk, dv, dla, dbeta, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? KDA_OK : fail(KDA_ERR_LAUNCH, "kda_bwd_gradients: %s", hipGetErrorString(e));
}

#define KDA_GRAD(T, O, DD) template kda_status launch_gradients<T, O, DD>(const Problem &, const T *, const T *, const T *, const T *, \
    const O *, const float *, const float *, const float *, const float *, float *, float *, float *, float *, float *, hipStream_t)
KDA_GRAD(float, float, 64);
KDA_GRAD(float, float, 128);
KDA_GRAD(__hip_bfloat16, float, 64);
KDA_GRAD(__hip_bfloat16, float, 128);
KDA_GRAD(__hip_bfloat16, __hip_bfloat16, 64);
KDA_GRAD(__hip_bfloat16, __hip_bfloat16, 128);
#undef KDA_GRAD

}  // namespace f32
}  // namespace kda
