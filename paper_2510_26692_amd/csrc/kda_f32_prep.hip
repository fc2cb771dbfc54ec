// Per-chunk kernel of the fp32 path (prefill of fp32 inputs and backward pass): everything of a chunk that does
// not depend on the state, one workgroup of four waves per (chunk, head).
//
//   A[r,i] = sum_d k_r,d k_i,d e^(G_r,d - G_i,d), i < r     P[r,i] likewise with q_r, i <= r
//   Q = A (I + Diag(beta) A)^-1
//
// With Y = V - (Gamma.K) S0, the residual R = V - S^T k of the delta rule obeys (I + A Diag(beta)) R = Y, and
// (I + A Diag(beta))^-1 = I - Q Diag(beta), (I + Diag(beta) A)^-1 = I - Diag(beta) Q with the same Q: the walks
// (kda_f32_walk.hip) need one C x C matrix for both directions, and no division by beta appears anywhere.
#include <type_traits>

#include "kda_f32_tile.h"

namespace kda {
namespace f32 {

constexpr int kPrepThreads = 256;
constexpr int kPairs = 6;                                    // pairs of different token blocks
constexpr size_t kPrepLds = (size_t)(3 * kC * kLdT + kPairs * 64 + kC) * 4;
static_assert(3 * kPrepLds <= 160 * 1024, "three workgroups share a compute unit");

// Four waves; the channels are taken 64 at a time, 16 per wave.  LDS: Kp = k 2^(G - pref), Qp = q 2^(G - pref) and
// Kn = k 2^(nref - G) of those 64 channels, 51 KiB, so that three workgroups share a compute unit.  The inputs of the next
// 64 channels are on their way while the products of these are formed.
template <typename Tin, int D, bool kRows>
__global__ __launch_bounds__(kPrepThreads, 3)
void kda_f32_prep_kernel(const Tin *__restrict__ q, const Tin *__restrict__ k, const Tin *__restrict__ log_alpha,
                         const Tin *__restrict__ beta, float *__restrict__ slots, const Problem p)
{
    using SL = Slot<D>;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *sKp = smem, *sQp = sKp + kC * kLdT, *sKn = sQp + kC * kLdT;
    float *sF = sKn + kC * kLdT;                             // [kPairs][64]: decay between the blocks of a pair
    float *sBeta = sF + kPairs * 64;

    Chunk c;
    if (!locate(p.cu, p.num_seqs, p.T, p.H, p.chunks_per_seq, blockIdx.x, c)) return;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t stride = (int64_t)p.H * D, base = (c.tok0 * p.H + c.h) * (int64_t)D;
    float *slot = slots + c.slot * SL::kFloats;
    // (kRows: the operands that the forward walk multiplies from the left, in its order)
    auto st = [&](float *frag, const f32x4 &x) __attribute__((always_inline)) {
        if (kRows) st4(frag + 4 * turned_lane(lane), quad_transpose(x, lane));
        else st4(frag + 4 * lane, x);
    };
    if (tid < kC) {
        const float b = tid < c.nv ? load_as_float(beta + (c.tok0 + tid) * p.H + c.h) : 0.f;
        sBeta[tid] = b;
        slot[SL::kBeta + tid] = b;
    }

    // tiles of A (u < 10) and P (u >= 10), five per wave
    f32x4 acc[5] = {};
    auto block_of = [](int b, int &R, int &I) { R = b >= 6 ? 3 : b >= 3 ? 2 : b >= 1 ? 1 : 0; I = b - tri(R, 0); };
    auto pair_of = [](int R, int I) { return R * (R - 1) / 2 + I; };
    TileFetch<Tin> fg, fk, fq;
    auto fetch = [&](int t) __attribute__((always_inline)) {
        fg.fetch(log_alpha + base + 16 * t, stride, c.nv, lane);
        fk.fetch(k + base + 16 * t, stride, c.nv, lane);
        fq.fetch(q + base + 16 * t, stride, c.nv, lane);
    };
    fetch(w);
    bool strong = false;
#pragma unroll
    for (int hf = 0; hf < D / 64; ++hf) {
        const int t = 4 * hf + w;
        f32x4 kk[4], qq[4];
        Decay d;
        if (hf) lds_barrier();                               // the previous channels' tiles are read
        char *pg = reinterpret_cast<char *>(sKn + 16 * w), *pk = reinterpret_cast<char *>(sKp + 16 * w),
             *pq = reinterpret_cast<char *>(sQp + 16 * w);
        fg.put(pg, 4 * kLdT, c.nv, lane);
        fk.put(pk, 4 * kLdT, c.nv, lane);
        fq.put(pq, 4 * kLdT, c.nv, lane);
        wave_lds_fence();
        fg.get(d.x, pg, 4 * kLdT, lane);
        fk.get(kk, pk, 4 * kLdT, lane);
        fq.get(qq, pq, 4 * kLdT, lane);
        wave_lds_fence();
        sum_decay(d, lane);
        strong |= d.strong();
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            const Exponents x(d, R);
            const f32x4 gam = exp2_4(x.start);
            float *frag = slot + (R * SL::kTiles + t) * kFrag;
            st(frag + SL::kKg, kk[R] * gam);
            st(frag + SL::kQg, qq[R] * gam);
            st4(frag + SL::kKt + 4 * lane, kk[R] * exp2_4(x.end));
            const f32x4 pf = exp2_4(x.row), nf = exp2_4(x.column);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int at = (16 * R + 4 * g + j) * kLdT + 16 * w + m;
                sKp[at] = kk[R][j] * pf[j];
                sQp[at] = qq[R][j] * pf[j];
                sKn[at] = kk[R][j] * nf[j];
            }
            __builtin_amdgcn_sched_barrier(0);               // (one block's values in registers at a time)
        }
        if (g == 0) {
            slot[SL::kGc + 16 * t + m] = fast_exp2(d.whole());
#pragma unroll
            for (int R = 1; R < 4; ++R)
#pragma unroll
                for (int I = 0; I < R; ++I) sF[pair_of(R, I) * 64 + 16 * w + m] = fast_exp2(d.across(R, I));
        }
        pin_memory_order();
        if (4 * hf + 4 < SL::kTiles) {                       // (no earlier: this tile's values need the registers)
            int next = t + 4;
            asm volatile("" : "+s"(next));                   // (nor its addresses)
            fetch(next);
        }
        lds_barrier();
        // (three tiles side by side, then two: the products of one are a chain, in which each waits half as long again as it takes, and
        // for its operands.  With the substitution's reads ahead of its chain, below: a chunk on its own 15.6 -> 14.6 us at d 128)
        auto multiply = [&](auto first, auto count) __attribute__((always_inline)) {
            constexpr int i0 = decltype(first)::value, N = decltype(count)::value;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                f32x4 fa[N], fb[N];
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int u = w + 4 * (i0 + i), b = u < 10 ? u : u - 10;
                    int R, I;
                    block_of(b, R, I);
                    fa[i] = ld4((u < 10 ? sKp : sQp) + (16 * R + m) * kLdT + 4 * g + 16 * kt);
                    fb[i] = ld4(sKn + (16 * I + m) * kLdT + 4 * g + 16 * kt);
                    if (R > I) fb[i] *= ld4(sF + pair_of(R, I) * 64 + 4 * g + 16 * kt);
                }
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int i = 0; i < N; ++i) acc[i0 + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][ks], fb[i][ks], acc[i0 + i], 0, 0, 0);
            }
        };
        multiply(std::integral_constant<int, 0>{}, std::integral_constant<int, 3>{});
        multiply(std::integral_constant<int, 3>{}, std::integral_constant<int, 2>{});
    }
    if (__syncthreads_or(strong)) {
        // some channel's decay inside a block is beyond the factors' range: the diagonal blocks again, all of them and
        // all channels, pair by pair in the log domain
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int u = w + 4 * i, b = u < 10 ? u : u - 10;
            int R, I;
            block_of(b, R, I);
            if (R == I) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll 1
        for (int hf = 0; hf < D / 64; ++hf) {
            const int t = 4 * hf + w;
            f32x4 kk[4], qq[4];
            Decay d;
            load_tile(d.x, log_alpha + base + m + 16 * t, stride, c.nv, g);
            load_tile(kk, k + base + m + 16 * t, stride, c.nv, g);
            load_tile(qq, q + base + m + 16 * t, stride, c.nv, g);
            sum_decay(d, lane);
            __syncthreads();
#pragma unroll
            for (int R = 0; R < 4; ++R) {
                const f32x4 L = d.in_block(R);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int at = (16 * R + 4 * g + j) * kLdT + 16 * w + m;
                    sKp[at] = kk[R][j]; sQp[at] = qq[R][j]; sKn[at] = L[j];
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                const int u = w + 4 * i, b = u < 10 ? u : u - 10;
                int R, I;
                block_of(b, R, I);
                if (R != I) continue;
                const float *row = u < 10 ? sKp : sQp;
#pragma unroll 1
                for (int ch = 0; ch < 64; ++ch) {
                    const int ci = (16 * R + m) * kLdT + ch;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int ri = (16 * R + 4 * g + j) * kLdT + ch;
                        acc[i][j] = fmaf(row[ri] * sKp[ci], fast_exp2(fminf(sKn[ri] - sKn[ci], 0.f)), acc[i][j]);
                    }
                }
            }
        }
        __syncthreads();
    }
    // A as [64][kLdT] (strict lower; the diagonal blocks' upper parts are zero), P straight to the slot
    float *sA = sKp, *sQ = sQp;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int u = w + 4 * i, b = u < 10 ? u : u - 10;
        int R, I;
        block_of(b, R, I);
        if (R == I) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (m > 4 * g + j || (u < 10 && m == 4 * g + j)) acc[i][j] = 0.f;
        }
        if (u >= 10) st(slot + SL::kP + b * kFrag, acc[i]);
        else {
#pragma unroll
            for (int j = 0; j < 4; ++j) sA[(16 * R + 4 * g + j) * kLdT + 16 * I + m] = acc[i][j];
        }
    }
    lds_barrier();
    // (I + A Diag(beta)) Q = A by 16 x 16 blocks; wave w takes the column block w.  Diagonal block: substitution,
    // a lane holds its column.
    f32x4 Q[4];
    {
        // (the rows of A are read ahead of the chain: nothing is stored between them)
        float x[16], q[16];
        const float *a = sA + (16 * w) * kLdT + 16 * w;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float s = a[r * kLdT + m];
#pragma unroll
            for (int i = 0; i < r; ++i) s = fmaf(-a[r * kLdT + i], x[i], s);
            q[r] = s;
            x[r] = s * sBeta[16 * w + r];                    // beta_i Q[i][m] is what the rows below take
        }
        f32x4 own;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float q0 = q[j], q1 = q[4 + j], q2 = q[8 + j], q3 = q[12 + j], lo = g & 1 ? q1 : q0, hi = g & 1 ? q3 : q2;
            own[j] = g & 2 ? hi : lo;
            sQ[(16 * w + 4 * g + j) * kLdT + 16 * w + m] = own[j];
        }
#pragma unroll
        for (int ww = 0; ww < 4; ++ww)
            if (ww == w) Q[ww] = own;
    }
    lds_barrier();
    f32x4 bt[4];
#pragma unroll
    for (int R = 0; R < 4; ++R) bt[R] = ld4(sBeta + 16 * R + 4 * g);
    // Q_RI = (I - Q_RR Diag(beta_R)) (A_RI - sum_{I <= J < R} A_RJ Diag(beta_J) Q_JI)
#pragma unroll
    for (int R = 1; R < 4; ++R) {
        if (R <= w) continue;
        f32x4 s = {0.f, 0.f, 0.f, 0.f}, a;
#pragma unroll
        for (int J = 0; J < R; ++J)
            if (J >= w) s = mfma16(ld4(sA + (16 * R + m) * kLdT + 16 * J + 4 * g), bt[J] * Q[J], s);
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = sA[(16 * R + 4 * g + j) * kLdT + 16 * w + m];
        const f32x4 x = a - s;
        Q[R] = x - mfma16(ld4(sQ + (16 * R + m) * kLdT + 16 * R + 4 * g), bt[R] * x, f32x4{0.f, 0.f, 0.f, 0.f});
    }
#pragma unroll
    for (int R = 0; R < 4; ++R)
        if (R >= w) st(slot + SL::kQ + tri(R, w) * kFrag, Q[R]);
}

template <typename Tin, int D, bool kRows>
kda_status launch_prep(const Problem &p, const Tin *q, const Tin *k, const Tin *log_alpha, const Tin *beta, float *slots,
                       hipStream_t stream)
{
    const int64_t blocks = p.slots * p.H;
    if (blocks == 0) return KDA_OK;
    if (blocks > 0x7fffffffLL) return fail(KDA_ERR_UNSUPPORTED, "%lld chunks in one call", (long long)blocks);
    hipLaunchKernelGGL((kda_f32_prep_kernel<Tin, D, kRows>), dim3((unsigned)blocks), dim3(kPrepThreads), kPrepLds, stream, q, k,
                       log_alpha, beta, slots, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? KDA_OK : fail(KDA_ERR_LAUNCH, "kda_f32_prep: %s", hipGetErrorString(e));
}

#define KDA_PREP(T, DD, ROWS) template kda_status launch_prep<T, DD, ROWS>(const Problem &, const T *, const T *, const T *, const T *, \
                                                                             float *, hipStream_t)
KDA_PREP(float, 64, false);
KDA_PREP(float, 128, false);
KDA_PREP(__hip_bfloat16, 64, false);
KDA_PREP(__hip_bfloat16, 128, false);
KDA_PREP(float, 64, true);
KDA_PREP(float, 128, true);
KDA_PREP(__hip_bfloat16, 64, true);
KDA_PREP(__hip_bfloat16, 128, true);
#undef KDA_PREP

}  // namespace f32
}  // namespace kda
