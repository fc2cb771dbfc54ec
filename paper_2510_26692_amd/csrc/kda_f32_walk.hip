// The two sequential walks of the fp32 path over the chunks of a (sequence, head), on the operands that
// kda_f32_prep leaves per chunk (Kg = Gamma.K, Kt = Gamma^{i->C}.K, Qg = Gamma.Q, P = Tril(A_qk), Q):
//
//   forward    Y = V - Kg S0,   R = Y - Q (beta Y),   Vn = beta R,   S1 = Diag(e^(G_C)) S0 + Kt^T Vn
//              (and, for the prefill, O = scale (Qg S0 + P Vn))
//   backward   dVn = Kt dS1 + P^T dO,   Z = dVn - Q^T (beta dVn),   X = beta Z = dV,
//              dS0 = Diag(e^(G_C)) dS1 + Qg^T dO - Kg^T X                       (dO carries the scale)
//
// The columns of S (and of dS) never mix, so a workgroup owns 16 NC of them.  Its four waves share every product
// by ROWS: wave w has the token rows 16 w .. and the state rows of D / 64 channel tiles, so an operand fragment is
// loaded by one wave of the workgroup, from memory straight into registers (no LDS, no second copy), and the
// right-hand sides (S, Y, Vn: what the waves hand each other) go through LDS in accumulator order, which is B
// operand order.  Three barriers a chunk.  Each operand's registers are refilled for the next chunk right after
// their last use, so a load has most of a step to arrive.
//
// The two walks do not depend on each other (the backward one needs no forward state): one launch runs both, which
// doubles the workgroups in flight.
#include "kda_f32_tile.h"

namespace kda {
namespace f32 {

constexpr int kWalkThreads = 256;

template <int D, int NC> constexpr size_t walk_lds(bool both) { return (size_t)(NC * (D / 16) + (both ? 4 : 2) * NC * 4) * kFrag * 4; }

struct Where { int64_t tok_base, len, nchunks, slot0, state; };

__device__ __forceinline__ Where where(const Problem &p, int64_t n, int h, int D)
{
    Where x;
    if (p.cu) { x.tok_base = p.cu[n]; x.len = (int64_t)p.cu[n + 1] - x.tok_base; }
    else      { x.tok_base = n * p.T; x.len = p.T; }
    x.nchunks = (x.len + kC - 1) / kC;
    x.slot0 = first_slot(p.cu, n, p.chunks_per_seq) * p.H + h;               // slots of a sequence are H apart
    x.state = (n * p.H + h) * (int64_t)D * D;
    return x;
}

// Rows row0 .. row0 + 3 of NC column tiles of a [tokens, H, D] tensor (rows past nv: the last one's, masked when used).
// They are held as the 32-bit words they lie in and taken apart where they are used, behind an opaque point: left to
// itself the compiler widens a bf16 value where it is loaded, or at the head of the loop, and waits for it there.
template <typename T, int NC> struct Rows {
    uint32_t raw[NC][4];
    __device__ __forceinline__ void load_row(int j, const T *base, int m, int64_t stride, int row0, int nv)
    {
        const int r = row0 + j;
        const T *p = base + (int64_t)(r < nv ? r : nv - 1) * stride + (sizeof(T) == 2 ? m & ~1 : m);
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) raw[nc][j] = *reinterpret_cast<const uint32_t *>(p + 16 * nc);
    }
    __device__ __forceinline__ f32x4 tile(int nc, int m, int row0, int nv) const
    {
        f32x4 x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t u = raw[nc][j];
            asm volatile("" : "+v"(u));
            if (sizeof(T) == 2) u = m & 1 ? u & 0xffff0000u : u << 16;
            x[j] = row0 + j < nv ? __uint_as_float(u) : 0.f;
        }
        return x;
    }
};

// Four token tiles of B fragments from LDS: all fetched at once, so that one wait covers them, unless that takes more
// than 32 registers.
template <int NC> struct Four {
    static constexpr bool kHeld = NC <= 2;
    f32x4 b[kHeld ? 4 : 1][kHeld ? NC : 1];
    const float *p;
    __device__ __forceinline__ Four(const float *src, int lane) : p(src + 4 * lane)
    {
        if constexpr (kHeld) {
#pragma unroll
            for (int R = 0; R < 4; ++R)
#pragma unroll
                for (int nc = 0; nc < NC; ++nc) b[R][nc] = ld4(p + (nc * 4 + R) * kFrag);
            pin_memory_order();
        }
    }
    __device__ __forceinline__ f32x4 get(int R, int nc) const
    {
        if constexpr (kHeld) return b[R][nc];
        else return ld4(p + (nc * 4 + R) * kFrag);
    }
};

// acc[nc] += A_t B_t over N contraction tiles, B fragments from LDS fetched kAhead tiles ahead of the products.
// after(t): the loads that refill what tile t has used, and stores.  They go out one or two at a time between the
// products: a burst of them holds the wave up at issue (the L1 hands a compute unit 64 bytes a clock).
template <int N, int NC, int kAhead, typename FA, typename FB, typename FH>
__device__ __forceinline__ void product(f32x4 (&acc)[NC], FA &&a, FB &&b, FH &&after)
{
    f32x4 ring[kAhead + 1][NC];
#pragma unroll
    for (int t = 0; t < kAhead && t < N; ++t)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) ring[t][nc] = b(t, nc);
#pragma unroll
    for (int t = 0; t < N; ++t) {
        if (t + kAhead < N) {
#pragma unroll
            for (int nc = 0; nc < NC; ++nc) ring[(t + kAhead) % (kAhead + 1)][nc] = b(t + kAhead, nc);
        }
        pin_memory_order();
        const f32x4 at = a(t);
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) acc[nc] = mfma16(at, ring[t % (kAhead + 1)][nc], acc[nc]);
        after(t);
    }
}

// S[tt][nc] += A_tt,R B_R over the four token tiles, likewise.
template <int TW, int NC, typename FH>
__device__ __forceinline__ void update_state(f32x4 (&S)[TW][NC], const f32x4 (&a)[TW][4], const Four<NC> &b, FH &&after)
{
#pragma unroll
    for (int R = 0; R < 4; ++R) {
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            const f32x4 x = b.get(R, nc);
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) S[tt][nc] = mfma16(a[tt][R], x, S[tt][nc]);
        }
        pin_memory_order();
        after(R);
    }
}

template <int D, int NC>
__device__ __forceinline__ void load_state(f32x4 (&S)[D / 64][NC], const float *src, int t0, int g)
{
#pragma unroll
    for (int tt = 0; tt < D / 64; ++tt)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc)
#pragma unroll
            for (int j = 0; j < 4; ++j) S[tt][nc][j] = src ? src[(int64_t)(16 * (t0 + tt) + 4 * g + j) * D + 16 * nc] : 0.f;
}
template <int D, int NC>
__device__ __forceinline__ void store_state(float *dst, const f32x4 (&S)[D / 64][NC], int t0, int g)
{
#pragma unroll
    for (int tt = 0; tt < D / 64; ++tt)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc)
#pragma unroll
            for (int j = 0; j < 4; ++j) dst[(int64_t)(16 * (t0 + tt) + 4 * g + j) * D + 16 * nc] = S[tt][nc][j];
}

// One token tile of R or Z, NC column tiles from `tile` on.
template <int D, int NC>
__device__ __forceinline__ void store_rows(float *dst, const f32x4 (&x)[NC], int64_t tok0, int H, int h, int nv, int R, int tile, int lane)
{
    const int token = 4 * (lane >> 4) + (lane & 3), n = tile_tokens(nv, R);
    float *p = dst + token_rows(tok0, H, h, nv, D);
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) {
        const f32x4 t = quad_transpose(x[nc], lane);
        if (token < n) st4(p + row_form(R, tile + nc, (lane >> 2) & 3, token, n, D), t);
    }
}

// What the walk leaves besides the final state: o (the prefill), S0 and R (the backward pass), or nothing, where four
// other waves of the workgroup form o from the S0 and Vn in LDS (output_role).
enum Leaves { kOutputs, kStates, kNothing };

template <typename Tin, int D, int NC, Leaves kLeaves>
__device__ __forceinline__ void forward_walk(float *smem, const Problem &p, const Tin *v, const float *h0,
                                             const float *slots, float *S0, float *Rw, float *o, float *hT, int64_t n, int h,
                                             int slice)
{
    using SL = Slot<D>;
    constexpr bool kOut = kLeaves == kOutputs, kRows = kLeaves != kStates;      // kRows: the slots are in row form
    constexpr int NT = SL::kTiles, TW = NT / 4;
    float *sS = smem, *sY = sS + NC * NT * kFrag, *sV = sY + NC * 4 * kFrag;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4, turned = 4 * turned_lane(lane), left = kRows ? 4 * lane : turned;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), row0 = 16 * w + 4 * g, t0 = TW * w;
    auto turn = [&](const f32x4 &a) __attribute__((always_inline)) { return kRows ? a : quad_transpose(a, lane); };
    const Where x = where(p, n, h, D);
    const int64_t stride = (int64_t)p.H * D;
    const int col0 = 16 * NC * slice;

    f32x4 S[TW][NC];
    load_state<D, NC>(S, h0 ? h0 + x.state + col0 + m : nullptr, t0, g);
    constexpr int kAhead = NC == 1 ? 4 : NC == 2 ? 2 : 1;
    f32x4 kg[NT], qm[4], kt[TW][4], gam[TW], qg[kOut ? NT : 1], pm[kOut ? 4 : 1];
    f32x4 bt;
    Rows<Tin, NC> vv;
    auto load_kg = [&](const float *slot, int t) __attribute__((always_inline)) { kg[t] = ld4(slot + SL::kKg + (w * NT + t) * kFrag + left); };
    auto load_qg = [&](const float *slot, int t) __attribute__((always_inline)) { qg[kOut ? t : 0] = ld4(slot + SL::kQg + (w * NT + t) * kFrag + left); };
    auto load_q = [&](const float *slot, int J) __attribute__((always_inline)) { qm[J] = ld4(slot + SL::kQ + tri(w, J < w ? J : w) * kFrag + left); };
    auto load_p = [&](const float *slot, int J) __attribute__((always_inline)) { pm[kOut ? J : 0] = ld4(slot + SL::kP + tri(w, J < w ? J : w) * kFrag + left); };
    auto load_kt = [&](const float *slot, int tt, int R) __attribute__((always_inline)) { kt[tt][R] = ld4(slot + SL::kKt + (R * NT + t0 + tt) * kFrag + 4 * lane); };
    auto load_gam = [&](const float *slot, int tt) __attribute__((always_inline)) { gam[tt] = ld4(slot + SL::kGc + 16 * (t0 + tt) + 4 * g); };
    auto valid = [&](int64_t ci) { return (int)(x.len - ci * kC < kC ? x.len - ci * kC : kC); };
    auto load_v = [&](int64_t ci, int j) __attribute__((always_inline)) {
        vv.load_row(j, v + ((x.tok_base + ci * kC) * p.H + h) * D + col0, m, stride, row0, valid(ci));
    };
    auto load_b = [&](const float *slot) __attribute__((always_inline)) { bt = ld4(slot + SL::kBeta + row0); };
    auto share_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int tt = 0; tt < TW; ++tt)
#pragma unroll
            for (int nc = 0; nc < NC; ++nc) st4(sS + (nc * NT + t0 + tt) * kFrag + 4 * lane, S[tt][nc]);
    };
    if (x.nchunks > 0) {
        const float *slot = slots + x.slot0 * SL::kFloats;
        // (in the order of the loop: the compiler's waits take the worse of the two ways into it)
#pragma unroll
        for (int t = 0; t < NT; ++t) load_kg(slot, t);
        if (kOut) {
#pragma unroll
            for (int t = 0; t < NT; ++t) load_qg(slot, t);
        }
        pin_memory_order();
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            load_q(slot, R); load_v(0, R);
            if (R == 0) load_b(slot);
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) load_kt(slot, tt, R);
            if (R < TW) load_gam(slot, R < TW ? R : 0);
            pin_memory_order();
        }
        share_state();
        lds_barrier();
    }
#pragma unroll 1
    for (int64_t ci = 0; ci < x.nchunks; ++ci) {
        const int nv = valid(ci);
        const int64_t cn = ci + 1 < x.nchunks ? ci + 1 : ci;                  // (the last step fetches its own operands again)
        const float *next = slots + (x.slot0 + cn * p.H) * SL::kFloats, *here = slots + (x.slot0 + ci * p.H) * SL::kFloats;
        float *s0 = kLeaves != kStates ? nullptr : S0 + (x.slot0 + ci * p.H) * (int64_t)(D * D) + turned;
        // Y = V - Kg S0
        f32x4 y[NC] = {}, oo[kOut ? NC : 1] = {};
        product<NT, NC, kAhead>(y, [&](int t) { return turn(kg[t]); },
                                [&](int t, int nc) { return ld4(sS + (nc * NT + t) * kFrag + 4 * lane); },
                                [&](int t) {
                                    load_kg(next, t);
                                    if (kOut && t < 4) load_p(here, t);
                                    const int tt = t / NC, nc = t % NC;
                                    if (kLeaves == kStates && tt < TW)
                                        st4(s0 + ((t0 + tt) * NT + NC * slice + nc) * kFrag, quad_transpose(S[tt < TW ? tt : 0][nc], lane));
                                });
        const f32x4 b4 = bt;
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            y[nc] = vv.tile(nc, m, row0, nv) - y[nc];
            st4(sY + (nc * 4 + w) * kFrag + 4 * lane, b4 * y[nc]);
        }
        if constexpr (kOut)                                                   // O = scale (Qg S0 + P Vn), the first half
            product<NT, NC, kAhead>(oo, [&](int t) { return turn(qg[t]); },
                                    [&](int t, int nc) { return ld4(sS + (nc * NT + t) * kFrag + 4 * lane); },
                                    [&](int t) { load_qg(next, t); });
        lds_barrier();
        // R = Y - Q (beta Y)
        f32x4 r[NC] = {};
        {
            const Four<NC> by(sY, lane);
#pragma unroll
            for (int tt = 0; tt < TW; ++tt)
#pragma unroll
                for (int nc = 0; nc < NC; ++nc) S[tt][nc] *= gam[tt];
#pragma unroll
            for (int J = 0; J < 4; ++J)
                if (J <= w) {
                    const f32x4 a = turn(qm[J]);
#pragma unroll
                    for (int nc = 0; nc < NC; ++nc) r[nc] = mfma16(a, by.get(J, nc), r[nc]);
                }
        }
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            r[nc] = y[nc] - r[nc];
            st4(sV + (nc * 4 + w) * kFrag + 4 * lane, b4 * r[nc]);
        }
        if (kLeaves == kStates) {
            store_rows<D, NC>(Rw, r, x.tok_base + ci * kC, p.H, h, nv, w, NC * slice, lane);
        }
        lds_barrier();
        // S1 = Diag(e^(G_C)) S0 + Kt^T Vn
        {
            const Four<NC> bv(sV, lane);
            update_state<TW, NC>(S, kt, bv, [&](int R) {
                load_q(next, R);
                load_v(cn, R);
                if (R == 0) load_b(next);
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) load_kt(next, tt, R);
                if (R < TW) load_gam(next, R < TW ? R : 0);
            });
            share_state();
            if (kOut) {
#pragma unroll
                for (int J = 0; J < 4; ++J)
                    if (J <= w) {
                        const f32x4 a = turn(pm[kOut ? J : 0]);
#pragma unroll
                        for (int nc = 0; nc < NC; ++nc) oo[kOut ? nc : 0] = mfma16(a, bv.get(J, nc), oo[kOut ? nc : 0]);
                    }
                float *po = o + ((x.tok_base + ci * kC) * p.H + h) * (int64_t)D + col0 + m;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (row0 + j < nv) {
#pragma unroll
                        for (int nc = 0; nc < NC; ++nc) po[(row0 + j) * stride + 16 * nc] = p.scale * oo[kOut ? nc : 0][j];
                    }
            }
        }
        lds_barrier();
    }
    if (hT) store_state<D, NC>(hT + x.state + col0 + m, S, t0, g);
}

// The four waves that form o = scale (Qg S0 + P Vn) beside four that walk (forward_walk of kNothing, one column tile):
// the products that no later step waits for leave the chain of the steps.  In step with the walk's three barriers a
// chunk: S0 is read before the second one and Vn between the second and the third, which is when LDS holds them.
template <int D>
__device__ __forceinline__ void output_role(const float *smem, const Problem &p, const float *slots, float *o, int64_t n, int h,
                                            int slice)
{
    using SL = Slot<D>;
    constexpr int NT = SL::kTiles, kAhead = 4;
    const float *sS = smem, *sV = sS + (NT + 4) * kFrag;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) - 4, row0 = 16 * w + 4 * g;
    const Where x = where(p, n, h, D);
    const int64_t stride = (int64_t)p.H * D;
    f32x4 qg[NT], pm[4];
    auto load_qg = [&](const float *slot, int t) __attribute__((always_inline)) { qg[t] = ld4(slot + SL::kQg + (w * NT + t) * kFrag + 4 * lane); };
    auto load_p = [&](const float *slot, int J) __attribute__((always_inline)) { pm[J] = ld4(slot + SL::kP + tri(w, J < w ? J : w) * kFrag + 4 * lane); };
    if (x.nchunks > 0) {
        const float *slot = slots + x.slot0 * SL::kFloats;
#pragma unroll
        for (int t = 0; t < NT; ++t) load_qg(slot, t);
#pragma unroll
        for (int J = 0; J < 4; ++J) load_p(slot, J);
        lds_barrier();
    }
#pragma unroll 1
    for (int64_t ci = 0; ci < x.nchunks; ++ci) {
        const int nv = (int)(x.len - ci * kC < kC ? x.len - ci * kC : kC);
        const int64_t cn = ci + 1 < x.nchunks ? ci + 1 : ci;
        const float *next = slots + (x.slot0 + cn * p.H) * SL::kFloats;
        f32x4 oo[1] = {};
        auto half = [&](int first) __attribute__((always_inline)) {
            product<NT / 2, 1, kAhead>(oo, [&](int t) { return qg[first + t]; },
                                       [&](int t, int) { return ld4(sS + (first + t) * kFrag + 4 * lane); },
                                       [&](int t) { load_qg(next, first + t); });
        };
        half(0);
        lds_barrier();
        half(NT / 2);
        lds_barrier();
        const Four<1> bv(sV, lane);
#pragma unroll
        for (int J = 0; J < 4; ++J)
            if (J <= w) oo[0] = mfma16(pm[J], bv.get(J, 0), oo[0]);
        float *po = o + ((x.tok_base + ci * kC) * p.H + h) * (int64_t)D + 16 * slice + m;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (row0 + j < nv) po[(row0 + j) * stride] = p.scale * oo[0][j];
#pragma unroll
        for (int J = 0; J < 4; ++J) load_p(next, J);
        lds_barrier();
    }
}

// kHelped (one column tile): four other waves of the workgroup leave P^T dO and Qg^T dO of the chunk in LDS (gradient_role).
template <typename Tdo, int D, int NC, bool kHelped>
__device__ __forceinline__ void backward_walk(float *smem, const Problem &p, const Tdo *d_o, const float *d_hT,
                                              const float *slots, float *dS1, float *Zw, float *dh0, int64_t n, int h, int slice)
{
    using SL = Slot<D>;
    constexpr int NT = SL::kTiles, TW = NT / 4;
    float *sS = smem, *sY = sS + NC * NT * kFrag, *sX = sY + NC * 4 * kFrag, *sO = sX + NC * 4 * kFrag;    // sO: two buffers
    static_assert(!kHelped || NC == 1, "one column tile");
    const float *sE = sO + 4 * kFrag;                                         // kHelped: [4] P^T dO, [NT] Qg^T dO
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4, turned = 4 * turned_lane(lane);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), row0 = 16 * w + 4 * g, t0 = TW * w;
    const Where x = where(p, n, h, D);
    const int64_t stride = (int64_t)p.H * D;
    const int col0 = 16 * NC * slice;

    f32x4 S[TW][NC];
    load_state<D, NC>(S, d_hT ? d_hT + x.state + col0 + m : nullptr, t0, g);
    constexpr int kAhead = NC == 1 ? 4 : NC == 2 ? 2 : 1;
    f32x4 kt[NT], pm[4], qm[4], kg[TW][4], qg[TW][4], gam[TW];
    f32x4 bt;
    Rows<Tdo, NC> vo;
    auto load_kt = [&](const float *slot, int t) __attribute__((always_inline)) { kt[t] = ld4(slot + SL::kKt + (w * NT + t) * kFrag + turned); };
    auto load_p = [&](const float *slot, int R) __attribute__((always_inline)) { pm[R] = ld4(slot + SL::kP + tri(R > w ? R : w, w) * kFrag + 4 * lane); };
    auto load_q = [&](const float *slot, int R) __attribute__((always_inline)) { qm[R] = ld4(slot + SL::kQ + tri(R > w ? R : w, w) * kFrag + 4 * lane); };
    auto load_kg = [&](const float *slot, int tt, int R) __attribute__((always_inline)) { kg[tt][R] = ld4(slot + SL::kKg + (R * NT + t0 + tt) * kFrag + 4 * lane); };
    auto load_qg = [&](const float *slot, int tt, int R) __attribute__((always_inline)) { qg[tt][R] = ld4(slot + SL::kQg + (R * NT + t0 + tt) * kFrag + 4 * lane); };
    auto load_gam = [&](const float *slot, int tt) __attribute__((always_inline)) { gam[tt] = ld4(slot + SL::kGc + 16 * (t0 + tt) + 4 * g); };
    auto valid = [&](int64_t ci) { return (int)(x.len - ci * kC < kC ? x.len - ci * kC : kC); };
    auto load_o = [&](int64_t ci, int j) __attribute__((always_inline)) {
        vo.load_row(j, d_o + ((x.tok_base + ci * kC) * p.H + h) * (int64_t)D + col0, m, stride, row0, valid(ci));
    };
    auto load_b = [&](const float *slot) __attribute__((always_inline)) { bt = ld4(slot + SL::kBeta + row0); };
    auto share_o = [&](int64_t ci, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) st4(sO + ((buf * NC + nc) * 4 + w) * kFrag + 4 * lane, vo.tile(nc, m, row0, valid(ci)) * p.scale);
    };
    auto share_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int tt = 0; tt < TW; ++tt)
#pragma unroll
            for (int nc = 0; nc < NC; ++nc) st4(sS + (nc * NT + t0 + tt) * kFrag + 4 * lane, S[tt][nc]);
    };
    const int64_t last = x.nchunks - 1;
    if (last >= 0) {
        const float *slot = slots + (x.slot0 + last * p.H) * SL::kFloats;
        if (!kHelped) {
#pragma unroll
            for (int j = 0; j < 4; ++j) load_o(last, j);
            share_o(last, 0);
        }
        // (in the order of the loop: the compiler's waits take the worse of the two ways into it)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            load_kt(slot, t);
            if (!kHelped && t < 4) load_p(slot, t);
        }
        pin_memory_order();
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            load_q(slot, R);
            if (R == 0) load_b(slot);
            if (!kHelped) {
                load_o(last > 0 ? last - 1 : 0, R);
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) load_qg(slot, tt, R);
            }
            if (R < TW) load_gam(slot, R < TW ? R : 0);
            pin_memory_order();
        }
#pragma unroll
        for (int R = 0; R < 4; ++R) {
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) load_kg(slot, tt, R);
            pin_memory_order();
        }
        share_state();
        if (kHelped) lds_barrier();                                           // (the helpers' own, over the rows of dO)
        lds_barrier();
    }
    int buf = 0;
#pragma unroll 1
    for (int64_t ci = last; ci >= 0; --ci, buf ^= 1) {
        const int64_t cn = ci > 0 ? ci - 1 : 0, cnn = cn > 0 ? cn - 1 : 0;
        const float *next = slots + (x.slot0 + cn * p.H) * SL::kFloats;
        float *ds1 = dS1 + (x.slot0 + ci * p.H) * (int64_t)(D * D) + turned;
        const int nv = valid(ci);
        const float *so = sO + buf * (NC * 4 * kFrag);
        // dVn = Kt dS1 + P^T dO.  (Two accumulators: 128 terms added to the second product, as large as they are in sum, are
        // rounded at its size: 23 % more error in dv at slow decay.)
        f32x4 y[NC] = {}, e[NC] = {};
        if constexpr (kHelped) {
            e[0] = ld4(sE + w * kFrag + 4 * lane);
        } else {
            const Four<NC> bo(so, lane);
#pragma unroll
            for (int R = 0; R < 4; ++R)
                if (R >= w) {
#pragma unroll
                    for (int nc = 0; nc < NC; ++nc) e[nc] = mfma16(pm[R], bo.get(R, nc), e[nc]);
                }
        }
        product<NT, NC, kAhead>(y, [&](int t) { return quad_transpose(kt[t], lane); },
                                [&](int t, int nc) { return ld4(sS + (nc * NT + t) * kFrag + 4 * lane); },
                                [&](int t) {
                                    load_kt(next, t);
                                    if (!kHelped && t < 4) load_p(next, t);
                                    const int tt = t / NC, nc = t % NC;
                                    if (tt < TW)
                                        st4(ds1 + ((t0 + tt) * NT + NC * slice + nc) * kFrag, quad_transpose(S[tt < TW ? tt : 0][nc], lane));
                                });
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) y[nc] += e[nc];
        const f32x4 b4 = bt;
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) st4(sY + (nc * 4 + w) * kFrag + 4 * lane, b4 * y[nc]);
        if (!kHelped) share_o(cn, buf ^ 1);
        lds_barrier();
        // Z = dVn - Q^T (beta dVn)
        f32x4 z[NC] = {};
        {
            const Four<NC> by(sY, lane);
#pragma unroll
            for (int tt = 0; tt < TW; ++tt)
#pragma unroll
                for (int nc = 0; nc < NC; ++nc) S[tt][nc] *= gam[tt];
#pragma unroll
            for (int R = 0; R < 4; ++R)
                if (R >= w) {
#pragma unroll
                    for (int nc = 0; nc < NC; ++nc) z[nc] = mfma16(qm[R], by.get(R, nc), z[nc]);
                }
        }
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
            z[nc] = y[nc] - z[nc];
            st4(sX + (nc * 4 + w) * kFrag + 4 * lane, -b4 * z[nc]);
        }
        // dS0 = Diag(e^(G_C)) dS1 + Qg^T dO - Kg^T X  (the first product is done while X is on its way)
        auto refill = [&](int R) __attribute__((always_inline)) {
            load_q(next, R);
            if (R == 0) load_b(next);
            if (!kHelped) {
                load_o(cnn, R);
#pragma unroll
                for (int tt = 0; tt < TW; ++tt) load_qg(next, tt, R);
            }
            if (R < TW) load_gam(next, R < TW ? R : 0);
        };
        if constexpr (kHelped) {
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) S[tt][0] += ld4(sE + (4 + t0 + tt) * kFrag + 4 * lane);
#pragma unroll
            for (int R = 0; R < 4; ++R) { refill(R); pin_memory_order(); }
        } else {
            update_state<TW, NC>(S, qg, Four<NC>(so, lane), refill);
        }
        store_rows<D, NC>(Zw, z, x.tok_base + ci * kC, p.H, h, nv, w, NC * slice, lane);
        lds_barrier();
        update_state<TW, NC>(S, kg, Four<NC>(sX, lane), [&](int R) {
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) load_kg(next, tt, R);
        });
        share_state();
        lds_barrier();
    }
    if (dh0) store_state<D, NC>(dh0 + x.state + col0 + m, S, t0, g);
}

// The four waves that leave P^T dO and Qg^T dO of a chunk in LDS while four others walk the chunk before it
// (backward_walk of kHelped): these products need no state, so they leave the chain of the steps.  In step with the
// walk's three barriers a chunk: the rows of dO are exchanged before the first; the walk reads the products of its chunk
// before the second, and the next chunk's replace them between the second and the third.
template <typename Tdo, int D>
__device__ __forceinline__ void gradient_role(float *smem, const Problem &p, const Tdo *d_o, const float *slots, int64_t n, int h,
                                              int slice)
{
    using SL = Slot<D>;
    constexpr int NT = SL::kTiles, TW = NT / 4;
    float *sO = smem + (NT + 8) * kFrag, *sE = sO + 4 * kFrag;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) - 4, row0 = 16 * w + 4 * g, t0 = TW * w;
    const Where x = where(p, n, h, D);
    const int64_t stride = (int64_t)p.H * D;
    f32x4 pm[4], qg[TW][4];
    Rows<Tdo, 1> vo;
    auto valid = [&](int64_t ci) { return (int)(x.len - ci * kC < kC ? x.len - ci * kC : kC); };
    auto load_o = [&](int64_t ci) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            vo.load_row(j, d_o + ((x.tok_base + ci * kC) * p.H + h) * (int64_t)D + 16 * slice, m, stride, row0, valid(ci));
    };
    auto share_o = [&](int64_t ci) __attribute__((always_inline)) { st4(sO + w * kFrag + 4 * lane, vo.tile(0, m, row0, valid(ci)) * p.scale); };
    auto load_ops = [&](int64_t ci) __attribute__((always_inline)) {
        const float *slot = slots + (x.slot0 + ci * p.H) * SL::kFloats;
#pragma unroll
        for (int R = 0; R < 4; ++R) {
            pm[R] = ld4(slot + SL::kP + tri(R > w ? R : w, w) * kFrag + 4 * lane);
#pragma unroll
            for (int tt = 0; tt < TW; ++tt) qg[tt][R] = ld4(slot + SL::kQg + (R * NT + t0 + tt) * kFrag + 4 * lane);
        }
    };
    f32x4 y, E[TW][1];
    auto multiply = [&]() __attribute__((always_inline)) {
        const Four<1> bo(sO, lane);
        y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int R = 0; R < 4; ++R)
            if (R >= w) y = mfma16(pm[R], bo.get(R, 0), y);
#pragma unroll
        for (int tt = 0; tt < TW; ++tt) E[tt][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        update_state<TW, 1>(E, qg, bo, [](int) {});
    };
    auto leave = [&]() __attribute__((always_inline)) {
        st4(sE + w * kFrag + 4 * lane, y);
#pragma unroll
        for (int tt = 0; tt < TW; ++tt) st4(sE + (4 + t0 + tt) * kFrag + 4 * lane, E[tt][0]);
    };
    const int64_t last = x.nchunks - 1;
    if (last < 0) return;
    load_o(last);
    load_ops(last);
    share_o(last);
    lds_barrier();
    multiply();
    leave();
    load_o(last > 0 ? last - 1 : 0);
    load_ops(last > 0 ? last - 1 : 0);
    lds_barrier();
#pragma unroll 1
    for (int64_t ci = last; ci >= 0; --ci) {
        const int64_t cn = ci > 0 ? ci - 1 : 0, cnn = cn > 0 ? cn - 1 : 0;    // (the last ones are formed again, unused)
        share_o(cn);
        load_o(cnn);
        lds_barrier();
        multiply();
        load_ops(cnn);
        lds_barrier();
        leave();
        lds_barrier();
    }
}

// Workgroups are handed to the eight dies in turn: the slices of a (sequence, head), which read the same operands at
// about the same time, are placed eight workgroups apart, on one die's L2.
template <int D, int NC>
__device__ __forceinline__ bool place(const Problem &p, int64_t bid, int64_t &n, int &h, int &slice)
{
    constexpr int kSlices = D / (16 * NC);
    const int64_t rest = bid >> 3, pair = (rest / kSlices) * 8 + (bid & 7);
    slice = (int)(rest % kSlices);
    n = pair / p.H;
    h = (int)(pair - n * p.H);
    return pair < (int64_t)p.num_seqs * p.H;
}
static int64_t walk_workgroups(const Problem &p, int slices) { return ((int64_t)p.num_seqs * p.H + 7) / 8 * 8 * slices; }

template <typename Tin, int D, int NC>
__global__ __launch_bounds__(kWalkThreads, 2)
void kda_f32_forward_walk_kernel(const Tin *__restrict__ v, const float *__restrict__ h0,
                                 const float *__restrict__ slots, float *__restrict__ o, float *__restrict__ hT, const Problem p)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    int64_t n;
    int h, slice;
    if (!place<D, NC>(p, blockIdx.x, n, h, slice)) return;
    forward_walk<Tin, D, NC, kOutputs>(smem, p, v, h0, slots, nullptr, nullptr, o, hT, n, h, slice);
}

template <typename Tin, int D>
__global__ __launch_bounds__(2 * kWalkThreads, 2)
void kda_f32_forward_roles_kernel(const Tin *__restrict__ v, const float *__restrict__ h0,
                                  const float *__restrict__ slots, float *__restrict__ o, float *__restrict__ hT, const Problem p)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    int64_t n;
    int h, slice;
    if (!place<D, 1>(p, blockIdx.x, n, h, slice)) return;
    if (threadIdx.x < kWalkThreads) {
        __builtin_amdgcn_s_setprio(1);                                        // the chain first
        forward_walk<Tin, D, 1, kNothing>(smem, p, v, h0, slots, nullptr, nullptr, nullptr, hT, n, h, slice);
    } else {
        output_role<D>(smem, p, slots, o, n, h, slice);
    }
}

// The backward walk, the longer of the two, goes first.  kHelped: four waves more, which help the backward walk (and
// leave at once in the forward one, whose chain holds every product it has).
template <typename Tin, typename Tdo, int D, int NC, bool kHelped>
__global__ __launch_bounds__(kHelped ? 2 * kWalkThreads : kWalkThreads, 2)
void kda_f32_both_walks_kernel(const Tin *__restrict__ v, const float *__restrict__ h0,
                               const Tdo *__restrict__ d_o, const float *__restrict__ d_hT, const float *__restrict__ slots,
                               float *__restrict__ S0, float *__restrict__ Rw, float *__restrict__ dS1, float *__restrict__ Zw,
                               float *__restrict__ dh0, int64_t half, const Problem p)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int64_t bid = blockIdx.x;
    int64_t n;
    int h, slice;
    if (!place<D, NC>(p, bid < half ? bid : bid - half, n, h, slice)) return;
    if (kHelped && threadIdx.x >= kWalkThreads) {
        if (bid < half) gradient_role<Tdo, D>(smem, p, d_o, slots, n, h, slice);
        return;
    }
    if (kHelped) __builtin_amdgcn_s_setprio(1);                               // the chain first
    if (bid < half) backward_walk<Tdo, D, NC, kHelped>(smem, p, d_o, d_hT, slots, dS1, Zw, dh0, n, h, slice);
    else forward_walk<Tin, D, NC, kStates>(smem, p, v, h0, slots, S0, Rw, nullptr, nullptr, n, h, slice);
}

// Column tiles per workgroup: the fewest that still give every compute unit at most two workgroups (more than two
// would queue; fewer columns than needed load the same operands more often), and at most 2 tiles at d 128, 4 at d 64: two
// workgroups of the widest fit a compute unit with their registers.  (Four tiles at d 128 take a whole one, and were never faster:
// 2048 tokens, fp32 inputs, 2 against 4 tiles, backward pass 96 pairs 975 / 1077 us, 128 pairs 1252 / 1247, 136 pairs
// 1389 / 1515, 256 pairs 2454 / 2458; prefill 136 pairs 638 / 800, 256 pairs 947 / 972.  The other lines, 1 against 2 tiles:
// backward pass d 128, 32 pairs 373 / 396, 48 pairs 563 / 568, 64 pairs 717 / 659; d 64, 64 pairs 312 / 308, 96 pairs 452 / 452,
// 128 pairs 586 / 538; prefill d 128, 32 pairs 159 / 217, 64 pairs 291 / 273, 128 pairs 550 / 489; d 64, 128 pairs 266 / 249, 256
// pairs 506 / 460.  2 against 4 tiles, d 64: backward pass 128 pairs 538 / 570, 256 pairs 1034 / 1017; prefill 256 pairs 460 / 470.)
static int column_tiles(const Problem &p, int D, int walks, int compute_units)
{
    const int widest = D == 128 ? 2 : 4;
    for (int nc = 1; nc < widest; nc *= 2)
        if (walks * walk_workgroups(p, D / (16 * nc)) <= 2 * (int64_t)compute_units) return nc;
    return widest;
}

template <typename F, typename... Args>
static kda_status launch_walk(F kern, const char *name, int64_t blocks, int threads, size_t lds, hipStream_t stream, Args... args)
{
    if (blocks > 0x7fffffffLL) return fail(KDA_ERR_UNSUPPORTED, "%s: %lld workgroups", name, (long long)blocks);
    hipError_t e = hipSuccess;
    if (lds > 65536)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3((unsigned)threads), lds, stream, args...);
        e = hipGetLastError();
    }
    return e == hipSuccess ? KDA_OK : fail(KDA_ERR_LAUNCH, "%s: %s", name, hipGetErrorString(e));
}

template <typename Tin, int D>
kda_status launch_forward_walk(const Problem &p, const Tin *v, const float *h0, const float *slots, float *o,
                               float *hT, int compute_units, hipStream_t stream)
{
#define KDA_GO(NC) launch_walk(kda_f32_forward_walk_kernel<Tin, D, NC>, "kda_f32_forward_walk", walk_workgroups(p, D / (16 * NC)), kWalkThreads, \
                               walk_lds<D, NC>(false), stream, v, h0, slots, o, hT, p)
    const int nc = column_tiles(p, D, 1, compute_units);
    // Where every workgroup of one column tile has a compute unit to itself, four more waves share its matrix cores with the
    // walking ones (16 pairs of 2048 tokens, whole call: d 64 112 -> 97 us, d 128 164 -> 141 us; 64 pairs, d 64: 161 -> 155 us).  Two such
    // workgroups do not fit a compute unit at d 128, and there two plain ones overlap as well.
    if (walk_workgroups(p, D / 16) <= compute_units)
        return launch_walk(kda_f32_forward_roles_kernel<Tin, D>, "kda_f32_forward_roles", walk_workgroups(p, D / 16), 2 * kWalkThreads,
                           walk_lds<D, 1>(false), stream, v, h0, slots, o, hT, p);
    if constexpr (D == 64)
        if (nc == 4) return KDA_GO(4);
    return nc == 1 ? KDA_GO(1) : KDA_GO(2);
#undef KDA_GO
}

template <typename Tin, typename Tdo, int D>
kda_status launch_both_walks(const Problem &p, const Tin *v, const float *h0, const Tdo *d_o, const float *d_hT,
                             const float *slots, float *S0, float *R, float *dS1, float *Z, float *dh0, int compute_units,
                             hipStream_t stream)
{
#define KDA_GO(NC, HELPED, THREADS, LDS) launch_walk(kda_f32_both_walks_kernel<Tin, Tdo, D, NC, HELPED>, "kda_f32_both_walks", \
                               2 * walk_workgroups(p, D / (16 * NC)), THREADS, LDS, stream, v, h0, d_o, d_hT, slots, S0, R, dS1, Z, dh0, \
                               walk_workgroups(p, D / (16 * NC)), p)
    const int nc = column_tiles(p, D, 2, compute_units);
    // Where every workgroup of one column tile has a compute unit to itself, four more waves help the backward walks (whole
    // pass, d 128, 4096 tokens: 4 pairs 271 -> 250 us, 16 pairs 424 -> 399 us; d 64, 32 pairs: 336 -> 326 us).
    if (2 * walk_workgroups(p, D / 16) <= compute_units)
        return KDA_GO(1, true, 2 * kWalkThreads, (size_t)(2 * (D / 16) + 16) * kFrag * 4);
    if constexpr (D == 64)
        if (nc == 4) return KDA_GO(4, false, kWalkThreads, (walk_lds<D, 4>(true)));
    return nc == 1 ? KDA_GO(1, false, kWalkThreads, (walk_lds<D, 1>(true))) : KDA_GO(2, false, kWalkThreads, (walk_lds<D, 2>(true)));
#undef KDA_GO
}

#define KDA_FWD(T, DD) template kda_status launch_forward_walk<T, DD>(const Problem &, const T *, const float *, \
                                                                      const float *, float *, float *, int, hipStream_t)
KDA_FWD(float, 64);
KDA_FWD(float, 128);
KDA_FWD(__hip_bfloat16, 64);
KDA_FWD(__hip_bfloat16, 128);
#define KDA_BOTH(T, O, DD) template kda_status launch_both_walks<T, O, DD>(const Problem &, const T *, const float *, \
    const O *, const float *, const float *, float *, float *, float *, float *, float *, int, hipStream_t)
KDA_BOTH(float, float, 64);
KDA_BOTH(float, float, 128);
KDA_BOTH(__hip_bfloat16, float, 64);
KDA_BOTH(__hip_bfloat16, float, 128);
KDA_BOTH(__hip_bfloat16, __hip_bfloat16, 64);
KDA_BOTH(__hip_bfloat16, __hip_bfloat16, 128);
#undef KDA_FWD
#undef KDA_BOTH

}  // namespace f32
}  // namespace kda
