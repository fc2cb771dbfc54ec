// kda_scan4: the sequential stage of the matrix-core prefill (Section 3.1: chunk state update,
// inter- and intra-chunk output), as a device function for a workgroup of FOUR waves that needs half
// a compute unit (80 KiB of LDS, at most 256 registers per lane), so that it shares a compute unit
// with a workgroup of the per-chunk stage or with another one of its kind.
//
// Per chunk of one (sequence, head), with the operands the per-chunk stage left in the slot and V from the input:
//
//     Y = Diag(bY) (V - (Gamma.K) S)      O = (Gamma.Q) S + P Y      S <- Diag(gamma^C) S + K~^T Y
//     (P = Tril(A_qk) M, K~ = M^T (Gamma^{i->C}.K): the pseudo-value M Y is not formed)
//
// Every column of S is an independent recurrence.  Wave c owns the 32 columns 32 c .. 32 c + 31 of
// S for ALL of d_k (four 32x32 accumulator tiles), and with them the same columns of Y and O
// for both 32-token tiles: nothing is exchanged between the waves, and the B operands of every
// product (S and Y as fp16) come straight out of the wave's own accumulators.  What the waves
// share is read-only: the A operands Gamma.K, Gamma.Q, K~^T and P, 54 fragments of
// 1 KiB per chunk, which all four waves read from LDS.
//
// Operand path.  LDS holds one step's operands: Gamma.K, V, Gamma.Q and K~^T, 16 KiB each, a small piece (P
// and gamma^C, 6.5 KiB) and bY, a copy for each wave.  All of them arrive by LDS-direct loads (global_load_lds, buffer_load .. lds: no registers
// in between); a piece's place is refilled for the next step as soon as nobody reads it any more, so every piece has
// the two phases of a step it is not used in to arrive.  A step has three phases (Y; O; state update) and
// one workgroup barrier in front of each, which says two things at once: every wave's part of the phase's pieces has
// landed, and every wave is done reading the pieces of the phase before.  V is each wave's own affair: its 32 columns
// (4 KiB, rows of the input) go to its quarter of the region and are turned into accumulator order on the way to
// registers at the beginning of phase Y; that quarter is refilled as soon as they are there.  A pass without outputs has
// hardly any phase O, and no Gamma.Q: Gamma.K and K~^T go round the three places the latter leaves, each fetched a step ahead.
// (16 pairs x 47 chunks, whose ranges take the general way: 99 us with a place each, 91 so.)
//
// All vector-memory instructions of the loop are issued from inline assembly in a fixed order
// and waited for with explicit vmcnt counts (they retire in issue order), because a wait that the
// compiler derives cannot tell the loads apart and would drain the whole prefetch queue at every
// use.  The registers that such a load writes are defined and consumed inside one loop iteration.
#pragma once
#include <type_traits>

#include "kda_intra.h"

namespace kda {
namespace mfma {

// What one pass over a range of chunks computes (the time-split scan uses the last two):
//   kRoleFull   the scan itself: state from state_in (zero if NULL), outputs written
//   kRoleT      the d_k x d_k transition of the range: starts from the identity, drops V (the
//               recurrence is affine in the state: S_out = T S_in + B), writes no output
//   kRoleB      the offset of the range: starts from zero, keeps V, writes no output
// A kRoleT pass returns whether the transition it ended with is exactly zero (every other pass: false).
constexpr int kRoleFull = 0, kRoleT = 1, kRoleB = 2;

namespace scan4 {


constexpr int kBig = 16 * kFragBytes;                       // Gamma.K, V, Gamma.Q or K~^T of one chunk
constexpr int kPlaceK = 0, kPlaceV = kBig, kPlaceQ = 2 * kBig, kPlaceKt = 3 * kBig;
constexpr int kSmall = 4 * kBig;                            // byte offset of the small piece: P, gamma^C twice
constexpr int kSmallGc = 6 * kFragBytes;                    // .. gamma^C in it
// Partial mean squares of the output gate, [token tile][wave][32 tokens] fp32; kRoleT's four flags
constexpr int kRed = kSmall + kSmallGc + 2 * D * 4;
constexpr int kBy = kRed + 2 * 4 * 32 * 4;                  // bY, one copy per wave
constexpr int kLds = 80 * 1024;                             // two workgroups fit a compute unit
static_assert(kBy + 4 * kChunk * 4 <= kLds - 16, "the last word is the time-split scan's");
static_assert(kOffGc == kOffP + kSmallGc, "the small piece follows the slot layout");

// compile-time loop: f(integral_constant<int, I>) for I in [0, N)
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// ---- vector memory from inline assembly (device-scope policy sc1: the slots are written by
// workgroups of the same launch, on any die).  A slot is read once, and o is written once: both marked nt, so that they
// leave the L2 to what is wanted again.  us without / with: 4 x 4096 x 16 heads
// 217 / 205, eight packed sequences (20 000 chunks and heads) 894 / 840, gated layer 449 / 441, 2^17 tokens x 32 heads 2625 / 2588.
// (nt on the slot's stores: worse everywhere, 226 for
// the first.  On o in bf16, of whose lines an instruction writes pieces: 4 x 4096 x 16 heads 174, without 170, 8 x 2048 x 16 171 / 168.) ----
// A memory instruction may read a scalar register five wait states after a vector instruction wrote it, not before, and the compiler, which
// brings spilled scalar registers back with v_readlane, keeps that distance for its own instructions and not for
// text.  Every address therefore passes through a scalar move here (whose read is interlocked), and a descriptor, of four registers, is waited for.  (A flag load right behind
// the v_readlane of its base's upper half read from 4 GiB multiples away.  us before / now: 333 tokens x 32 heads 28.3 / 28.8, 16 pairs x 47 chunks with
// slow decay 125.8 / 126.7, 8 pairs x 24 chunks with the gate 75.8 / 76.2, 4 x 4096 x 16 heads 166, 4 x 8192 x 32 613 either way; with waits everywhere 29.3, 128.0, 78.7.)
constexpr int kCacheStream = 2;                              // nt, for stores
// Four LDS-direct loads: lane L of the wave moves 16 bytes from src + voff + 1024 j to LDS byte
// m0 + 1024 j + 16 L, j = 0..3 (the instruction offset applies to both addresses).
__device__ __forceinline__ void dma4(uint32_t m0, uint32_t voff, const uint8_t *src)
{
    const uint8_t *at;
    asm volatile("s_mov_b32 m0, %1\n\t"
                 "s_mov_b64 %0, %3\n\t"
                 "global_load_lds_dwordx4 %2, %0 sc1 nt\n\t"
                 "global_load_lds_dwordx4 %2, %0 offset:1024 sc1 nt\n\t"
                 "global_load_lds_dwordx4 %2, %0 offset:2048 sc1 nt\n\t"
                 "global_load_lds_dwordx4 %2, %0 offset:3072 sc1 nt"
                 : "=&s"(at) : "s"(m0), "v"(voff), "s"(src) : "memory", "m0");
}
// One LDS-direct load of 16 bytes per lane: LDS byte m0 + 16 L <- src[voff(L)].
__device__ __forceinline__ void dma1(uint32_t m0, uint32_t voff, const uint8_t *src)
{
    const uint8_t *at;
    asm volatile("s_mov_b32 m0, %1\n\t"
                 "s_mov_b64 %0, %3\n\t"
                 "global_load_lds_dwordx4 %2, %0 sc1 nt"
                 : "=&s"(at) : "s"(m0), "v"(voff), "s"(src) : "memory", "m0");
}
// The same of 4 bytes per lane: LDS byte m0 + 4 L <- src[voff(L)].
__device__ __forceinline__ void dma1_word(uint32_t m0, uint32_t voff, const uint8_t *src)
{
    const uint8_t *at;
    asm volatile("s_mov_b32 m0, %1\n\t"
                 "s_mov_b64 %0, %3\n\t"
                 "global_load_lds_dword %2, %0 sc1 nt"
                 : "=&s"(at) : "s"(m0), "v"(voff), "s"(src) : "memory", "m0");
}
// One LDS-direct load of 16 bytes per lane through a descriptor (zeros past its end): LDS byte m0 + 16 L <- row byte voff(L).
__device__ __forceinline__ void dma1_row(uint32_t m0, uint32_t voff, const u32x4 &rsrc)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 3\n\t"
                 "buffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(m0), "v"(voff), "s"(rsrc) : "memory", "m0");
}
__device__ __forceinline__ void load1(u32x4 &a, uint32_t voff, const uint8_t *src)
{
    const uint8_t *at;
    asm volatile("s_mov_b64 %1, %3\n\tglobal_load_dwordx4 %0, %2, %1 sc1 nt" : "=&v"(a), "=&s"(at) : "v"(voff), "s"(src) : "memory");
}
// lane i of each quad of four lanes receives the value of lane kSel[i] of the quad
template <int kCtrl> __device__ __forceinline__ float quad_perm(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
// every lane of each row of 16 lanes receives the value of the row's lane N
template <int N> __device__ __forceinline__ float row_broadcast(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + N, 0xf, 0xf, true));
}
// 4 x 4 transpose across the four lanes of a quad, one component: on entry r[q] belongs to register
// group q of this lane, on exit r[i] is what lane 4 (lane / 4) + i held for group lane % 4.
__device__ __forceinline__ void quad_transpose(float (&r)[4], int lane)
{
    const bool l0 = lane & 1, l1 = lane & 2;
    // 2 x 2 blocks across lanes that differ in bit 0 (quad_perm 1,0,3,2), then across bit 1 (2,3,0,1):
    // each lane sends the register its partner wants and puts what it receives in that register's place
#pragma unroll
    for (int b = 0; b < 4; b += 2) {
        const float t = quad_perm<0xB1>(l0 ? r[b] : r[b + 1]);
        if (l0) r[b] = t; else r[b + 1] = t;
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const float t = quad_perm<0x4E>(l1 ? r[b] : r[b + 2]);
        if (l1) r[b] = t; else r[b + 2] = t;
    }
}
__device__ __forceinline__ void load_word(uint32_t &w, uint32_t voff, const uint32_t *src)
{
    const uint32_t *at;
    asm volatile("s_mov_b64 %1, %3\n\tglobal_load_dword %0, %2, %1 sc1" : "=&v"(w), "=&s"(at) : "v"(voff), "s"(src) : "memory");
}
template <int N> __device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
// every wave's loads for the next phase have landed and every wave has left the phase before
template <int N> __device__ __forceinline__ void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    wait_vm<N>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Waits until *flag == epoch; gives up after `limit` ticks of the 100 MHz wall clock (0: at once).
// (a rare path: an ordinary load, and the wait the compiler puts behind it drains everything)
__device__ __noinline__ bool wait_flag(const uint32_t *flag, uint32_t epoch, uint64_t limit)
{
    const uint64_t t0 = wall_clock64();
    for (;;) {
        if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch) return true;
        if (wall_clock64() - t0 >= limit) return false;
        __builtin_amdgcn_s_sleep(8);
    }
}

// One pass over the chunks [c_begin, c_end) of one (sequence, head): 256 threads, kLds bytes at `lds`.
//   slot0, slot_stride   the slot of chunk c_begin and the byte distance to the next chunk's
//   v                    the input [tokens][heads][128] bf16
//   ready                flag of chunk c_begin (consecutive chunks follow); epoch: value of a raised flag
//   st_base              element offset of this lane's column in the [d_k][d_v] states: pair * D * D + 32 c + x
//   poisoned             start from NaN instead of state_in (the caller could not obtain the initial state)
//   status               word that records a wait that ran out (the state is then poisoned with NaN, so
//                        every later output of this pass and its final state are NaN)
//   kGate, gate           the output gate of Section 4 applied to O before it is stored:
//                        o <- Sigmoid(g) * RMSNorm(o) * w, the mean square taken over the d_v values of a token
//                        (the four waves of the workgroup); gate.factors: w_j Sigmoid(g_tj) as fp16 in accumulator
//                        order, as the per-chunk role leaves them, kGateSlotBytes per chunk, this pair's first
//                        chunk of the pass
struct GateParams {
    const uint8_t *factors;
    float eps;
};
template <bool kFlags, bool kOutBf16, int kRole = kRoleFull, bool kGate = false>
__device__ __forceinline__ bool kda_scan4_body(uint8_t *lds, const uint8_t *slot0, int64_t slot_stride, const uint16_t *v,
                                               const float *state_in, float *state_out, void *o, int64_t st_base,
                                               int64_t tok_base, int64_t len, int H, int64_t c_begin, int64_t c_end,
                                               int h, const uint32_t *ready, uint32_t epoch, uint32_t *status,
                                               uint64_t wait_limit, bool poisoned = false,
                                               const GateParams gate = GateParams{nullptr, 0.f})
{
    static_assert(!kGate || kRole == kRoleFull, "only a pass that writes outputs has a gate to apply");
    const int tid = threadIdx.x, lane = tid & 63;
    const int c = __builtin_amdgcn_readfirstlane(tid >> 6);       // the wave: column slice of S, Y, O
    // The chain of steps is the critical path of the whole prefill, the per-chunk workgroups that share the
    // compute unit are throughput work: the waves of this role go first where both want to issue.
    __builtin_amdgcn_s_setprio(3);
    const int x = lane & 31, hh = lane >> 5;
    const uint32_t lane16 = (uint32_t)lane * 16;
    constexpr bool kFull = kRole == kRoleFull;

    // vector-memory instructions per step, in issue order (see the loop)
    constexpr bool kTakesV = kRole != kRoleT;
    constexpr bool kRowsOut = kFull && !kOutBf16 && !kGate;       // O in the lanes as it is stored: a column per lane
    constexpr int nSt = kFull ? (kOutBf16 ? 4 : kRowsOut ? 32 : 8) : 0;
    constexpr int G0 = kGate ? 4 : 0;                             // phase Y: the step's own gate factors
    constexpr int G1 = (kFlags ? 1 : 0) + 4;                      //          K~^T of this step (no outputs: Gamma.K of the next) and a flag
    constexpr int G2 = kTakesV ? 5 : 1;                           //          V and bY of the next step
    constexpr int G3 = kFull ? 4 : 0, G5a = kGate ? 0 : nSt / 2;  // phase O: Gamma.K of the next step; the first half of this step's output
    constexpr int G4a = kFull ? 3 : 1, G4 = G4a + 4;              // phase S: the small piece, then Gamma.Q (no outputs: K~^T) of the next step;
    constexpr int G5b = nSt - G5a;                                //          the other half of the output, or all of it

    // own state tiles in accumulator order: S[t][j] = S(dk = 32 t + acc_row(j, hh), dv = 32 c + x)
    f32x16 S[4];
    auto fill_state = [&](auto value) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j) S[t][j] = value(32 * t + acc_row(j, hh));
    };
    if constexpr (kRole == kRoleT)      fill_state([&](int row) { return (row == 32 * c + x) ? 1.f : 0.f; });
    else if constexpr (kRole == kRoleB) fill_state([](int) { return 0.f; });
    // (one branch around all of the loads: asked element by element, some variants of the kernel wait for each load before the next)
    else if (state_in && !poisoned)     fill_state([&](int row) { return state_in[st_base + (int64_t)row * D]; });
    else                                fill_state([fill = poisoned ? __builtin_nanf("") : 0.f](int) { return fill; });

    if (c_begin < c_end) {
        const uint32_t lds0 = (uint32_t)(uintptr_t)lds;          // LDS byte address of the ring
        const int nsteps = (int)(c_end - c_begin);               // (a segment holds at most 65 535 chunk indices)
        const int64_t tok0 = tok_base + c_begin * kChunk, left64 = len - c_begin * kChunk;
        const int left = (int)(left64 < (1 << 30) ? left64 : (1 << 30));        // tokens from the pass's first on
        auto tokens_of = [&](int rel) __attribute__((always_inline)) { const int n = left - rel * kChunk; return n < kChunk ? n : kChunk; };
        // this wave's share of a piece: fragments 4 c .. 4 c + 3 of a big one, c and 4 + c % 2 of P and half of gamma^C
        const uint32_t voff_big = lane16 + (uint32_t)c * 4096;
        const int off_p0 = kOffP + c * 1024, off_p1 = kOffP + (4 + (c & 1)) * 1024;
        const uint32_t voff_gc = (uint32_t)lane * 4 + (uint32_t)(c & 1) * 256;
        // its 64 bytes of a row of V: load i takes 16 tokens, four lanes each
        const uint32_t v_pitch = (uint32_t)H * (D * 2);
        const uint32_t voff_v = (uint32_t)(lane >> 2) * v_pitch + (uint32_t)c * 64 + (uint32_t)(lane & 3) * 16;
        // gate factors of this wave: tiles (P, c), P = 0, 1, two 16-byte units per lane and tile
        const uint32_t voff_g = lane16 + (uint32_t)c * kGateTileBytes;
        bool gave_up = false;
        // (past the end: the last chunk once more)
        auto gate_of = [&](int rel) __attribute__((always_inline)) { return gate.factors + (int64_t)(rel < nsteps ? rel : nsteps - 1) * kGateSlotBytes; };
        auto slot_of = [&](int rel) __attribute__((always_inline)) { return slot0 + (int64_t)(rel < nsteps ? rel : nsteps - 1) * slot_stride; };
        auto flag_of = [&](int rel) __attribute__((always_inline)) { return ready + (rel < nsteps ? rel : nsteps - 1); };
        // V of a chunk, its real tokens
        auto rows_of = [&](int rel) __attribute__((always_inline)) {
            const int r = rel < nsteps ? rel : nsteps - 1;
            const uint64_t base = (uint64_t)(uintptr_t)(v + ((tok0 + r * kChunk) * H + h) * (int64_t)D);
            return u32x4{(uint32_t)uni((int)(uint32_t)base), (uint32_t)uni((int)(uint32_t)(base >> 32)) & 0xffffu,
                         (uint32_t)uni((int)((uint32_t)(tokens_of(r) - 1) * v_pitch + D * 2)), 0x00020000u};
        };
        h8 Sb[8];                                                // fp16 copy of S as it enters a step: (tau, s) -> Sb[2 tau + s]
        auto copy_state = [&](const int t, const int k) __attribute__((always_inline)) {     // a quarter of tile t
#pragma unroll
            for (int z = 0; z < 4; ++z) Sb[2 * t + k / 2][4 * (k % 2) + z] = (_Float16)S[t][4 * k + z];
        };
        // (done here: left to itself the compiler moves the copies to where they are first used, behind the barrier)
        auto pin_state = [&](const int t) __attribute__((always_inline)) { asm volatile("" : "+v"(Sb[2 * t]), "+v"(Sb[2 * t + 1])); };
        auto copy_states = [&]() __attribute__((always_inline)) {                            // of what phase Y does not copy itself
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int k = 0; k < 4; ++k) copy_state(t, k);
        };
        auto poison = [&]() __attribute__((always_inline)) {
            gave_up = true;
            if (lane == 0) __hip_atomic_fetch_or(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float bad = __builtin_nanf("");
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int j = 0; j < 16; ++j) S[t][j] = bad;
            if (!kGate) copy_states();
        };

        // (kGate, and a pass without outputs: what depends on the lane number is formed afresh in every step: carried in registers across the loop
        // these were the values too many, and a reload from scratch memory waits for every load in flight, once per
        // step; a volatile statement, or the compiler forms them once ahead of the loop all the same)
        auto lane_now = [&]() __attribute__((always_inline)) {
            int l;
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
            return l;
        };
        float by[2];                                             // bY: lane l of a row of 16 lanes holds that of the token its register l of tile P stands for
        u32x2 vt[8];                                             // V in accumulator order: registers 4 q .. 4 q + 3 of tile P in vt[4 P + q]
        // (64 bytes a token: the 32 lanes that go together read 32 different pairs of banks)
        auto get_v = [&]() __attribute__((always_inline)) {
            const int l = kFull ? lane : lane_now();
            const uint8_t *blk = lds + kPlaceV + c * 4096 + (4 * (l >> 5)) * 64 + 32 * ((l >> 4) & 1);
#pragma unroll
            for (int i = 0; i < 8; ++i) vt[i] = lds_read_tr4(blk + 8 * i * 64, 32, l);
        };
        auto get_by = [&]() __attribute__((always_inline)) {
            const int l = kFull ? lane : lane_now();
            const float *b = reinterpret_cast<const float *>(lds + kBy + c * 256) + acc_row(l & 15, l >> 5);
            by[0] = b[0]; by[1] = b[32];
        };
        // where this wave's part of a piece goes in LDS
        const uint32_t m0K = lds0 + kPlaceK + (uint32_t)c * 4096, m0V = lds0 + kPlaceV + (uint32_t)c * 4096;
        const uint32_t m0Q = lds0 + kPlaceQ + (uint32_t)c * 4096, m0Kt = lds0 + kPlaceKt + (uint32_t)c * 4096;
        // no outputs: place of Gamma.K of step n is 2 n % 3 of these, of K~^T the next one
        auto place_of = [](int i) __attribute__((always_inline)) { return (uint32_t)(i == 0 ? kPlaceK : i == 1 ? kPlaceQ : kPlaceKt); };
        const uint32_t m0By = lds0 + kBy + (uint32_t)c * 256;
        const uint32_t m0P0 = lds0 + kSmall + (uint32_t)c * 1024, m0P1 = lds0 + kSmall + (uint32_t)(4 + (c & 1)) * 1024, m0Gc = lds0 + kSmall + kSmallGc + (uint32_t)c * 256;

        // ---- prologue: the whole first slot, waited for in full ----
        uint32_t seen = epoch;
        if (kFlags && !wait_flag(flag_of(0), epoch, wait_limit)) poison();
        {
            const uint8_t *s0 = slot_of(0);
            if (kFlags) load_word(seen, 0u, flag_of(1));
            dma4(m0K, voff_big, s0 + kOffKg);
            if (kFull) {
                dma1(m0P0, lane16, s0 + off_p0);
                dma1(m0P1, lane16, s0 + off_p1);
            } else {
                dma4(place_of(1) + m0K, voff_big, s0 + kOffKt);
            }
            dma1_word(m0Gc, voff_gc, s0 + kOffGc);
            dma1_word(m0By, (uint32_t)lane * 4, s0 + kOffBy);
            if (kTakesV) {
                const u32x4 rows = rows_of(0);
#pragma unroll
                for (int j = 0; j < 4; ++j) dma1_row(m0V + j * 1024, voff_v + (uint32_t)(16 * j) * v_pitch, rows);
            }
            if (kFull) dma4(m0Q, voff_big, s0 + kOffQp);
        }
        phase_barrier<0>();
        if (!kGate) copy_states();
        bool next_ok = !kFlags || (uint32_t)__builtin_amdgcn_readfirstlane((int)seen) == epoch;

        const uint32_t o_rstride = (uint32_t)H * D * (kOutBf16 ? 2 : 4);   // bytes between consecutive tokens of o
        constexpr int LA = 4, RING = LA + 2;                     // operand fragments read ahead of the product that uses them
        // Vector-memory instructions are handed to the memory pipe one at a time between the matrix
        // products (a burst of them stalls the wave at issue, and the products behind it), in this order:
        //   phase Y  K~^T of this step, (gate: the factors of this step, G0,) the flag of the step after next (G1), V and bY of the next (G2)
        //   phase O  Gamma.K of the next step (G3), then the stores of output tile 0 (G5a; not with the gate, which needs all of it first)
        //   phase S  the small piece and Gamma.Q of the next step (G4), then the stores of tile 1, or of both (G5b)
        // (gate: the stores, all of them in phase S, ahead of the loads there: behind them they hold up the phase's end, a store of
        // bf16 rows touching 32 lines: 8 pairs x 24 chunks with the gate 77.5 -> 74.0 us, 32 pairs x 15 62.4 -> 60.9)
        // (no outputs: Gamma.K of the next step in phase Y, K~^T of the next in phase S)
        // Where the next step's operands are, moved on in phase S, where the scalar instructions hide behind the products
        int turn = 0;                                            // no outputs: 2 rel % 3
        const uint8_t *cur = slot0, *nxt = slot_of(1), *gate_cur = kGate ? gate_of(0) : nullptr;
        u32x4 rows = kTakesV ? rows_of(1) : u32x4{0u, 0u, 0u, 0u};
        uint8_t *obase = static_cast<uint8_t *>(o) + (tok0 * H + h) * (int64_t)(D * (kOutBf16 ? 2 : 4));

        for (int rel = 0; rel < nsteps; ++rel) {
            const uint32_t at_k = kFull ? kPlaceK : place_of(turn), at_kt = kFull ? kPlaceKt : place_of(turn == 2 ? 0 : turn + 1);
            const uint32_t at_next = place_of(turn == 0 ? 2 : turn - 1);          // no outputs: of Gamma.K of the next step
            const uint8_t *ldsY = lds + at_k + lane16, *ldsQ = lds + kPlaceQ + lane16, *ldsK = lds + at_kt + lane16;
            const uint8_t *ldsP = lds + kSmall + lane16;
            const int hh_step = kGate ? (lane_now() >> 5) : hh;
            // gamma^C: lane l of a row of 16 lanes holds that of the row its register l of a tile stands for
            const float *gc = reinterpret_cast<const float *>(lds + kSmall + kSmallGc) + (kGate ? acc_row(lane_now() & 15, hh_step) : acc_row(lane & 15, hh));
            u32x4 gr[4];                                         // kGate: gate factors of tiles (0, c), (1, c), two 16-byte units each
            float *red = reinterpret_cast<float *>(lds + kRed);
            if (kFlags && !next_ok && !gave_up) {
                if (!wait_flag(flag_of(rel + 1), epoch, wait_limit)) poison();
            }
            __builtin_amdgcn_sched_barrier(0);

            // ---- phase Y: Y[P] = bY (V[P] + (-Gamma.K)(P, tau, s) S(tau, s)), slot i: P = i / 8, (tau, s) = i % 8.  Tile 0 starts from
            // zero and has its V added at the end, by which time V has come through the LDS; tile 1 starts from V ----
            h8 Yb[2][2];                                         // fp16 copy of Y: registers 8 s .. 8 s + 7 of a tile are its slots of K-step s as a B operand
            f32x16 av[2];                                        // Y / bY: token tile P, columns of this wave
            auto v_of = [&](const int P, const int j) __attribute__((always_inline)) {
                const uint32_t w = vt[4 * P + j / 4][(j % 4) / 2];
                return kTakesV ? __uint_as_float((j & 1) ? (w & 0xffff0000u) : (w << 16)) : 0.f;
            };
            {
                h8 ring[RING];
                auto frag = [&](const int i) __attribute__((always_inline)) {
                    return *reinterpret_cast<const h8 *>(ldsY + frag_rts(i / 8, (i % 8) / 2, i % 2) * kFragBytes);
                };
                static_for<0, LA>([&](auto ic) __attribute__((always_inline)) { ring[decltype(ic)::value % RING] = frag(decltype(ic)::value); });
                if (kTakesV) get_v();
                get_by();
                if (kGate) { copy_state(0, 0); copy_state(0, 1); }
                av[0] = f32x16{0.f};
                static_for<0, 16>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value, P = i / 8, ks = i % 8;
                    if constexpr (i + LA < 16) ring[(i + LA) % RING] = frag(i + LA);
                    if constexpr (kGate ? P == 0 && ks < 7 : i == 2 || i == 4) {                         // (for the slot after the next, or the next)
                        constexpr int t = kGate ? (ks + 1) / 2 : 3, k = kGate ? 2 * ((ks + 1) % 2) : i - 2;
                        copy_state(t, k); copy_state(t, k + 1);
                    }
                    av[P] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ring[i % RING], Sb[ks], av[P], 0, 0, 0);
                    // tile 1 of V (slots 4 .. 7), and Y of tile 0 (slots 9 .. 12)
                    if constexpr (i >= 4 && i < 8) {
#pragma unroll
                        for (int z = 0; z < 4; ++z) av[1][4 * (i - 4) + z] = v_of(1, 4 * (i - 4) + z);
                    }
                    if constexpr (i >= 9 && i < 13) {
                        static_for<4 * (i - 9), 4 * (i - 8)>([&](auto jc) __attribute__((always_inline)) {
                            constexpr int j = decltype(jc)::value;
                            Yb[0][j / 8][j % 8] = (_Float16)((av[0][j] + v_of(0, j)) * row_broadcast<j>(by[0]));
                        });
                    }
                    // G1 (and G0, this step's gate factors) and G2, one instruction per slot; V of the next step goes over that of this
                    // one, which has to be in registers first
                    constexpr int y = i - 4 - G0;
                    if constexpr (i < 4) {
                        if (kFull) dma1(m0Kt + i * 1024, voff_big, cur + kOffKt + i * 1024);
                        else dma1(m0K + at_next + i * 1024, voff_big, nxt + kOffKg + i * 1024);
                    }
                    else if constexpr (y < 0) load1(gr[i - 4], voff_g, gate_cur + ((i - 4) / 2) * 4 * kGateTileBytes + ((i - 4) % 2) * 1024);
                    else if constexpr (y == 0) { if (kFlags) load_word(seen, (uint32_t)(rel + 2 < nsteps ? rel + 2 : nsteps - 1) * 4u, ready); }
                    else if constexpr (y <= 4 && kTakesV) {
                        if constexpr (y == 1) {
#pragma unroll
                            for (int z = 0; z < 8; ++z) asm volatile("" :: "v"(vt[z]));
                        }
                        dma1_row(m0V + (y - 1) * 1024, voff_v + (uint32_t)(16 * (y - 1)) * v_pitch, rows);
                    } else if constexpr (y == 5) {
                        asm volatile("" :: "v"(by[0]), "v"(by[1]));
                        dma1_word(m0By, (uint32_t)(kFull ? lane : lane_now()) * 4, nxt + kOffBy);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            phase_barrier<(kGate ? 0 : kFull ? G5b : G4 - G4a) + G0 + G1 + G2>();                  // Gamma.Q and the small piece of this step

            // ---- phase O: O^T[P] = S^T (Gamma.Q)(P)^T + Y^T P(P, rho)^T; between the products the state is scaled,
            // S <- Diag(gamma^C) S (the products read the fp16 copy taken in phase Y), and Y of tile 1 becomes an operand ----
            f32x16 ao[2] = {{0.f}, {0.f}};
            float gcv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) gcv[t] = gc[32 * t];
            auto scale_state = [&](auto tc, auto qc) __attribute__((always_inline)) {
                constexpr int t = decltype(tc)::value, q4 = decltype(qc)::value;
                static_for<0, 4>([&](auto zc) __attribute__((always_inline)) {
                    constexpr int j = 4 * q4 + decltype(zc)::value;
                    S[t][j] *= row_broadcast<j>(gcv[t]);
                });
            };
            auto take_y1 = [&](auto pc) __attribute__((always_inline)) {                         // a pair
                static_for<2 * decltype(pc)::value, 2 * decltype(pc)::value + 2>([&](auto jc) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value;
                    Yb[1][j / 8][j % 8] = (_Float16)(av[1][j] * row_broadcast<j>(by[1]));
                });
            };
            // O^T accumulator: lane (token 32 P + x, hh), registers 4 q .. 4 q + 3 = columns 32 c + 8 q + 4 hh + 0..3:
            // a token's 128 bytes of this wave's columns sit in two lanes, 16 bytes per register group.  Stored
            // that way, one instruction touches 32 cache lines and every line is written four times over; the
            // memory pipe pays per line.  The four lanes of a quad therefore transpose their 4 x 4 register
            // groups (between the products): afterwards lane (x, hh) holds group x % 4 of the tokens
            // 4 (x / 4) + 0..3, so that store i writes the whole line of token 4 (x / 4) + i from eight lanes:
            // eight lines per instruction, each once.
            u32x4 ot[2][4];
            auto prepare_out = [&](const int P, const int z) __attribute__((always_inline)) {
                if constexpr (!kOutBf16) {
                    float r[4] = {ao[P][z], ao[P][4 + z], ao[P][8 + z], ao[P][12 + z]};
                    quad_transpose(r, lane);
#pragma unroll
                    for (int i = 0; i < 4; ++i) ot[P][i][z] = __float_as_uint(r[i]);
                } else if (z == 0) {
                    // bf16: w[2 q4 + z] = columns 8 q4 + 4 hh + 2 z, + 1.  The two lanes of a token trade
                    // halves, so each ends up with two runs of eight consecutive columns: two stores.
                    uint32_t w[8];
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        w[2 * q4] = pack_bf16x2(ao[P][4 * q4], ao[P][4 * q4 + 1]);
                        w[2 * q4 + 1] = pack_bf16x2(ao[P][4 * q4 + 2], ao[P][4 * q4 + 3]);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const auto sw = __builtin_amdgcn_permlane32_swap(w[i], w[4 + i], false, false);
                        w[i] = sw[0]; w[4 + i] = sw[1];
                    }
#pragma unroll
                    for (int qq = 0; qq < 2; ++qq) {
                        u32x4 val = {w[2 * qq], w[2 * qq + 1], w[4 + 2 * qq], w[4 + 2 * qq + 1]};
                        ot[P][qq] = val;
                    }
                }
            };
            // The stores go through a buffer descriptor that covers the chunk's real tokens: rows of
            // tokens past the end of the sequence are dropped by the hardware, and the number of
            // store instructions does not depend on the data.
            const uint32_t nvalid = (uint32_t)tokens_of(rel);
            // (kRowsOut: one descriptor for each of four consecutive rows, so that the lanes' offsets are the same in every step)
            __amdgpu_buffer_rsrc_t orsrc[kRowsOut ? 4 : 1];
#pragma unroll
            for (int z = 0; z < (kRowsOut ? 4 : 1); ++z)
                orsrc[z] = __builtin_amdgcn_make_buffer_rsrc(obase + z * o_rstride, 0, nvalid > (uint32_t)z ? (int)((nvalid - z) * o_rstride) : 0, 0x00020000);
            // fp32: store i of tile P: token 32 P + 4 (x / 4) + i, columns 32 c + 8 (x % 4) + 4 hh + 0..3
            // bf16: store qq of tile P: token 32 P + x, columns 32 c + 8 (qq + 2 hh) + 0..7
            // kRowsOut: group q of tile P, register z: token 32 P + 8 q + 4 hh + z, column 32 c + x
            auto out_offset = [&](const int l) __attribute__((always_inline)) {
                const int xl = l & 31, hl = l >> 5;
                return kRowsOut ? (uint32_t)(4 * hl) * o_rstride + (uint32_t)(32 * c + xl) * 4
                       : kOutBf16 ? (uint32_t)xl * o_rstride + (uint32_t)(32 * c + 16 * hl) * 2
                                  : (uint32_t)(xl & ~3) * o_rstride + (uint32_t)(32 * c + 8 * (xl & 3) + 4 * hl) * 4;
            };
            uint32_t ol = kGate ? 0u : out_offset(lane);
            // store k of tile P, k = 0 .. nSt / 2 - 1
            auto put_out = [&](auto Pc, auto kc) __attribute__((always_inline)) {
                constexpr int P = decltype(Pc)::value, k = decltype(kc)::value;
                if constexpr (kRowsOut)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ao[P][k]), orsrc[k % 4], (int)(ol + (uint32_t)(32 * P + 8 * (k / 4)) * o_rstride), 0, kCacheStream);
                else
                    __builtin_amdgcn_raw_buffer_store_b128(ot[P][k], orsrc[0], (int)(ol + (uint32_t)(32 * P) * o_rstride + (kOutBf16 ? (uint32_t)k * 16 : (uint32_t)k * o_rstride)), 0, kOutBf16 ? 0 : kCacheStream);
            };
            // those of tile P whose turn is slot i when they are spread over slots first .. last
            auto put_share = [&](auto Pc, auto ic, auto firstc, auto lastc) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, first = decltype(firstc)::value, n = decltype(lastc)::value - first + 1, all = nSt / 2;
                if constexpr (i >= first && i < first + n)
                    static_for<(i - first) * all / n, (i - first + 1) * all / n>([&](auto kc) __attribute__((always_inline)) { put_out(Pc, kc); });
            };
            if constexpr (kFull) {
                h8 ring[RING];
                // output tile 0, then tile 1: Gamma.Q (P, tau, s), slots 0 .. 7 and 10 .. 17, and P (0,0,s), slots 8 .. 9, (1,0,s) (1,1,s), 18 .. 21
                constexpr auto q_of = [](int i) { return i < 8 ? i : i >= 10 && i < 18 ? i - 2 : -1; };
                auto frag = [&](const int i) __attribute__((always_inline)) {
                    const int qi = q_of(i);
                    if (qi < 0) return *reinterpret_cast<const h8 *>(ldsP + (i < 10 ? i - 8 : i - 16) * kFragBytes);
                    return *reinterpret_cast<const h8 *>(ldsQ + frag_rts(qi / 8, (qi % 8) / 2, qi % 2) * kFragBytes);
                };
                static_for<0, LA>([&](auto ic) __attribute__((always_inline)) { ring[decltype(ic)::value % RING] = frag(decltype(ic)::value); });
                static_for<0, 22>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value, qi = q_of(i), rr = i < 10 ? 0 : 1, ri = i < 20 ? 0 : 1;
                    if constexpr (i + LA < 22) ring[(i + LA) % RING] = frag(i + LA);
                    const h8 &b = qi >= 0 ? Sb[qi & 7] : Yb[ri][i % 2];
                    ao[rr] = kRowsOut ? __builtin_amdgcn_mfma_f32_32x32x16_f16(ring[i % RING], b, ao[rr], 0, 0, 0)
                                      : __builtin_amdgcn_mfma_f32_32x32x16_f16(b, ring[i % RING], ao[rr], 0, 0, 0);
                    if constexpr (qi >= 0) scale_state(std::integral_constant<int, qi / 4>{}, std::integral_constant<int, qi % 4>{});
                    if constexpr (i < 8) take_y1(ic);
                    if constexpr (i < 4) dma1(m0K + i * 1024, voff_big, nxt + kOffKg + i * 1024);      // G3
                    if constexpr (G5a > 0) {                                                           // G5a
                        if constexpr (!kRowsOut && i == 11) prepare_out(0, 0);
                        put_share(std::integral_constant<int, 0>{}, ic, std::integral_constant<int, 12>{}, std::integral_constant<int, 21>{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            } else {
                static_for<0, 8>([&](auto ic) __attribute__((always_inline)) { take_y1(ic); });
                static_for<0, 16>([&](auto ic) __attribute__((always_inline)) {
                    scale_state(std::integral_constant<int, decltype(ic)::value / 4>{}, std::integral_constant<int, decltype(ic)::value % 4>{});
                });
            }
            if (kGate) {
                // A token's 128 outputs sit in two lanes of each of the four waves: lane-local sum of squares, the
                // two lanes by a swap, the four waves through LDS (the barrier that ends the phase publishes it).
                const int ln = lane_now();
#pragma unroll
                for (int P = 0; P < 2; ++P) {
                    float ssq = 0.f;
#pragma unroll
                    for (int j = 0; j < 16; ++j) ssq = fmaf(ao[P][j], ao[P][j], ssq);
                    ssq += __shfl_xor(ssq, 32);
                    if (ln < 32) red[(P * 4 + c) * 32 + ln] = ssq;
                }
                // (the barrier below waits for vector memory only: the LDS stores above are waited for here)
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            // O <- Sigmoid(g) * RMSNorm(O) * w on tile P, in place (phase S, before the tile is turned for the stores)
            auto apply_gate = [&](const int P) __attribute__((always_inline)) {
                const int xl = lane_now() & 31;
                const float tot = red[(P * 4 + 0) * 32 + xl] + red[(P * 4 + 1) * 32 + xl] + red[(P * 4 + 2) * 32 + xl] +
                                  red[(P * 4 + 3) * 32 + xl];
                const float rstd = __builtin_amdgcn_rsqf(tot * (1.0f / D) + gate.eps);
#pragma unroll
                for (int half = 0; half < 2; ++half)
#pragma unroll
                    for (int wd = 0; wd < 4; ++wd) {
                        // word wd of unit `half`: columns 32 c + 8 q4 + 4 hh + 2 w, + 1 with q4 = 2 half + wd / 2, w = wd % 2
                        // (through a scalar: a bit cast applied to a vector element directly reads element 0)
                        const uint32_t w2 = gr[2 * P + half][wd];
                        const h2 pr = __builtin_bit_cast(h2, w2);
                        const int idx = 4 * (2 * half + (wd >> 1)) + 2 * (wd & 1);
                        ao[P][idx] *= rstd * (float)pr[0];
                        ao[P][idx + 1] *= rstd * (float)pr[1];
                    }
            };
            if (kGate) ol = out_offset(lane_now());
            phase_barrier<(kFull ? 0 : G1) + G2 + G3 + G5a>();                      // K~^T of this step (kGate: and its factors)

            // ---- phase S: S += K~^T Y (S is already scaled), slot i: tau = i / 4, (rho, s) = i % 4, so that
            // a tile that is done becomes an operand of the next step while the next ones are formed.  The small piece and
            // Gamma.Q of the next step go out first, then this step's output ----
            {
                h8 ring[RING];
                auto frag = [&](const int i) __attribute__((always_inline)) {
                    return *reinterpret_cast<const h8 *>(ldsK + frag_trs(i / 4, (i % 4) / 2, i % 2) * kFragBytes);
                };
                static_for<0, LA>([&](auto ic) __attribute__((always_inline)) { ring[decltype(ic)::value % RING] = frag(decltype(ic)::value); });
                static_for<0, 16>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value, tau = i / 4, rho = (i % 4) / 2, s = i % 2;
                    if constexpr (i + LA < 16) ring[(i + LA) % RING] = frag(i + LA);
                    S[tau] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ring[i % RING], Yb[rho][s], S[tau], 0, 0, 0);
                    constexpr int z = kGate ? i - 9 : i;                                               // G4
                    const uint8_t *ahead = kGate ? cur : nxt;                                          // (slot 8 moves them on)
                    if constexpr (kFull && z == 0) dma1(m0P0, lane16, ahead + off_p0);
                    else if constexpr (kFull && z == 1) dma1(m0P1, lane16, ahead + off_p1);
                    else if constexpr (z == 2) dma1_word(m0Gc, voff_gc, ahead + kOffGc);
                    if constexpr (!kFull && i >= 4 && i < 8) dma1(m0K + at_k + (i - 4) * 1024, voff_big, ahead + kOffKt + (i - 4) * 1024);
                    if constexpr (kGate ? i >= 12 : kFull && (kRowsOut ? i < 4 : i >= 4 && i < 8)) dma1(m0Q + (i % 4) * 1024, voff_big, ahead + kOffQp + (i % 4) * 1024);
                    if constexpr (kGate && (i == 0 || i == 4)) apply_gate(i / 4);
                    if constexpr (kGate) {                                                             // G5b
                        if constexpr (i < 8) prepare_out(i / 4, i % 4);
                        put_share(std::integral_constant<int, 0>{}, ic, std::integral_constant<int, kOutBf16 ? 1 : 4>{}, std::integral_constant<int, kOutBf16 ? 4 : 7>{});
                        put_share(std::integral_constant<int, 1>{}, ic, std::integral_constant<int, kOutBf16 ? 5 : 8>{}, std::integral_constant<int, kOutBf16 ? 8 : 11>{});
                    } else if constexpr (kFull) {
                        if constexpr (!kRowsOut && i == 7) prepare_out(1, 0);
                        put_share(std::integral_constant<int, 1>{}, ic, std::integral_constant<int, kRowsOut ? 4 : 8>{}, std::integral_constant<int, 15>{});
                    }
                    if constexpr (!kGate && i >= 6) {
                        if constexpr (i < 14) copy_state((i - 6) / 4, (i - 6) % 4);
                        else { copy_state(2, 2 * (i - 14)); copy_state(2, 2 * (i - 14) + 1); }
                        if constexpr (i == 9 || i == 13 || i == 15) pin_state((i - 6) / 4);
                    }
                    if constexpr (i == 8) {
                        // (past the last step but one, the last chunk's again)
                        const bool more = rel + 2 < nsteps;
                        cur = nxt;
                        nxt += more ? slot_stride : 0;
                        if (kGate) gate_cur += kGateSlotBytes;
                        if (kTakesV && more) {
                            const uint64_t base = ((uint64_t)rows[1] << 32 | rows[0]) + (uint64_t)v_pitch * kChunk;
                            rows[0] = (uint32_t)base; rows[1] = (uint32_t)(base >> 32);
                            rows[2] = (uint32_t)(tokens_of(rel + 2) - 1) * v_pitch + D * 2;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                turn = turn == 0 ? 2 : turn - 1;
                if (kFull) obase += (int64_t)o_rstride * kChunk;
            }

            // kRoleT, every eighth step: has this wave's slice of the transition vanished, bit for bit?  Decay takes a
            // range's transition to exact zero within a few chunks (S is scaled by gamma^C every step and what the
            // products add is formed from it), and zero stays zero under every further step, so the rest of the range
            // need not be walked.  Every wave still loads its share of the operands for the others, so the four
            // waves leave together: flags through LDS.
            const bool probe = kRole == kRoleT && (rel & 7) == 7;
            if (probe) {
                uint32_t bits = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int j = 0; j < 16; ++j) bits |= __float_as_uint(S[t][j]);
                const bool zero = __builtin_amdgcn_ballot_w64((bits & 0x7fffffffu) != 0) == 0;
                if (lane == 0) reinterpret_cast<uint32_t *>(red)[c] = zero ? 1u : 0u;
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }

            // ---- the next step's Gamma.K and V are here; note whether the flag read in phase Y was up ----
            phase_barrier<G5a + G4 + G5b>();
            if (kFlags) next_ok = (uint32_t)__builtin_amdgcn_readfirstlane((int)seen) == epoch;
            if (probe) {
                const uint32_t *zf = reinterpret_cast<const uint32_t *>(red);
                const bool all_zero = (zf[0] & zf[1] & zf[2] & zf[3]) != 0;
                // (nobody writes the next flags before everybody has read these: eight steps of barriers lie between)
                if (all_zero) break;                             // the same answer in every thread of the workgroup
            }
        }
        // the loads issued for a step that does not exist (clamped to the last slot) must not land after the
        // workgroup has given its LDS back
        wait_vm<0>();
    }

    // A state that is not finite at the end of the pass means that an fp16 operand overflowed on the way
    // (values outside the documented domain) or that a wait ran out: recorded as bit 1 of the status word.
    {
        bool bad = false;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j) bad |= !(__builtin_fabsf(S[t][j]) < __builtin_inff());
        if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0)
            __hip_atomic_fetch_or(status, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (state_out && (state_out != state_in || c_begin < c_end)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j)
                state_out[st_base + (int64_t)(32 * t + acc_row(j, hh)) * D] = S[t][j];
    }
    bool vanished = false;
    if (kRole == kRoleT) {
        // the transition as it stands at the end of the pass, whichever way the loop was left: all four slices zero?
        uint32_t bits = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j) bits |= __float_as_uint(S[t][j]);
        const bool zero = __builtin_amdgcn_ballot_w64((bits & 0x7fffffffu) != 0) == 0;
        volatile uint32_t *zf = reinterpret_cast<volatile uint32_t *>(lds);
        __syncthreads();                                         // nobody reads operands from the LDS any more
        if (lane == 0) zf[c] = zero ? 1u : 0u;
        __syncthreads();
        vanished = (zf[0] & zf[1] & zf[2] & zf[3]) != 0;
        __syncthreads();                                         // the words are free again
    }
    return vanished;
}

}  // namespace scan4
}  // namespace mfma
}  // namespace kda
