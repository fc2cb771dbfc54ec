// Building blocks of the fp32 kernels (prefill of fp32 inputs, backward pass): 16 x 16 tiles on
// v_mfma_f32_16x16x4_f32, whose operands are arranged so that four contraction steps take one 16-byte word.
//
// With m = lane % 16 and g = lane / 16 the instruction takes A[m][g] and B[g][m] from a lane and leaves
// D[4 g + j][m] in its register j.  Contraction slot g of step ks (four steps per 16-wide tile) is made to
// stand for index 4 g + ks of the tile.  Then
//
//   - an accumulator tile D is, as it stands, the B operand of the next product (register ks of lane group g is
//     row 4 g + ks), so states and pseudo-values are fed back with no data movement, and it is also the A
//     operand of its own transpose;
//   - an operand with its contraction index along memory is one float4 per lane and tile.
//
// A "fragment" is one such tile in memory: 64 lanes x float4 = 1 KiB in lane order.  "Column form" is the
// accumulator order (lane m holds rows 4 g .. 4 g + 3 of column m); "row form" is its transpose (lane m
// holds columns 4 g .. 4 g + 3 of row m).  quad_transpose turns one into the other, up to the lane order
// turned_lane(), while the tile is being loaded or stored.
#pragma once
#include "kda_common.h"

namespace kda {
namespace f32 {

constexpr int kC = kChunk;
constexpr int kFrag = 256;                                   // floats of a fragment
constexpr int kTri = 10;                                     // 16 x 16 blocks of a lower-triangular C x C matrix
__host__ __device__ constexpr int tri(int R, int I) { return R * (R + 1) / 2 + I; }      // block (R, I), I <= R

// What the per-chunk kernel leaves per (chunk, head), in floats: Gamma.K, Gamma^{i->C}.K and Gamma.Q as
// [token tile][channel tile] fragments, the blocks of Q and Tril(A_qk), e^(G_C) and beta (zero past the chunk's end).  All in
// column form where both walks read them (one of the two turns each operand as it loads it); for the prefill all but
// Gamma^{i->C}.K in row form, so that nothing is turned in the walk, whose steps are a chain: a turn is about 100 cycles
// beside the 128 of a tile's products.
template <int D> struct Slot {
    static constexpr int kTiles = D / 16;
    static constexpr int kKg = 0;
    static constexpr int kKt = kKg + 4 * kTiles * kFrag;
    static constexpr int kQg = kKt + 4 * kTiles * kFrag;
    static constexpr int kQ = kQg + 4 * kTiles * kFrag;
    static constexpr int kP = kQ + kTri * kFrag;
    static constexpr int kGc = kP + kTri * kFrag;
    static constexpr int kBeta = kGc + D;
    static constexpr int kFloats = 3 * kC * D + 2 * kC * (kC + 2) + D;       // (the published size; 13 KiB of it are spare)
    static_assert(kBeta + kC <= kFloats && kFloats % 64 == 0, "slots stay 256-byte aligned");
};

__device__ __forceinline__ f32x4 mfma16(const f32x4 &a, const f32x4 &b, f32x4 acc)      // a 16 x 16 x 16 product
{
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ks], b[ks], acc, 0, 0, 0);
    return acc;
}

// ---- fp32 products on the bf16 matrix cores ----
// A value is the exact sum of three bf16 pieces, x = h + m + l (each the rest rounded to nearest: 8 bits a piece, and |m| <= 2^-8 |x|,
// |l| <= 2^-17 |x|).  Of the nine products of two such sums six are formed, two at a time in the 32 contraction slots of one 16x16x32
// instruction (slots 8 g .. 8 g + 3 are one piece of the values 4 g .. 4 g + 3 of the tile, slots 8 g + 4 .. 8 g + 7 another); the three
// left out, m l', l m' and l l', come to at most 2^-24 of the product (and a little: 2^-24.007), the rounding of one fp32 multiplication.
// Three instructions of 16 cycles for a 16 x 16 x 16 product against four of 32 (measured: 386 against 142 TFLOP/s), fp32
// accumulation, and sums rounded less often: 2-norm error of a sum of 128 products of normal values 1.6e-7, on the fp32 instruction 2.05e-7,
// down to values of 2^-110.  Below, l (and from 2^-118 m) is a subnormal bf16, which ends at 2^-133: 2^-116 2e-6, 2^-122 1.3e-4.  Above,
// every finite value is taken; one that is not finite becomes NaN in its pieces.  Splitting a fragment costs 26 vector instructions, so it
// pays where a fragment meets several others.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct Pieces { u32x2 h, m, l; };
__device__ __forceinline__ uint32_t round_pair(float a, float b)
{
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    asm("" : "+v"(u));                                       // (or the compiler converts the halves once more by themselves)
    return u;
}
// The largest finite bf16 for anything larger: rounded up, the first piece of the largest fp32 values would be an infinity, and what is
// left of them no number.  (Backward pass at 4 x 4096 tokens x 16 heads 1.19 ms as without it, five packed sequences of 100 to 3000 tokens x 16
// heads 487.7 -> 491, 9 x 1 tokens x 32 heads 111.6 -> 112.2 us; clamping d_o alone costs as much.)
__device__ __forceinline__ float within_bf16(float x)
{
    constexpr float most = 0x1.fep127f;
    return __builtin_amdgcn_fmed3f(x, -most, most);
}
__device__ __forceinline__ Pieces split(const f32x4 &x)
{
    Pieces p;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
        const uint32_t h = round_pair(within_bf16(a), within_bf16(b));
        a -= __uint_as_float(h << 16); b -= __uint_as_float(h & 0xffff0000u);
        const uint32_t m = round_pair(a, b);
        a -= __uint_as_float(m << 16); b -= __uint_as_float(m & 0xffff0000u);
        p.h[i] = h; p.m[i] = m; p.l[i] = round_pair(a, b);
    }
    return p;
}
__device__ __forceinline__ bf16x8 slots(const u32x2 &a, const u32x2 &b)
{
    const u32x4 v = {a[0], a[1], b[0], b[1]};
    return __builtin_bit_cast(bf16x8, v);
}
// The operands of a product's instructions, for its left and its right factor; instruction k of kSteps.  (Several products go
// instruction by instruction, so that none waits for the one before it.)
struct Right {
    bf16x8 hl, mh, hm;
    __device__ __forceinline__ void set(const Pieces &p) { hl = slots(p.h, p.l); mh = slots(p.m, p.h); hm = slots(p.h, p.m); }
};
struct Left {
    static constexpr int kSteps = 3;
    bf16x8 lh, hm;
    __device__ __forceinline__ void set(const Pieces &p) { lh = slots(p.l, p.h); hm = slots(p.h, p.m); }
    __device__ __forceinline__ f32x4 step(int k, const Right &b, f32x4 acc) const
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(k == 0 ? lh : hm, k == 0 ? b.hl : k == 1 ? b.mh : b.hm, acc, 0, 0, 0);
    }
};
struct LeftExact {                                           // bf16 as it stands
    static constexpr int kSteps = 2;
    bf16x8 ox, xx;
    __device__ __forceinline__ void set(const u32x2 &x) { ox = slots(u32x2{0u, 0u}, x); xx = slots(x, x); }
    __device__ __forceinline__ f32x4 step(int k, const Right &b, f32x4 acc) const
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(k == 0 ? ox : xx, k == 0 ? b.hl : b.hm, acc, 0, 0, 0);
    }
};
// A fragment of pieces in LDS: (h, m) of the 64 lanes, then l.
constexpr int kSplitFrag = 384;                              // floats
__device__ __forceinline__ void put_pieces(float *frag, const Pieces &p, int lane)
{
    *reinterpret_cast<u32x4 *>(frag + 4 * lane) = u32x4{p.h[0], p.h[1], p.m[0], p.m[1]};
    *reinterpret_cast<u32x2 *>(frag + kFrag + 2 * lane) = p.l;
}
__device__ __forceinline__ Pieces get_pieces(const float *frag, int lane)
{
    const u32x4 x = *reinterpret_cast<const u32x4 *>(frag + 4 * lane);
    return Pieces{u32x2{x[0], x[1]}, u32x2{x[2], x[3]}, *reinterpret_cast<const u32x2 *>(frag + kFrag + 2 * lane)};
}

// 4 x 4 transpose across the lanes of a quad: lane b register j -> lane j register b.
template <int kCtrl> __device__ __forceinline__ float quad_swap(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ f32x4 quad_transpose(f32x4 r, int lane)
{
    const bool b0 = lane & 1, b1 = lane & 2;
    // (the swaps come first: in an arm of a conditional they would run with half of the lanes switched off)
    const f32x4 s = {quad_swap<0xB1>(r[0]), quad_swap<0xB1>(r[1]), quad_swap<0xB1>(r[2]), quad_swap<0xB1>(r[3])};
    const f32x4 t = {b0 ? s[1] : r[0], b0 ? r[1] : s[0], b0 ? s[3] : r[2], b0 ? r[3] : s[2]};
    const f32x4 u = {quad_swap<0x4E>(t[0]), quad_swap<0x4E>(t[1]), quad_swap<0x4E>(t[2]), quad_swap<0x4E>(t[3])};
    r[0] = b1 ? u[2] : t[0]; r[2] = b1 ? t[2] : u[0];
    r[1] = b1 ? u[3] : t[1]; r[3] = b1 ? t[3] : u[1];
    return r;
}
// The lane of the other form that a lane reads (before the quads turn) or writes (after).
__device__ __forceinline__ int turned_lane(int lane) { return ((lane >> 2) & 3) * 16 + (lane >> 4) * 4 + (lane & 3); }

__device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ void st4(float *p, const f32x4 &v) { *reinterpret_cast<f32x4 *>(p) = v; }

// Between the LDS accesses of one wave whose lanes hand each other values: the hardware keeps a wave's LDS accesses in order,
// and this keeps the compiler from moving them across (it sees each lane's addresses, not who reads what).  No instruction.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Workgroup barrier for LDS traffic: global loads and stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Loads, stores and LDS accesses stay on their side of this point; arithmetic may cross it.
__device__ __forceinline__ void pin_memory_order() { __builtin_amdgcn_sched_barrier(0x0f); }

// R and Z, [tokens x heads x D] floats in all: the rows of a (chunk, head) lie together, token tile by token tile, a tile
// of n <= 16 valid tokens as [column tile][4 columns][n tokens] float4, which for n = 16 is the fragment in row form.
__device__ __forceinline__ int64_t token_rows(int64_t tok0, int H, int h, int nv, int D) { return (tok0 * H + (int64_t)h * nv) * D; }
__device__ __forceinline__ int tile_tokens(int nv, int R) { return nv - 16 * R < 16 ? nv - 16 * R : 16; }
__device__ __forceinline__ int row_form(int R, int column_tile, int group, int token, int n, int D)
{
    return 16 * R * D + ((4 * column_tile + group) * n + token) * 4;
}

// ---- which chunk a workgroup works on ----
struct Chunk {
    int64_t tok0, slot;      // first token; workspace slot (times H + h)
    int nv, h;               // valid tokens, head
};

// First slot of sequence n: packed batches floor(cu[n] / C) + n, strictly increasing over (n, chunk) and
// bounded by floor(total / C) + N.
__device__ __forceinline__ int64_t first_slot(const int32_t *cu, int64_t n, int64_t chunks_per_seq)
{
    return cu ? (int64_t)(cu[n] / kC) + n : n * chunks_per_seq;
}

// Chunk of workgroup `bid` of a grid of (slots x heads); false: a slot that no chunk uses (past a sequence's last chunk, or
// ahead of the first sequence where that does not start at token 0).
__device__ __forceinline__ bool locate(const int32_t *cu, int num_seqs, int64_t T, int H, int64_t chunks_per_seq,
                                       int64_t bid, Chunk &c)
{
    // (32 bits, which a grid and a sequence's chunks fit: a division of 64 takes half a microsecond at the head of every workgroup)
    const int64_t s = (uint32_t)bid / (uint32_t)H;
    c.h = (int)(bid - s * H);
    c.slot = bid;
    int64_t len, c0;
    if (!cu) {
        const int64_t n = (uint32_t)s / (uint32_t)chunks_per_seq;
        c0 = (s - n * chunks_per_seq) * kC; len = T; c.tok0 = n * T + c0;
    } else {
        int lo = 0, hi = num_seqs - 1;                       // the last sequence whose first slot is <= s
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (first_slot(cu, mid, 0) <= s) lo = mid; else hi = mid - 1;
        }
        c0 = (s - first_slot(cu, lo, 0)) * kC; len = (int64_t)cu[lo + 1] - cu[lo]; c.tok0 = cu[lo] + c0;
    }
    c.nv = (int)(len - c0 < kC ? len - c0 : kC);
    return c0 >= 0 && c0 < len;
}

// ---- one 16-channel tile of a chunk in column form: register j of [R] is token 16 R + 4 g + j, channel m ----
// Every decay is summed from the log alpha it consists of, never taken as a difference of running sums (whose rounding, 2^-24
// of the decay since the chunk's start, is that of the result).  The in-block decay of a pair r >= i is split in the
// middle of the 16-token block, between its tokens 7 and 8: a row factor 2^row(R), the decay from there to token r, and a
// column factor 2^column(I), from token i to there, each below 1 on one side of the middle and above it on the other;
// a block pair R > I carries 2^across(R, I) <= 1 besides.  Both factors stay within 2^(+-kMaxDecay): nothing overflows or
// underflows, and a factor 2^x is off by |x| 2^-24 ln 2 (its exponent's rounding) and the exponential's own.  A channel
// that decays by more than 2^-kMaxDecay in one half of a block ("strong") splits at the block's two ends instead (every
// factor at most 1), contributes nothing to the diagonal products and is added there pair by pair.
// (60: a pair of blocks whose neighbouring halves both come close to it has 2^across = 2^-120, still a normal number, beside
// factors of 2^60 each.  Backward pass of 4 x 4096 tokens x 16 heads: 1.24 ms at e^-3.5 a token on average, where hardly any
// channel is strong, 1.46 ms at e^-4, 1.94 ms from e^-4.5 on, where every chunk has some.)
// (2-norm errors at log alpha = -softplus(normal - 2), d 128, against running sums over the chunk split at half of a block's
// decay: dq 3.4e-7 -> 2.3e-7, dk 3.8e-7 -> 2.4e-7, o 3.4e-7 -> 2.3e-7, hT 3.1e-7 -> 0.9e-7; dq and dk 2.9 times less at a mean
// of 0.)
constexpr float kMaxDecay = 60.f;

struct Decay {
    f32x4 x[4];                              // log alpha (0 past the end); sums are natural ones, scaled when used
    float nb[4], h1[4], h2[4];               // sums over the block's tokens: the neighbouring lane group's, either half's
    bool weak[4];                            // the channel is not strong in this block
    bool second, odd;                        // this lane's tokens lie in the block's second half; in a half's second group
    __device__ __forceinline__ f32x4 prefix(int R) const         // over the lane's own tokens: up to each, behind each
    {
        const float a = x[R][0] + x[R][1], b = a + x[R][2];
        return f32x4{x[R][0], a, b, b + x[R][3]};
    }
    __device__ __forceinline__ f32x4 suffix(int R) const
    {
        const float a = x[R][2] + x[R][3];
        return f32x4{x[R][1] + a, a, x[R][3], 0.f};
    }
    __device__ __forceinline__ float up(int R) const         // the block's groups ahead of this one
    {
        const float n = odd ? nb[R] : 0.f, h = second ? h1[R] : 0.f;
        return n + h;
    }
    __device__ __forceinline__ float before(int R) const { float s = 0.f; for (int b = 0; b < R; ++b) s += h1[b] + h2[b]; return s; }
    __device__ __forceinline__ float after(int R) const { float s = 0.f; for (int b = 3; b > R; --b) s += h1[b] + h2[b]; return s; }
    __device__ __forceinline__ f32x4 in_block(int R) const { return (prefix(R) + up(R)) * kLog2e; }
    __device__ __forceinline__ float across(int R, int I) const
    {
        const float r = weak[R] ? h1[R] : 0.f, i = weak[I] ? h2[I] : 0.f;
        float s = r + i;
        for (int b = I + 1; b < R; ++b) s += h1[b] + h2[b];
        return s * kLog2e;
    }
    __device__ __forceinline__ float whole() const { return before(4) * kLog2e; }
    __device__ __forceinline__ bool strong() const { return !(weak[0] && weak[1] && weak[2] && weak[3]); }
};

// The four exponents of a block, in log2 units: from the chunk's start to each token and from each to the chunk's end, and
// those of its row and column factors.
struct Exponents {
    f32x4 start, end, row, column;
    __device__ __forceinline__ Exponents(const Decay &d, int R)
    {
        const f32x4 p = d.prefix(R), e = d.suffix(R);
        const float up = d.up(R), dn = d.odd ? 0.f : d.nb[R], dh = d.second ? 0.f : d.h2[R], down = dn + dh;
        const float n = d.second == d.odd ? d.nb[R] : 0.f, mid = d.second ? n : -n;              // from the middle to this group
        const bool r = d.second || !d.weak[R], c = !d.second || !d.weak[R];
        const float ro = d.weak[R] ? mid : up, co = d.weak[R] ? -mid : down;
        start = (p + (up + d.before(R))) * kLog2e;
        end = (e + (down + d.after(R))) * kLog2e;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            row[j] = ((r ? p[j] : -e[j]) + ro) * kLog2e;
            column[j] = ((c ? e[j] : -p[j]) + co) * kLog2e;
        }
    }
};

// A wave brings such a tile of a [tokens, H, D] tensor in with 16-byte loads (fetch: a lane holds a piece of a row) and
// turns it through LDS (put, a fence, get: `at`, rows `ld` bytes apart, belongs to the wave alone for the moment).
template <typename T> struct TileFetch {
    static constexpr int kPerRow = (int)sizeof(T);           // 16-byte pieces of a row of 16 channels
    uint4 raw[kPerRow];
    // (the base is the workgroup's, so that the lanes' 32-bit offsets serve every tensor; 64 rows of 65535 heads fit them)
    __device__ __forceinline__ void fetch(const T *base, int64_t stride, int nv, int lane)
    {
#pragma unroll
        for (int u = 0; u < kPerRow; ++u) {
            const uint32_t r = (lane + 64 * u) / kPerRow, piece = lane % kPerRow, last = nv - 1;
            const uint32_t off = (r < last ? r : last) * (uint32_t)(stride * sizeof(T)) + 16 * piece;
            raw[u] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(base) + off);
        }
    }
    __device__ __forceinline__ void put(char *at, int ld, int nv, int lane) const
    {
#pragma unroll
        for (int u = 0; u < kPerRow; ++u) {
            const int r = (lane + 64 * u) / kPerRow, piece = lane % kPerRow;
            *reinterpret_cast<uint4 *>(at + r * ld + piece * 16) = r < nv ? raw[u] : make_uint4(0u, 0u, 0u, 0u);
        }
    }
    static __device__ __forceinline__ void get(f32x4 (&x)[4], const char *at, int ld, int lane)
    {
        const int m = lane & 15, g = lane >> 4;
#pragma unroll
        for (int R = 0; R < 4; ++R)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[R][j] = load_as_float(reinterpret_cast<const T *>(at + (16 * R + 4 * g + j) * ld) + m);
    }
    __device__ __forceinline__ void turn(f32x4 (&x)[4], char *at, int ld, int nv, int lane) const
    {
        put(at, ld, nv, lane);
        wave_lds_fence();
        get(x, at, ld, lane);
        wave_lds_fence();                                    // (the next tile comes through the same place)
    }
};

template <typename T> __device__ __forceinline__ void load_tile(f32x4 (&x)[4], const T *base, int64_t stride, int nv, int g)
{
#pragma unroll
    for (int R = 0; R < 4; ++R)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 16 * R + 4 * g + j;
            x[R][j] = load_as_float(base + (int64_t)(r < nv ? r : nv - 1) * stride);
        }
    if (nv < kC) {
#pragma unroll
        for (int R = 0; R < 4; ++R)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (16 * R + 4 * g + j >= nv) x[R][j] = 0.f;
    }
}

__device__ __forceinline__ void sum_decay(Decay &d, int lane)     // d.x holds log alpha on entry
{
    d.second = lane & 32;
    d.odd = lane & 16;
#pragma unroll
    for (int R = 0; R < 4; ++R) {
        const float own = d.prefix(R)[3];
        d.nb[R] = __shfl_xor(own, 16);
        const float mine = own + d.nb[R], other = __shfl_xor(mine, 32);
        d.h1[R] = d.second ? other : mine;
        d.h2[R] = d.second ? mine : other;
        d.weak[R] = fminf(d.h1[R], d.h2[R]) >= -kMaxDecay / kLog2e;
    }
}

__device__ __forceinline__ f32x4 exp2_4(const f32x4 &x)
{
    return f32x4{fast_exp2(x[0]), fast_exp2(x[1]), fast_exp2(x[2]), fast_exp2(x[3])};
}

constexpr int kLdT = 68;     // row stride of a C x C (or C x 64-channel) tile in LDS: 4 rows apart = 16 banks apart

// ---- launches (one per source file) ----
struct Problem {
    const int32_t *cu;
    int64_t T, chunks_per_seq, slots;      // slots: of the whole call, heads not counted
    int num_seqs, H;
    float scale;
};

template <typename Tin, int D, bool kRows>
kda_status launch_prep(const Problem &p, const Tin *q, const Tin *k, const Tin *log_alpha, const Tin *beta, float *slots,
                       hipStream_t stream);
// Forward walk that writes o and the final states.
template <typename Tin, int D>
kda_status launch_forward_walk(const Problem &p, const Tin *v, const float *h0, const float *slots, float *o,
                               float *hT, int compute_units, hipStream_t stream);
// Forward and backward walks side by side: S0 of every chunk and R = v - S^T k of every token; dS1 of every chunk,
// Z' = dV / beta of every token, dh0.
template <typename Tin, typename Tdo, int D>
kda_status launch_both_walks(const Problem &p, const Tin *v, const float *h0, const Tdo *d_o, const float *d_hT,
                             const float *slots, float *S0, float *R, float *dS1, float *Z, float *dh0, int compute_units,
                             hipStream_t stream);
template <typename Tin, typename Tdo, int D>
kda_status launch_gradients(const Problem &p, const Tin *q, const Tin *k, const Tin *log_alpha, const Tin *beta, const Tdo *d_o,
                            const float *S0, const float *R, const float *dS1, const float *Z, float *dq, float *dk, float *dv,
                            float *dla, float *dbeta, int compute_units, hipStream_t stream);

}  // namespace f32
}  // namespace kda
