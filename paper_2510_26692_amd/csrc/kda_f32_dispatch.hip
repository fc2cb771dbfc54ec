// Host side of the fp32 path: workspace layouts and launches of the prefill of fp32 inputs (per-chunk kernel, forward
// walk) and of the backward pass (per-chunk kernel, both walks, gradients).  No kernel lives here.  Nothing is
// allocated and the host never waits.
#include "kda_f32_tile.h"

namespace kda {

int current_compute_units();                                 // kda_prefill_dispatch.hip

namespace {

using f32::Problem;
constexpr int kC = kChunk;

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }
size_t slot_bytes(int D) { return 4 * (size_t)(D == 128 ? f32::Slot<128>::kFloats : f32::Slot<64>::kFloats); }

struct Plan {
    int64_t chunks_per_seq, max_chunks, slots;               // slots: heads not counted
    size_t S0, dS1, R, Z, ops, total;
};

// backward: all areas; forward: the per-chunk operands only.  (The sizes are the published ones, which callers keep with their
// plans and buffers; the backward pass leaves a [tokens, H, D] array and 2 C^2 + D floats per chunk and head of its own
// unused, the slots 13 KiB each.)
Plan make_plan(const kda_dims *d, bool packed, bool backward)
{
    Plan p{};
    const size_t D = (size_t)d->dk;
    p.chunks_per_seq = (d->seqlen + kC - 1) / kC;
    const int64_t longest = packed && d->max_seqlen > 0 && d->max_seqlen < d->seqlen ? d->max_seqlen : d->seqlen;
    p.max_chunks = (longest + kC - 1) / kC;
    p.slots = packed ? d->seqlen / kC + d->num_seqs : (int64_t)d->num_seqs * p.chunks_per_seq;
    const size_t n = (size_t)p.slots * d->heads;
    size_t at = 0;
    if (backward) {
        p.S0 = at;  at = up256(at + n * D * D * 4);
        p.dS1 = at; at = up256(at + n * D * D * 4);
        const size_t rows = (size_t)(packed ? d->seqlen : (int64_t)d->batch * d->seqlen) * d->heads * D * 4;
        p.R = at;   at = up256(at + rows);
        p.Z = at;   at = up256(at + rows);
        at = up256(at + rows + n * (2 * kC * kC + D) * 4);
    }
    p.ops = at;
    p.total = up256(at + n * slot_bytes(d->dk));
    return p;
}

// The size entry points do not see cu_seqlens.  A batch of one row may or may not come with it, and the
// packed layout (one extra slot per sequence) is the larger of the two, so a single row is sized as packed:
// whatever the dispatcher then lays out fits.
bool sized_as_packed(const kda_dims *d) { return d->num_seqs != d->batch || d->batch == 1; }

Problem problem(const kda_dims *d, const Plan &p, const int32_t *cu)
{
    return Problem{cu, d->seqlen, p.chunks_per_seq, p.slots, d->num_seqs, d->heads, d->scale};
}

template <typename Tin, typename Tdo, int D>
kda_status backward(const kda_dims *dm, const Plan &pl, const void *q, const void *k, const void *v, const void *la,
                    const void *beta, const float *h0, const int32_t *cu, const void *d_o, const float *d_hT, float *dq,
                    float *dk, float *dv, float *dla, float *dbeta, float *dh0, char *ws, int cus, hipStream_t stream)
{
    const Problem p = problem(dm, pl, cu);
    auto in = [](const void *x) { return static_cast<const Tin *>(x); };
    auto at = [&](size_t off) { return reinterpret_cast<float *>(ws + off); };
    const Tdo *go = static_cast<const Tdo *>(d_o);
    kda_status st = f32::launch_prep<Tin, D, false>(p, in(q), in(k), in(la), in(beta), at(pl.ops), stream);
    if (st == KDA_OK)
        st = f32::launch_both_walks<Tin, Tdo, D>(p, in(v), h0, go, d_hT, at(pl.ops), at(pl.S0), at(pl.R), at(pl.dS1),
                                                 at(pl.Z), dh0, cus, stream);
    if (st == KDA_OK)
        st = f32::launch_gradients<Tin, Tdo, D>(p, in(q), in(k), in(la), in(beta), go, at(pl.S0), at(pl.R), at(pl.dS1),
                                                at(pl.Z), dq, dk, dv, dla, dbeta, cus, stream);
    return st;
}

template <typename Tin, int D>
kda_status forward(const kda_dims *dm, const Plan &pl, const void *q, const void *k, const void *v, const void *la,
                   const void *beta, const float *h0, const int32_t *cu, float *o, float *hT, char *ws, int cus, hipStream_t stream)
{
    const Problem p = problem(dm, pl, cu);
    auto in = [](const void *x) { return static_cast<const Tin *>(x); };
    float *ops = reinterpret_cast<float *>(ws + pl.ops);
    const kda_status st = f32::launch_prep<Tin, D, true>(p, in(q), in(k), in(la), in(beta), ops, stream);
    if (st != KDA_OK) return st;
    return f32::launch_forward_walk<Tin, D>(p, in(v), h0, ops, o, hT, cus, stream);
}

}  // namespace

size_t chunk_bwd_workspace_size(const kda_dims *d) { return make_plan(d, sized_as_packed(d), true).total; }

kda_status chunk_bwd_dispatch(const kda_dims *dm, const void *q, const void *k, const void *v, const void *log_alpha,
                              const void *beta, const float *h0, const int32_t *cu, const void *d_o, const float *d_hT,
                              float *dq, float *dk, float *dv, float *dla, float *dbeta, float *dh0, void *workspace,
                              size_t workspace_bytes, hipStream_t stream)
{
    const Plan p = make_plan(dm, cu != nullptr, true);
    // (the size the library reports is the requirement, even where this call's own layout is smaller)
    const size_t need = chunk_bwd_workspace_size(dm) > p.total ? chunk_bwd_workspace_size(dm) : p.total;
    if (need > workspace_bytes || (need && !workspace))
        return fail(KDA_ERR_WORKSPACE, "kda_chunk_bwd needs %zu B of workspace, got %zu", need, workspace_bytes);
    if (p.max_chunks > 65535)
        return fail(KDA_ERR_UNSUPPORTED, "kda_chunk_bwd: sequences longer than %d tokens", 65535 * kC);
    const int cus = current_compute_units();
    if (cus <= 0) return fail(KDA_ERR_LAUNCH, "cannot query the device");
    char *ws = static_cast<char *>(workspace);
    const bool bf = dm->in_dtype == KDA_BF16;
#define KDA_BWD(TIN, TDO, DD) backward<TIN, TDO, DD>(dm, p, q, k, v, log_alpha, beta, h0, cu, d_o, d_hT, dq, dk, dv, \
                                                     dla, dbeta, dh0, ws, cus, stream)
    // d_o has dims->out_dtype: fp32, or bf16 (bf16 inputs only)
    if (dm->out_dtype == KDA_BF16)
        return dm->dk == 128 ? KDA_BWD(__hip_bfloat16, __hip_bfloat16, 128) : KDA_BWD(__hip_bfloat16, __hip_bfloat16, 64);
    if (dm->dk == 128) return bf ? KDA_BWD(__hip_bfloat16, float, 128) : KDA_BWD(float, float, 128);
    return bf ? KDA_BWD(__hip_bfloat16, float, 64) : KDA_BWD(float, float, 64);
#undef KDA_BWD
}

// The fp32 prefill with a workspace.  0 for sequences that are left to the single-kernel path of kda_chunk_f32.hip.
size_t chunk_f32_fast_workspace_size(const kda_dims *d)
{
    const Plan p = make_plan(d, sized_as_packed(d), false);
    return p.max_chunks > 65535 ? 0 : p.total;
}

kda_status chunk_f32_fast_dispatch(const kda_dims *dm, const void *q, const void *k, const void *v, const void *log_alpha,
                                   const void *beta, const float *h0, const int32_t *cu, void *o, float *hT, void *workspace,
                                   hipStream_t stream)
{
    const Plan p = make_plan(dm, cu != nullptr, false);
    const int cus = current_compute_units();
    if (cus <= 0) return fail(KDA_ERR_LAUNCH, "cannot query the device");
    char *ws = static_cast<char *>(workspace);
    float *of = static_cast<float *>(o);
    const bool bf = dm->in_dtype == KDA_BF16;
#define KDA_FWD(TIN, DD) forward<TIN, DD>(dm, p, q, k, v, log_alpha, beta, h0, cu, of, hT, ws, cus, stream)
    if (dm->dk == 128) return bf ? KDA_FWD(__hip_bfloat16, 128) : KDA_FWD(float, 128);
    return bf ? KDA_FWD(__hip_bfloat16, 64) : KDA_FWD(float, 64);
#undef KDA_FWD
}

}  // namespace kda
