"""The fp32 path (prefill of fp32 inputs, backward pass) where its tiling can go wrong: token tiles of 16 and chunks
of 64 with one token less and one more, each form of the walks (a helped workgroup of one column tile, or 1, 2 or, at d 64,
4 tiles to a workgroup, chosen by the number of (sequence, head) pairs and by the device's compute units), channels whose decay
inside 16 tokens is beyond what the factors of the products hold next to channels where it is not, and tokens with
beta = 0.

Bounds: a factor 2^x of a decay held in fp32 carries a relative error of |x| 2^-24 ln 2 (x in log2 units); with the
mild decay |x| stays below 60 in a chunk and the bound is the path's 1e-5.  The strong channels, and those with single strong
tokens, reach |x| = 320 and more, where the products underflow, but at |x| = 100 they still count:
100 * 2^-24 * ln 2 = 4e-6 per factor, a few of them to a term: 4e-5, as for the other strong-decay case of the backward pass."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from helpers import rel_err, to_device

pytestmark = pytest.mark.gpu

LENGTHS = [1, 15, 16, 17, 63, 64, 65, 127, 130]
REPEATS = [1, 3, 5, 9, 15, 30]                            # x 9 sequences x 1 head: 9, 27, 45, 81, 135 and 270 pairs


def _walk_form(D, walks, pairs, compute_units):
    """The rule of kda_f32_walk.hip: workgroups of a compute unit each are helped, then the fewest tiles that leave two, up to
    the most of which two workgroups fit a compute unit."""
    widest = 2 if D == 128 else 4
    groups = lambda tiles: walks * -(-pairs // 8) * 8 * (D // (16 * tiles))
    if groups(1) <= compute_units:
        return "helped"
    return next((n for n in (1, 2) if n < widest and groups(n) <= 2 * compute_units), widest)


def test_the_pair_counts_below_reach_every_form_of_the_walks():
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for D in (64, 128):
        for walks in (1, 2):                              # the prefill's; the backward pass's two side by side
            forms = {_walk_form(D, walks, 9 * r, units) for r in REPEATS}
            assert forms == ({"helped", 1, 2} if D == 128 else {"helped", 1, 2, 4}), (D, walks, units, forms)


def _inputs(lens, H, D, dtype, decay, seed):
    x = si.make_varlen(lens, H, D, D, dtype, -2.0, seed, 0.05)
    la = x["log_alpha"].float()
    if decay == "strong":                       # every fifth channel decays by 2^-8 per token and more
        la[..., ::5] = la[..., ::5] * 2.0 - 6.0
    elif decay == "spikes":                     # single tokens around 2^-60, where a channel turns strong, and beyond
        size = torch.tensor([-30.0, -41.25, -41.5, -41.75, -60.0, -100.0])
        # (the first and last tokens of the halves of a 16-token block; both halves that meet at a block's end and around its
        # middle, with tokens between them that see each other almost undecayed)
        for at, tokens in enumerate([(0,), (7,), (8, 14), (1, 14), (6, 9)]):
            for token in tokens:
                part = la[:, token::16, :, at::5]
                part[:] = size[torch.arange(part.shape[-1]) % 6]
    elif decay == "steep":                      # every token alike, around where a half of a block turns strong
        la[..., ::2] = la[..., ::2] * 0.5 - torch.linspace(4.0, 5.5, la[..., ::2].shape[-1])
    x["log_alpha"] = la.to(x["log_alpha"].dtype)
    x["beta"][:, ::7] = 0.0
    return x


@pytest.mark.parametrize("decay", ["mild", "strong", "spikes", "steep"])
@pytest.mark.parametrize("D,dtype,do_dtype", [(64, "f32", "f32"), (128, "f32", "f32"), (128, "bf16", "f32"), (128, "bf16", "bf16"),
                                              (64, "bf16", "f32"), (64, "bf16", "bf16")])
@pytest.mark.parametrize("repeat", REPEATS)
def test_tiles_of_the_fp32_path(repeat, D, dtype, do_dtype, decay):
    import paper_2510_26692_amd as kda
    x = _inputs(LENGTHS * repeat, 1, D, dtype, decay, 1300 + repeat)
    tol = 1e-5 if decay == "mild" else 4e-5
    g = torch.Generator().manual_seed(5)
    do = torch.randn(x["v"].shape, generator=g).to(torch.bfloat16 if do_dtype == "bf16" else torch.float32)
    dhT = 0.1 * torch.randn(x["h0"].shape, generator=g)
    dd = to_device(x)
    args = [si.to_np32(x[n]) for n in ("q", "k", "v", "log_alpha", "beta")]
    kw = dict(h0=x["h0"].numpy().astype(np.float64), cu_seqlens=x["cu_seqlens"].numpy().astype(np.int64))
    dev = [dd[n] for n in ("q", "k", "v", "log_alpha", "beta")]
    if do_dtype == "f32" and (dtype == "f32" or D == 64):      # (bf16 inputs with d 128 take other kernels)
        o, hT = kda.kda_chunk_fwd(*dev, h0=dd["h0"], cu_seqlens=dd["cu_seqlens"], max_seqlen=max(LENGTHS))
        torch.cuda.synchronize()
        o_ref, h_ref = oracle.kda_forward(*args, **kw)
        assert rel_err(o.cpu().numpy(), o_ref) <= tol and rel_err(hT.cpu().numpy(), h_ref) <= tol
    got = kda.kda_chunk_bwd(*dev, do.cuda(), dhT=dhT.cuda(), h0=dd["h0"], cu_seqlens=dd["cu_seqlens"], max_seqlen=max(LENGTHS))
    torch.cuda.synchronize()
    ref = oracle.kda_backward(*args, do.float().numpy(), dhT=dhT.numpy(), **kw)
    for name in ref:
        e = rel_err(got[name].cpu().numpy(), ref[name])
        assert e <= tol, "%s: error %.3e exceeds %.1e" % (name, e, tol)
