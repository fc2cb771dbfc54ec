"""Outputs that the binding allocates: rows of a packed batch that belong to no sequence are zero (o and every per-token
gradient), with row sizes that are and are not a multiple of 16 bytes (dbeta has 4 H bytes a row), whether the batch has
such rows or not, and no row that does belong to a sequence is touched.  The memory is dirtied first."""
import pytest
import torch

import synth_inputs as si
from helpers import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bound", [False, True], ids=["unbounded", "bounded"])
@pytest.mark.parametrize("lens,stray", [([70, 5], 0), ([70, 5], 1), ([0, 64], 300), ([0], 3), ([9000, 900], 700), ([200], 32900)])
@pytest.mark.parametrize("H,D,dtype", [(3, 64, "f32"), (4, 128, "bf16")])
def test_unowned_rows_are_zero_and_owned_ones_are_not_touched(lens, stray, H, D, dtype, bound):
    # (outputs of more than 8 and gradients of more than 64 MiB at four heads, mostly owned and mostly not, with the longest length given or not)
    more = dict(max_seqlen=max(lens)) if bound else {}
    import paper_2510_26692_amd as kda
    x = si.make_varlen(lens + [stray], H, D, D, dtype, -2.0, 77, 0.0)
    T, owned = sum(lens) + stray, sum(lens)
    x["cu_seqlens"] = x["cu_seqlens"][:-1].contiguous()
    dd = to_device(x)
    args = [dd[n] for n in ("q", "k", "v", "log_alpha", "beta")]
    do = torch.randn(1, T, H, D, device="cuda")

    def both():
        dirt = [torch.full((1 << 22,), float("nan"), device="cuda") for _ in range(8)]
        del dirt                                        # (freed blocks that the outputs are likely to be cut from)
        o, _ = kda.kda_chunk_fwd(*args, cu_seqlens=dd["cu_seqlens"], **more)
        g = kda.kda_chunk_bwd(*args, do, cu_seqlens=dd["cu_seqlens"], want_dh0=False, **more)
        torch.cuda.synchronize()
        return dict(g, o=o)

    got = both()
    into = {n: torch.full_like(t, 7.0) for n, t in got.items() if t is not None}
    kda.kda_chunk_fwd(*args, cu_seqlens=dd["cu_seqlens"], o=into["o"], **more)
    kda.kda_chunk_bwd(*args, do, cu_seqlens=dd["cu_seqlens"], want_dh0=False, **more,
                      out=dict({n: into[n] for n in into if n != "o"}, dh0=None))
    torch.cuda.synchronize()
    for n, t in into.items():
        assert torch.equal(got[n][:, :owned], t[:, :owned]), n
        assert bool((got[n][:, owned:] == 0).all()), n
        assert bool((t[:, owned:] == 7).all()), n       # a caller's own array keeps what it held


@pytest.mark.parametrize("cu", [[3, 3], [3, 10], [0, 10], [10, 10], [-5, 12], [0, -1]])
def test_rows_on_both_sides_of_the_sequences_are_cleared_and_nothing_else(cu):
    """The clearing call alone, with ends inside, at and beyond those of the array: it never leaves the array."""
    from paper_2510_26692_amd import kda as binding
    tokens, guard = 10, 64
    low, high = min(max(cu[0], 0), tokens), min(max(cu[1], 0), tokens)
    for width in (3, 8):                                # rows of 12 and of 32 bytes
        whole = torch.full((tokens * width + 2 * guard,), 7.0, device="cuda")
        binding._clear_unowned(torch.tensor(cu, dtype=torch.int32, device="cuda"),
                               [whole[guard:guard + tokens * width].view(1, tokens, width)])
        got = whole.cpu()
        rows = got[guard:-guard].view(tokens, width)
        owned = torch.zeros(tokens, dtype=torch.bool)
        owned[low:high] = True
        assert bool((rows[owned] == 7).all()) and bool((rows[~owned] == 0).all())
        assert bool((got[:guard] == 7).all()) and bool((got[-guard:] == 7).all())


@pytest.mark.parametrize("lead", [63, 64, 200])
@pytest.mark.parametrize("H,D,dtype", [(3, 64, "f32"), (2, 128, "f32"), (4, 128, "bf16")])
def test_rows_ahead_of_the_first_sequence_take_no_part(lead, H, D, dtype):
    """cu_seqlens that starts past token 0, by less than a chunk, a whole one and several: the rows ahead (and those
    behind) are zero in outputs that the binding allocates and as they were in a caller's own, whatever the inputs hold
    there, and the sequences' rows are bit for bit those of the same sequences alone."""
    import paper_2510_26692_amd as kda
    lens, tail = [70, 0, 5, 129], 90
    x = si.make_varlen([lead] + lens + [tail], H, D, D, dtype, -2.0, 78, 0.05)
    end = lead + sum(lens)
    x["cu_seqlens"], x["h0"] = x["cu_seqlens"][1:-1].contiguous(), x["h0"][1:-1].contiguous()
    names = ("q", "k", "v", "log_alpha", "beta")
    for n in names:
        x[n][:, :lead], x[n][:, end:] = float("nan"), float("nan")
    dd = to_device(x)
    do = torch.randn(1, end + tail, H, D, device="cuda")
    dhT = 0.1 * torch.randn(len(lens), H, D, D, device="cuda")

    def both(part, cu, o=None, hT=None, out=None):
        args = [dd[n][:, part].clone() for n in names]
        o, hT = kda.kda_chunk_fwd(*args, h0=dd["h0"], cu_seqlens=cu, o=o, hT=hT)
        g = kda.kda_chunk_bwd(*args, do[:, part].clone(), dhT=dhT, h0=dd["h0"], cu_seqlens=cu, out=out)
        torch.cuda.synchronize()
        return dict(g, o=o, hT=hT)

    whole, owned = slice(0, end + tail), slice(lead, end)
    alone = both(owned, dd["cu_seqlens"] - lead)
    got = both(whole, dd["cu_seqlens"])
    into = {n: torch.full_like(t, 7.0) for n, t in got.items()}
    both(whole, dd["cu_seqlens"], into["o"], into["hT"], {n: into[n] for n in into if n not in ("o", "hT")})
    for n in got:
        if n in ("hT", "dh0"):
            assert torch.equal(got[n], alone[n]) and torch.equal(into[n], alone[n]), n
            continue
        for t, rest in ((got[n], 0.0), (into[n], 7.0)):
            assert torch.equal(t[:, owned], alone[n]), n
            assert bool((t[:, :lead] == rest).all()) and bool((t[:, end:] == rest).all()), n


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_a_refused_packed_call_says_why_whatever_its_outputs(dtype):
    """Head dims outside the built set are refused as that (a row of such an output need not be a multiple of 4 bytes)."""
    import paper_2510_26692_amd as kda
    q, b = torch.zeros(1, 1 << 23, 1, 1, dtype=dtype, device="cuda"), torch.zeros(1, 1 << 23, 1, dtype=dtype, device="cuda")
    cu = torch.tensor([0, 5], dtype=torch.int32, device="cuda")
    args, unsupported = (q, q, q, q, b), 2                 # KDA_ERR_UNSUPPORTED
    for call in (lambda: kda.kda_chunk_fwd(*args, cu_seqlens=cu, out_dtype=dtype),
                 lambda: kda.kda_chunk_bwd(*args, q, cu_seqlens=cu)):
        with pytest.raises(kda.KdaError) as e:
            call()
        assert e.value.status == unsupported
