"""Size of the rounding errors of the fp32 path (prefill of fp32 inputs, backward pass) at slow, moderate and fast decay.

Bounds: the 2-norm errors of a chunkwise evaluation in fp32 that keeps every decay inside a 16-token block as an exponential of
its own and adds each product's 128 terms in a sum of its own, measured on these inputs against the fp64 oracle (mean over
the seeds).  A sum taken at the size of something larger, or a decay taken as the difference of long running sums, shows here
long before it reaches the 1e-5 of the parity tests.  The path is deterministic, and so are its errors."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from helpers import to_device

pytestmark = pytest.mark.gpu

LENGTHS = [200, 70, 129, 257]
BOUNDS = {      # (head dim, mean of the decay's argument): units of 1e-7
    (128, -2.0): dict(dq=3.13, dk=3.32, dv=3.67, dlog_alpha=5.59, dbeta=4.43, o=3.11, hT=2.68),
    (64, -2.0): dict(dq=2.79, dk=3.00, dv=3.40, dlog_alpha=5.55, dbeta=3.98, o=2.77, hT=2.52),
    (128, 0.0): dict(dq=6.26, dk=6.33, dv=6.54, dlog_alpha=13.9, dbeta=6.87, o=6.37, hT=4.99),
    (64, 0.0): dict(dq=5.84, dk=5.93, dv=6.07, dlog_alpha=13.5, dbeta=6.22, o=5.90, hT=3.90),
    (128, 4.0): dict(dq=3.05, dk=3.14, dv=3.19, dlog_alpha=99.7, dbeta=3.84, o=3.12),
    (64, 4.0): dict(dq=2.57, dk=2.61, dv=2.68, dlog_alpha=97.3, dbeta=2.98, o=2.59),
}


@pytest.mark.parametrize("mean", [-2.0, 0.0, 4.0])
@pytest.mark.parametrize("D,dtype", [(64, "f32"), (128, "f32"), (128, "bf16")])
@pytest.mark.parametrize("H", [2, 24])                   # 8 and 96 pairs: few and many columns to a workgroup of the walks
def test_errors_of_the_fp32_path_stay_as_small_as_they_can_be(H, D, dtype, mean):
    import paper_2510_26692_amd as kda
    errors = {}
    for seed in range(4000, 4003):
        x = si.make_varlen(LENGTHS, H, D, D, dtype, mean, seed, 0.05)
        g = torch.Generator().manual_seed(seed)
        do = torch.randn(x["v"].shape, generator=g)
        dhT = 0.1 * torch.randn(x["h0"].shape, generator=g)
        args = [si.to_np32(x[n]) for n in ("q", "k", "v", "log_alpha", "beta")]
        kw = dict(h0=x["h0"].numpy().astype(np.float64), cu_seqlens=x["cu_seqlens"].numpy().astype(np.int64))
        ref = dict(oracle.kda_backward(*args, do.numpy(), dhT=dhT.numpy(), **kw))
        dd = to_device(x)
        dev = [dd[n] for n in ("q", "k", "v", "log_alpha", "beta")]
        got = kda.kda_chunk_bwd(*dev, do.cuda(), dhT=dhT.cuda(), h0=dd["h0"], cu_seqlens=dd["cu_seqlens"])
        if dtype == "f32":
            got["o"], got["hT"] = kda.kda_chunk_fwd(*dev, h0=dd["h0"], cu_seqlens=dd["cu_seqlens"])
            ref["o"], ref["hT"] = oracle.kda_forward(*args, **kw)
        torch.cuda.synchronize()
        for n in BOUNDS[D, mean]:
            if n in got:
                e = got[n].cpu().numpy().astype(np.float64) - ref[n]
                errors.setdefault(n, []).append(np.linalg.norm(e) / np.linalg.norm(ref[n]))
    for n, e in errors.items():
        assert np.mean(e) <= 1e-7 * BOUNDS[D, mean][n], "%s: error %.3e exceeds %.2fe-7" % (n, np.mean(e), BOUNDS[D, mean][n])


def _sums(d_o, S0):
    """sum_v S0[k][v] d_o[v], as dq of one token with k = v = beta = log alpha = 0, and the same in 64 bits."""
    import paper_2510_26692_amd as kda
    N, H, D, _ = S0.shape
    zero = torch.zeros(N, 1, H, D, device="cuda")
    got = kda.kda_chunk_bwd(zero, zero, zero, zero, zero[..., 0].contiguous(), d_o.cuda(), h0=S0.cuda(), want_dh0=False)
    torch.cuda.synchronize()
    return got["dq"][:, 0].cpu().double(), torch.einsum("nhkv,nhv->nhk", S0.double(), d_o[:, 0].double())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("value", ["0x1.fep+127", "0x1.fefffep+127", "0x1.ffp+127", "0x1.fffffep+127", "-0x1.fffffep+127"])
def test_products_from_pieces_take_every_finite_value(D, value):
    """The gradients kernel forms products from bf16 pieces of their operands.  The largest numbers lie above the largest finite bf16 (the
    first of these values), by as much as the second piece holds: the result stays finite, and right to the bound below."""
    S0 = torch.randn(2, 2, D, D, generator=torch.Generator().manual_seed(1)) * 2.0 ** -8
    d_o = torch.zeros(2, 1, 2, D)
    d_o[1, 0, 0, D // 2 + 3] = float.fromhex(value)
    got, ref = _sums(d_o, S0)
    # (one product: the pieces left out, 2^-24 of it, the sum of those kept, and what the state's pieces round)
    assert ((got - ref).abs() <= 2.0 ** -22 * ref.abs()).all()
    S0[1, 1, 5, 9] = float.fromhex(value)                             # and a state's
    d_o = torch.full((2, 1, 2, D), 2.0 ** -9)
    got, ref = _sums(d_o, S0)
    assert torch.isfinite(got).all() and ((got - ref).norm() <= 1e-6 * ref.norm())


def test_products_from_pieces_of_the_worst_significands():
    """Operands whose left-out products are largest and of one sign (2^-24.01 of each product): with the sum's own roundings, 24
    additions of positive terms of up to half a unit of 2^-23, the result stays within 2^-24 + 24 * 2^-24."""
    value = float.fromhex("0x1.00ff8p+0")
    got, ref = _sums(torch.full((1, 1, 1, 128), value), torch.full((1, 1, 128, 128), value))
    assert ((got - ref).abs() <= 25 * 2.0 ** -24 * ref).all()


@pytest.mark.parametrize("exponent", [-100, -110, -113, -116, -122, -126])
@pytest.mark.parametrize("of_state", [False, True])
def test_products_from_pieces_of_the_smallest_values(exponent, of_state):
    """Down to 2^-110 as precise as ever; below, operands (of size 2^exponent) are rounded to multiples of 2^-133, a bf16's last."""
    g = torch.Generator().manual_seed(7)
    d_o, S0 = torch.randn(3, 1, 2, 128, generator=g), torch.randn(3, 2, 128, 128, generator=g)
    if of_state:
        S0 *= 2.0 ** exponent
    else:
        d_o *= 2.0 ** exponent
    got, ref = _sums(d_o, S0)
    bound = 3e-7 if exponent >= -110 else 3e-7 + 2.0 ** (-134 - exponent)
    assert (got - ref).norm() <= bound * ref.norm()


def test_an_infinite_gradient_stays_with_its_sequence_and_head():
    g = torch.Generator().manual_seed(8)
    d_o, S0 = torch.randn(3, 1, 2, 128, generator=g), torch.randn(3, 2, 128, 128, generator=g)
    finite, _ = _sums(d_o, S0)
    d_o[1, 0, 0, 17] = float("inf")
    got, _ = _sums(d_o, S0)
    assert not torch.isfinite(got[1, 0]).any()
    got[1, 0], finite[1, 0] = 0.0, 0.0
    assert torch.equal(got, finite)
