"""bf16 prefill at the top of fp16's range: the residual v - S^T k is formed before beta and the inverse meet it, so it is larger than the
pseudo-value beta (v - S^T k) and than either of its terms; a call whose states, values and pseudo-values stay below 65504 must come out
finite and right all the same.  Against the fp64 oracle."""
import pytest
import torch

import synth_inputs as si
from helpers import check_prefill

pytestmark = pytest.mark.gpu

TOL = 2e-3          # fp16 operands, as everywhere
D = 128


@pytest.mark.parametrize("tokens", [1, 40, 100])
@pytest.mark.parametrize("v,read,beta", [
    (4.0e4, -4.0e4, 0.5),          # residual 8e4
    (6.5e4, -6.5e4, 0.5),          # residual 1.3e5, pseudo-value 6.5e4
    (-6.5e4, 6.4e4, 0.498),
    (1.0e4, -5.0e4, 1.0),
    (6.0e4, 6.5e4, 1.0),
    (0.0, 4.5e5, 0.125),           # a key along every row of the state
    (0.0, 4.5e5, 0.14),
    (0.0, 6.0e5, 0.1),
    (0.0, 6.0e5, 0.05),
])
def test_residual_beyond_fp16(v, read, beta, tokens):
    """The first token's residual is v - read in every column; its key is along all channels alike, and it does not decay the state."""
    x = si.make_prefill(1, tokens, 2, D, D, "bf16", -2.0, 17, 0.1)
    x["k"][:, 0] = D ** -0.5
    x["log_alpha"][:, 0] = 0.0
    x["v"][:, 0] = v
    x["beta"][:, 0] = beta
    k = float(x["k"][0, 0, 0, 0])
    # (and a part that this key does not read, so that the write does not leave a state near zero to compare with)
    x["h0"] = torch.full_like(x["h0"], read / (D * k)) + 6.0e3 * torch.tensor([1.0, -1.0]).repeat(D // 2)[:, None]
    states = float(x["h0"].abs().max()) + beta * abs(v - read) * k
    assert states < 65504 and abs(float(x["v"][0, 0, 0, 0])) < 65504 and beta * abs(v - read) < 65504      # the domain
    eo, eh = check_prefill(x, TOL)
    print("v %g read %g beta %g, %d tokens: err_o %.2e err_hT %.2e" % (v, read, beta, tokens, eo, eh))
