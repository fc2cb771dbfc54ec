"""bf16 prefill with write gates that are nearly shut.  What a small beta multiplies is rounded to fp16 on its way through the matrix
cores, and keys of unit norm and scale * A_qk are small already: beta must not take them into the subnormals.  Against the
fp64 oracle, at the tolerance of every other bf16 prefill; the factors that beta is cut into keep the error near that of open gates (4.5e-4)."""
import pytest
import torch

import synth_inputs as si
from helpers import check_form, check_prefill

pytestmark = pytest.mark.gpu

TOL = 2e-3
D = 128


@pytest.mark.parametrize("scale", [1.0, D ** -0.5])
@pytest.mark.parametrize("mean", [-4.0, -6.0, -8.0, -10.0])
@pytest.mark.parametrize("form", ["plain", "scalar", "raw"])
def test_weak_beta(form, mean, scale):
    eo, eh = check_form(form, [333], 3, TOL, int(-10 * mean) + len(form), scale=scale, beta_mean=mean)
    print("%s mean %g scale %.2f: err_o %.2e err_hT %.2e" % (form, mean, scale, eo, eh))


def test_weak_beta_through_ranges():
    """The passes without outputs apply the factor of beta themselves: slow decay, so that their results count."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(1, 64 * 60 - 11, 2, D, D, "bf16", -6.0, 31, 0.0)
    x["beta"] = torch.sigmoid(torch.randn(x["beta"].shape, generator=torch.Generator().manual_seed(32)) - 8.0).to(torch.bfloat16)
    try:
        kda.kda_debug_set_time_split(8)
        eo, eh = check_prefill(x, TOL, scale=D ** -0.5)
    finally:
        kda.kda_debug_set_time_split(1)
    print("ranges: err_o %.2e err_hT %.2e" % (eo, eh))


@pytest.mark.parametrize("beta", [0.0, 2.0 ** -130, 2.0 ** -126, 2.0 ** -24, 2.0 ** -6, 2.0 ** -5, 2.0 ** -4 - 2.0 ** -12, 2.0 ** -4, 0.25 - 2.0 ** -10, 0.25,
                                  0.5, 0.5 + 2.0 ** -8, 1.0, 1.5, 2.0, 6.0])
def test_beta_at_the_edges_of_its_factors(beta):
    """One and the same beta for every token: zero, a subnormal, powers of two of odd and even exponent, their neighbours, and one
    above 1 (few tokens then: the recurrence itself grows)."""
    x = si.make_prefill(1, 150 if beta < 2.0 else 20, 2, D, D, "bf16", -2.0, 41, 0.5)
    x["beta"] = torch.full_like(x["beta"], beta)
    assert beta == 0.0 or float(x["beta"].float().max()) == beta
    eo, eh = check_prefill(x, TOL)
    print("beta %g: err_o %.2e err_hT %.2e" % (beta, eo, eh))
