"""bf16 prefill at the edges of a chunk's rows: pairs of lanes fetch two tokens' rows by whole lines and trade halves, V goes to LDS
as rows, and the fp16 operands of a short chunk end inside a pair, a quad or a 32-token tile.  Every sequence is followed by
another one in memory, whose rows must not show in it; against the fp64 oracle."""
import pytest

import synth_inputs as si
from helpers import check_prefill

pytestmark = pytest.mark.gpu

# fp16 matrix-core operands (unit roundoff 2^-11) with fp32 accumulation: near 4.5e-4 in all, up to 1.2e-3 for the worst slice of few tokens
TOL = 2e-3


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 95, 127, 129, 193])
def test_rows_of_a_short_chunk(n):
    x = si.make_varlen([n, 5, n, 64], 3, 128, 128, "bf16", -2.0, 700 + n, 0.05)
    eo, eh = check_prefill(x, TOL, scale=0.5)
    print("n=%d: err_o %.2e err_hT %.2e" % (n, eo, eh))


@pytest.mark.parametrize("chunks", [24, 31, 47])
def test_ranges_on_the_general_way(chunks):
    """Slow decay over few pairs: transitions do not vanish, so the passes without outputs walk whole ranges, whose operands go round
    three places in LDS."""
    x = si.make_prefill(1, 64 * chunks - 7, 2, 128, 128, "bf16", -7.0, 900 + chunks, 0.02)
    eo, eh = check_prefill(x, TOL, scale=0.5)
    print("chunks=%d: err_o %.2e err_hT %.2e" % (chunks, eo, eh))
