"""bf16 prefill at the edges of a chunk's rows: pairs of lanes fetch two tokens' rows by whole lines and trade halves, V goes to LDS
as rows, and the fp16 operands of a short chunk end inside a pair, a quad or a 32-token tile.  Every sequence is followed by
another one in memory, whose rows must not show in it; against the fp64 oracle.  And at the edges of the ranges of a time split."""
import pytest
import torch

import synth_inputs as si
from helpers import check_form, check_prefill

pytestmark = pytest.mark.gpu

# fp16 matrix-core operands (unit roundoff 2^-11) with fp32 accumulation: near 4.5e-4 in all, up to 1.2e-3 for the worst slice of few tokens
TOL = 2e-3
GENERAL_WAY = 512                                           # bit of the status word


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 95, 127, 129, 193])
def test_rows_of_a_short_chunk(n):
    x = si.make_varlen([n, 5, n, 64], 3, 128, 128, "bf16", -2.0, 700 + n, 0.05)
    eo, eh = check_prefill(x, TOL, scale=0.5)
    print("n=%d: err_o %.2e err_hT %.2e" % (n, eo, eh))


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n", [1, 2, 15, 17, 33, 63, 65, 127])
@pytest.mark.parametrize("form", ["plain", "scalar", "raw"])
def test_rows_of_a_short_chunk_in_every_form(form, n, out_dtype):
    """The lanes trade halves at another place in each form, and the output leaves in another order in each type."""
    eo, eh = check_form(form, [n, 5, n, 64], 3, TOL, 800 + n, scale=0.5, h0_std=0.05, out_dtype=out_dtype)
    print("%s n=%d %s: err_o %.2e err_hT %.2e" % (form, n, out_dtype, eo, eh))


@pytest.mark.parametrize("chunks,steps", [(47, 16), (50, 17), (53, 18), (24, 9), (26, 10), (28, 11)])
def test_ranges_on_the_general_way(chunks, steps):
    """Slow decay: transitions do not vanish, so the passes without outputs walk whole ranges, whose operands go round three places in
    LDS.  Three ranges for sure, the middle one of every remainder mod 3; in a second sequence it has one step and the last has none, in
    a third it has two."""
    import paper_2510_26692_amd as kda
    try:
        kda.kda_debug_set_time_split(3)
        first = kda.kda_debug_chunk_fwd_plan(_dims([64 * chunks - 7] * 3, 64 * chunks - 7), 1 << 30)[3]
        lens = [64 * chunks - 7, 64 * first + 1, 64 * (first + 2)]
        x = si.make_varlen(lens, 1, 128, 128, "bf16", -7.0, 900 + chunks, 0.02)
        dims = _dims(lens, max(lens))
        ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
        plan = kda.kda_debug_chunk_fwd_plan(dims, ws.numel())
        assert plan[1] == 1 and plan[2] == 3 and plan[3] == first and plan[4] == steps, plan
        eo, eh = check_prefill(x, TOL, scale=0.5, max_seqlen=max(lens), workspace=ws)
        assert kda.kda_debug_chunk_fwd_status(dims, ws) == GENERAL_WAY
    finally:
        kda.kda_debug_set_time_split(1)
    print("chunks=%d: err_o %.2e err_hT %.2e" % (chunks, eo, eh))


def _dims(lens, longest):
    import paper_2510_26692_amd as kda
    return kda.kda.KdaDims(batch=1, seqlen=sum(lens), heads=1, dk=128, dv=128, chunk=64, num_seqs=len(lens), in_dtype=1, out_dtype=0, scale=0.5,
                           max_seqlen=longest)
