"""GPU parity of kda_chunk_fwd against the fp64 oracle on seeded inputs."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import check_prefill, rel_err, to_device

pytestmark = pytest.mark.gpu

# fp32 path: fp32 products/accumulation over <= 128-term dot products and a 64-step
# substitution, hardware exp2 (1 ulp): errors sit near 1e-6; gate as stated for fp32.
TOL_F32 = 1e-5
# bf16 inputs: fp16 matrix-core operands (unit roundoff 2^-11) with fp32 accumulation;
# emulation of the operand roundings puts the error near 6e-4; gate as stated for bf16.
TOL_BF16 = 2e-3


def test_config0_tiny_fp32():
    c = si.CONFIGS["cfg0_tiny_fp32"]
    d = si.make_prefill(c["B"], c["T"], c["H"], c["dk"], c["dv"], c["dtype"], c["mu"], c["seed"],
                        c["h0_std"])
    eo, eh = check_prefill(d, TOL_F32)
    print("config 0: err_o %.2e err_hT %.2e" % (eo, eh))


@pytest.mark.parametrize("T", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_ragged_lengths_and_h0(T, d):
    x = si.make_prefill(2, T, 3, d, d, "f32", -1.0, 5 + T, 0.05)
    eo, eh = check_prefill(x, TOL_F32, scale=d ** -0.5)
    print("fp32 T=%d d=%d: err_o %.2e err_hT %.2e" % (T, d, eo, eh))


def test_fp32_packed_with_empty_sequence():
    lens = [70, 0, 5, 129]
    x = si.make_varlen(lens, 2, 64, 64, "f32", -1.0, 9, 0.05)
    eo, eh = check_prefill(x, TOL_F32)
    print("fp32 packed: err_o %.2e err_hT %.2e" % (eo, eh))


@pytest.mark.parametrize("T", [64, 128, 130])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_single_sequence_as_packed_batch(T, d):
    """One row given as a packed batch of one sequence (cu_seqlens = [0, T]).  The packed slot layout
    holds floor(T / 64) + 1 slots where the plain one holds ceil(T / 64); the workspace the library
    asks for covers it (check_prefill puts guard regions around the workspace, o and h_T)."""
    x = si.make_varlen([T], 2, d, d, "f32", -1.0, 40 + T + d, 0.05)
    eo, eh = check_prefill(x, TOL_F32)
    print("fp32 packed single T=%d d=%d: err_o %.2e err_hT %.2e" % (T, d, eo, eh))


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_both_kernel_paths(d):
    """With the workspace kda_chunk_fwd_workspace_size asks for, fp32 inputs run the parallel per-chunk
    kernel and the matrix-core walk; with none, the single sequential kernel.  Both against the oracle,
    and against each other."""
    import paper_2510_26692_amd as kda
    x = si.make_varlen([200, 0, 64, 321, 7], 2, d, d, "f32", -1.0, 23, 0.05)
    eo, eh = check_prefill(x, TOL_F32, scale=0.5)                            # workspace allocated by the binding
    eo2, eh2 = check_prefill(x, TOL_F32, scale=0.5, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    print("fp32 d=%d: with workspace %.2e %.2e, without %.2e %.2e" % (d, eo, eh, eo2, eh2))
    dd = to_device(x)
    a = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], cu_seqlens=dd["cu_seqlens"])
    b = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], cu_seqlens=dd["cu_seqlens"],
                          workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert rel_err(a[0].cpu().numpy(), b[0].cpu().numpy()) < 2e-5
    assert rel_err(a[1].cpu().numpy(), b[1].cpu().numpy()) < 2e-5


def test_bf16_inputs_with_head_dim_64_take_the_fp32_kernels():
    """bf16 values are exact in fp32, so the fp32 tolerance applies."""
    x = si.make_varlen([130, 64, 0, 9], 3, 64, 64, "bf16", -2.0, 24, 0.05)
    eo, eh = check_prefill(x, TOL_F32, scale=0.125)
    print("bf16 inputs, d=64: err_o %.2e err_hT %.2e" % (eo, eh))


def test_fp32_strong_decay():
    """log alpha down to about -20 per token: the pairwise log-domain products must
    neither overflow nor lose the surviving terms."""
    x = si.make_prefill(1, 130, 2, 64, 64, "f32", 0.0, 21, 0.05)
    x["log_alpha"] = (x["log_alpha"] * 6.0).contiguous()
    assert float(x["log_alpha"].min()) < -15.0
    eo, eh = check_prefill(x, TOL_F32)
    print("fp32 strong decay: err_o %.2e err_hT %.2e" % (eo, eh))


@pytest.mark.parametrize("T", [64, 200, 1024])
def test_bf16_small(T):
    x = si.make_prefill(2, T, 4, 128, 128, "bf16", -2.0, 31 + T, 0.02)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 T=%d: err_o %.2e err_hT %.2e" % (T, eo, eh))


def test_bf16_single_chunk_tail():
    x = si.make_prefill(1, 37, 2, 128, 128, "bf16", -2.0, 77, 0.02)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 T=37: err_o %.2e err_hT %.2e" % (eo, eh))


def test_bf16_packed_with_empty_sequence():
    lens = [70, 0, 5, 129, 64, 300]
    x = si.make_varlen(lens, 3, 128, 128, "bf16", -2.0, 9, 0.05)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 packed: err_o %.2e err_hT %.2e" % (eo, eh))


def test_bf16_packed_in_several_batches_of_pairs_takes_the_longest_sequences_first():
    """320 (sequence, head) pairs: more than one batch of the sequential role, so the library ranks the sequences by
    length (ties, empty sequences and a one-token sequence among them) and lays the batches out longest first.
    Results per sequence must not depend on that: against the oracle, and bit for bit against each sequence run
    alone; also in two time segments."""
    import paper_2510_26692_amd as kda
    lens = [300, 0, 64, 700, 64, 1, 129, 500, 0, 257]
    x = si.make_varlen(lens, 32, 128, 128, "bf16", -2.0, 11, 0.05)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 packed, three batches: err_o %.2e err_hT %.2e" % (eo, eh))
    dd = to_device(x)
    o, hT = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], cu_seqlens=dd["cu_seqlens"],
                              check=True)
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"], dd["cu_seqlens"])
    ws = torch.empty(int(kda.kda_chunk_fwd_workspace_size(dims) * 0.6) // 256 * 256, dtype=torch.uint8, device="cuda")
    assert kda.kda_debug_chunk_fwd_plan(dims, ws.numel())[1] == 2
    o_seg, h_seg = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                                     cu_seqlens=dd["cu_seqlens"], workspace=ws, check=True)
    assert torch.equal(o_seg, o) and torch.equal(h_seg, hT)
    cu = np.concatenate([[0], np.cumsum(lens)])
    for n, ln in enumerate(lens):
        if ln == 0:
            continue
        sl = slice(int(cu[n]), int(cu[n + 1]))
        o1, h1 = kda.kda_chunk_fwd(dd["q"][:, sl].contiguous(), dd["k"][:, sl].contiguous(), dd["v"][:, sl].contiguous(),
                                   dd["log_alpha"][:, sl].contiguous(), dd["beta"][:, sl].contiguous(),
                                   h0=dd["h0"][n:n + 1].contiguous(), check=True)
        assert torch.equal(o1, o[:, sl]) and torch.equal(h1[0], hT[n]), n


@pytest.mark.parametrize("H,batch", [(32, 96), (40, 80), (64, 90), (100, 88)])
def test_bf16_packed_results_do_not_depend_on_the_bound_of_the_lengths(H, batch):
    """Seven packed sequences in several batches of pairs: with their longest length given a per-chunk workgroup takes one chunk,
    without it, when most places of the grid are empty, four.  The same bits, and right ones."""
    import paper_2510_26692_amd as kda
    lens = [300, 290, 0, 257, 311, 320, 256]
    x = si.make_varlen(lens, H, 128, 128, "bf16", -2.0, 12, 0.05)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 packed, %d heads: err_o %.2e err_hT %.2e" % (H, eo, eh))
    dd = to_device(x)
    results = []
    for bound, per_workgroup in ((max(lens), 1), (0, 4)):
        dims = kda.kda.make_chunk_dims(dd["q"], dd["v"], dd["cu_seqlens"], max_seqlen=bound)
        assert kda.kda.kda_debug_prefill_grid(dims, True, torch.cuda.get_device_properties(0).multi_processor_count)[:2] == (batch, per_workgroup)
        results.append(kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], cu_seqlens=dd["cu_seqlens"],
                                         max_seqlen=bound, check=True))
    (o0, h0), (o1, h1) = results
    assert torch.equal(o0, o1) and torch.equal(h0, h1)


@pytest.mark.parametrize("B,T,H", [(1, 130, 128), (3, 130, 43), (5, 70, 29), (7, 64, 28), (5, 31 * 64, 13), (5, 31 * 64 + 1, 13),
                                   (5, 32 * 64, 19), (6, 32 * 64, 16)])
def test_bf16_batches_of_pairs_and_chunks_per_workgroup(B, T, H):
    """Both sides of the lines of the launch rule: 128 pairs (one batch) and 129 (two of 65 and 64), 145 (73 and 72), 196 (three:
    66, 66, 64); 65 pairs at 31 and at 32 chunks, 95 and 96 pairs at 32 chunks (four and one chunk per workgroup)."""
    eo, eh = check_prefill(si.make_prefill(B, T, H, 128, 128, "bf16", -2.0, B * T + H, 0.02), TOL_BF16)
    print("bf16 %dx%dx%d: err_o %.2e err_hT %.2e" % (B, T, H, eo, eh))


def test_bf16_strong_decay_takes_the_exact_subchunk_path():
    """Gates far stronger than the fast operands allow (sub-chunk decay below 2^-11 on
    most channels, log alpha down to about -20 per token)."""
    x = si.make_prefill(1, 200, 2, 128, 128, "bf16", 0.0, 21, 0.05)
    x["log_alpha"] = (x["log_alpha"].float() * 6.0).to(torch.bfloat16).contiguous()
    assert float(x["log_alpha"].float().min()) < -15.0
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 strong decay: err_o %.2e err_hT %.2e" % (eo, eh))


def test_bf16_mixed_decay_mu0():
    """mu = 0 gate (mean log alpha about -0.8): some channels strong, most not."""
    x = si.make_prefill(1, 512, 4, 128, 128, "bf16", 0.0, 5, 0.02)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 mu=0: err_o %.2e err_hT %.2e" % (eo, eh))


def test_bf16_segmented_workspace_matches_single_segment():
    """A workspace of the minimum size forces several time segments with the state
    carried between them; results must equal the single-segment run bit for bit."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(2, 1000, 2, 128, 128, "bf16", -2.0, 13, 0.02)
    dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
    full = kda.kda_chunk_fwd_workspace_size(dims)
    small = kda.kda_chunk_fwd_min_workspace_size(dims)
    assert 0 < small < full
    o1, h1 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"])
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    o2, h2 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                               workspace=ws)
    # and without hT, so the carry lives in the workspace
    o3, _ = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                              workspace=ws, want_hT=False)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(h1, h2) and torch.equal(o1, o3)
    with pytest.raises(kda.KdaError) as ei:
        kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"],
                          workspace=torch.empty(small - 256, dtype=torch.uint8, device="cuda"))
    assert ei.value.status == 3


def test_bf16_results_do_not_depend_on_what_the_workspace_held():
    """The sequential workgroups pick up each workspace slot when its flag goes up.  The flags are cleared
    by a kernel of the call itself, so slots and flags of an earlier call with other inputs, or garbage,
    must not matter: repeated calls give the same bits, and they match the oracle."""
    import paper_2510_26692_amd as kda
    ws = None
    for seed, fill in ((21, 0xFF), (22, None), (23, 0x01)):
        x = si.make_prefill(3, 1500, 4, 128, 128, "bf16", -2.0, seed, 0.02)
        dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
        dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
        if ws is None:
            ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
        if fill is not None:
            ws.fill_(fill)
        o1, h1 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                                   workspace=ws, check=True)
        o1, h1 = o1.clone(), h1.clone()
        o2, h2 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                                   workspace=ws, check=True)
        assert torch.equal(o1, o2) and torch.equal(h1, h2), seed
        check_prefill(x, TOL_BF16, workspace=ws)


def test_bf16_wait_that_runs_out_poisons_the_outputs_and_is_reported():
    """Failure handling of the bounded waits, forced from the host: with the per-chunk workgroups switched
    off no slot is ever produced, and with a wait limit of zero every sequential workgroup gives up at its
    first look.  Every kernel still runs to its end.  The call must not hand back stale or partial data:
    o and h_T are NaN, and kda_chunk_fwd_check reports the failure.  The next ordinary call is unaffected."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(2, 300, 3, 128, 128, "bf16", -2.0, 61, 0.02)
    dd = to_device(x)
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
    ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
    good_o, good_h = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], workspace=ws,
                                       check=True)
    good_o, good_h = good_o.clone(), good_h.clone()
    # the plain scan, and (T long enough) the time-split one: ranges too short to try the short way, and ranges that try it
    for split in (1, 8, 3):
        xs = x if split == 1 else si.make_prefill(1, 64 * (40 if split == 8 else 60), 2, 128, 128, "bf16", -2.0, 62, 0.02)
        ds = to_device(xs)
        dims_s = kda.kda.make_chunk_dims(ds["q"], ds["v"])
        ws_s = torch.empty(kda.kda_chunk_fwd_workspace_size(dims_s), dtype=torch.uint8, device="cuda")
        try:
            kda.kda_debug_set_time_split(split)
            kda.kda_debug_set_producers(0)
            kda.kda_debug_set_wait_limit(0)
            o, hT = kda.kda_chunk_fwd(ds["q"], ds["k"], ds["v"], ds["log_alpha"], ds["beta"], h0=ds["h0"], workspace=ws_s)
            torch.cuda.synchronize()
            assert torch.isnan(o).all() and torch.isnan(hT).all()
            with pytest.raises(kda.KdaError) as ei:
                kda.kda_chunk_fwd_check(dims_s, ws_s)
            assert ei.value.status == 4 and "gave up" in str(ei.value)
        finally:
            kda.kda_debug_set_producers(1)
            kda.kda_debug_set_wait_limit(200000000)
            kda.kda_debug_set_time_split(1)
    o, hT = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], workspace=ws, check=True)
    assert torch.equal(o, good_o) and torch.equal(hT, good_h)


@pytest.mark.parametrize("case", ["v_1e3", "v_1e5", "k_unnormalised"])
def test_bf16_values_at_and_beyond_the_fp16_domain(case):
    """The matrix-core operands are fp16.  |v| of 1e3 stays inside their range and must simply be right;
    |v| of 1e5 and keys with entries far above 3.9 leave it: the call must then either still match the
    oracle or report the state that overflowed (kda_chunk_fwd_check), never hand back finite wrong numbers
    without a word."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(1, 256, 2, 128, 128, "bf16", -2.0, 71, 0.02)
    if case == "v_1e3":
        x["v"] = (x["v"].float() * 1e3).to(torch.bfloat16)
    elif case == "v_1e5":
        x["v"] = (x["v"].float() * 1e5).to(torch.bfloat16)
    else:
        x["k"] = (x["k"].float() * 60.0).to(torch.bfloat16)          # entries up to ~20, |k| ~ 60
        x["beta"] = (x["beta"].float() * 1e-4).to(torch.bfloat16)    # keeps beta |k|^2 < 2, so the oracle itself stays bounded
    if case == "v_1e3":
        eo, eh = check_prefill(x, TOL_BF16)
        print("|v| ~ 1e3: err_o %.2e err_hT %.2e" % (eo, eh))
        return
    dd = to_device(x)
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
    ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
    o, hT = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], workspace=ws)
    torch.cuda.synchronize()
    reported = False
    try:
        kda.kda_chunk_fwd_check(dims, ws)
    except kda.KdaError as e:
        reported = True
        assert e.status == 1 and "fp16" in str(e), str(e)
    if not reported:
        from helpers import oracle_prefill, worst_slice_err, o_slices, state_slices
        o_ref, h_ref = oracle_prefill(x)
        assert np.isfinite(o.cpu().numpy()).all()
        assert worst_slice_err(o.cpu().numpy(), o_ref, o_slices(1, 2)) <= TOL_BF16
        assert worst_slice_err(hT.cpu().numpy(), h_ref, state_slices(1, 2)) <= TOL_BF16
    print(case, "reported" if reported else "within tolerance")


def test_bf16_prefill_inside_a_captured_graph_replays_correctly():
    """A caller may capture kda_chunk_fwd into a graph: the call is a fill kernel and one kernel whose
    workgroups hand slots to one another, all on the captured stream.  Every replay, with eager work in
    between, must reproduce the eager result bit for bit."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(2, 700, 4, 128, 128, "bf16", -2.0, 51, 0.02)
    dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
    ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
    o = torch.empty(2, 700, 4, 128, device="cuda")
    hT = torch.empty(2, 4, 128, 128, device="cuda")
    o_ref, h_ref = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], check=True)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], o=o, hT=hT,
                          workspace=ws)
    for rep in range(3):
        o.fill_(float("nan")); hT.fill_(float("nan")); ws.fill_(rep)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, o_ref) and torch.equal(hT, h_ref), rep
        # eager work between the replays
        o2, _ = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"])
        assert torch.equal(o2, o_ref)


@pytest.mark.parametrize("mu,mode,way", [(-6.0, 8, 512), (-2.0, 3, 256)])
def test_bf16_time_split_prefill_inside_a_captured_graph(mu, mode, way):
    """The same for a call whose sequential kernel is split into ranges: its workgroups wait for one
    another inside the one launch, and the words they use are cleared by a kernel of the graph, so
    a workspace full of garbage before each replay must not matter.  Once on the general way of the
    split (slow decay) and once on the short one; the status word says which was taken."""
    import paper_2510_26692_amd as kda
    T = 64 * 60 - 11
    x = si.make_prefill(1, T, 2, 128, 128, "bf16", mu, 52, 0.05)
    dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
    ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
    o = torch.empty(1, T, 2, 128, device="cuda")
    hT = torch.empty(1, 2, 128, 128, device="cuda")
    try:
        kda.kda_debug_set_time_split(mode)
        o_ref, h_ref = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], workspace=ws,
                                         check=True)
        assert kda.kda_debug_chunk_fwd_status(dims, ws) == way   # the reference really took the split path, this way
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], o=o, hT=hT,
                              workspace=ws)
        for rep in range(3):
            o.fill_(float("nan")); hT.fill_(float("nan")); ws.fill_(1 + rep)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, o_ref) and torch.equal(hT, h_ref), rep
            kda.kda_chunk_fwd_check(dims, ws)
            assert kda.kda_debug_chunk_fwd_status(dims, ws) == way
            o2, _ = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"])
            assert torch.equal(o2, o_ref)
    finally:
        kda.kda_debug_set_time_split(1)


@pytest.mark.parametrize("seed", list(range(10)))
def test_bf16_random_shapes_and_layouts(seed):
    """Seeded sweep over small problems: batch or packed layout (with empty and one-token sequences),
    any number of heads, ragged lengths, with or without initial state, slow to fast decay."""
    rng = np.random.default_rng(1000 + seed)
    H = int(rng.integers(1, 6))
    mu = float(rng.choice([-3.0, -1.0, 0.5]))
    h0_std = float(rng.choice([0.0, 0.05]))
    scale = float(rng.choice([1.0, 128 ** -0.5]))
    if rng.random() < 0.5:
        B, T = int(rng.integers(1, 4)), int(rng.integers(1, 700))
        x = si.make_prefill(B, T, H, 128, 128, "bf16", mu, 2000 + seed, h0_std)
        desc = "batch B=%d T=%d" % (B, T)
    else:
        lens = rng.integers(0, 400, int(rng.integers(1, 6)))
        lens[rng.integers(0, len(lens))] = int(rng.choice([0, 1, 64, 65]))
        if lens.sum() == 0:
            lens[0] = 3
        x = si.make_varlen(lens, H, 128, 128, "bf16", mu, 2000 + seed, h0_std)
        desc = "packed lens=%s" % lens.tolist()
    eo, eh = check_prefill(x, TOL_BF16, scale=scale)
    print("random %d: %s H=%d mu=%.1f h0=%.2f scale=%.3f: err_o %.2e err_hT %.2e" % (seed, desc, H, mu, h0_std, scale, eo, eh))


def test_bf16_decay_ladder_across_the_exact_path_threshold():
    """Channels with a fixed decay per token, chosen so that the decay over a 16-token sub-chunk is
    2^-D for D = 0 ... 48 in steps of 1.5: below D = 24 the half-decay split keeps them in the fp16
    operands, above it they take the exact fp32 path; both sides and the threshold itself are hit."""
    x = si.make_prefill(2, 300, 2, 128, 128, "bf16", -2.0, 77, 0.02)
    D = torch.arange(128, dtype=torch.float32) % 33 * 1.5                       # 0, 1.5, ..., 48
    per_token = -(D / 16.0) * float(np.log(2.0))
    x["log_alpha"] = per_token.view(1, 1, 1, 128).expand(2, 300, 2, 128).contiguous().to(torch.bfloat16)
    eo, eh = check_prefill(x, TOL_BF16)
    print("bf16 decay ladder: err_o %.2e err_hT %.2e" % (eo, eh))


SHORT_WAY, GENERAL_WAY = 256, 512                           # bits of the status word: the way pairs of a time-split call took


@pytest.mark.parametrize("case", ["three_ranges", "eight_ranges", "packed_ragged", "vanishing_transition",
                                  "vanishing_short_ranges", "mixed_ways", "twenty_ranges_short", "twenty_ranges_general",
                                  "forty_eight_pairs", "sixty_four_pairs_two_ranges"])
def test_bf16_time_split_scan(case):
    """Few (sequence, head) pairs and long sequences: the sequential kernel cuts the chunk axis into
    ranges that several workgroups walk side by side.  Where the transition of every range's last chunks
    is exactly zero, the ranges start from the offsets of those chunks (the short way); otherwise
    transition and offset of whole ranges are formed first and the true states after a fold (the general
    way).  Checked against the oracle, and against the plain scan, with which it must agree to rounding;
    the status word says which way was taken."""
    import paper_2510_26692_amd as kda
    # mu = -6: log alpha around -0.0025 per token, so a range's transition matrix is far from zero
    # and the fold of the ranges matters; mu = -2: the state is forgotten within a dozen chunks
    mode, want = 8, GENERAL_WAY
    if case == "three_ranges":
        x = si.make_prefill(1, 64 * 60 - 11, 2, 128, 128, "bf16", -6.0, 301, 0.05)
    elif case == "eight_ranges":
        x = si.make_prefill(2, 64 * 130 + 5, 1, 128, 128, "bf16", -6.0, 302, 0.05)
    elif case == "vanishing_transition":                      # four ranges of 50 chunks, tails of 32
        x = si.make_prefill(1, 64 * 200 + 9, 2, 128, 128, "bf16", -2.0, 304, 0.05)
        mode, want = 4, SHORT_WAY
    elif case == "vanishing_short_ranges":                    # five ranges of 20 chunks: the tail is the whole range
        x = si.make_prefill(1, 64 * 100 - 3, 3, 128, 128, "bf16", -2.0, 305, 0.05)
        mode, want = 5, SHORT_WAY
    elif case.startswith("twenty_ranges"):                    # one pair, 400 chunks: the fold runs through 18 middle ranges
        short = case.endswith("short")
        x = si.make_prefill(1, 64 * 400 - 30, 1, 128, 128, "bf16", -2.0 if short else -6.0, 308, 0.05)
        mode, want = 20, SHORT_WAY if short else GENERAL_WAY
    elif case == "forty_eight_pairs":                         # the most pairs that get three ranges
        x = si.make_prefill(3, 64 * 60 - 7, 16, 128, 128, "bf16", -2.0, 309, 0.05)
        mode, want = 3, SHORT_WAY
    elif case == "sixty_four_pairs_two_ranges":               # the most pairs the split is offered to
        x = si.make_prefill(4, 64 * 40 + 21, 16, 128, 128, "bf16", -2.0, 310, 0.05)
        mode, want = 2, SHORT_WAY
    elif case == "mixed_ways":                                # one head forgets, the other does not
        x = si.make_prefill(1, 64 * 120 + 1, 2, 128, 128, "bf16", -2.0, 306, 0.05)
        slow = si.make_prefill(1, 64 * 120 + 1, 2, 128, 128, "bf16", -6.0, 307, 0.05)
        x["log_alpha"][:, :, 1] = slow["log_alpha"][:, :, 1]
        mode, want = 3, SHORT_WAY | GENERAL_WAY
    else:                                                     # sequences that end before their ranges do
        x = si.make_varlen(np.array([64 * 130, 3001, 100, 0]), 1, 128, 128, "bf16", -2.0, 303, 0.05)
    try:
        kda.kda_debug_set_time_split(mode)                    # split for sure
        eo, eh = check_prefill(x, TOL_BF16)
        dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
        dims = kda.kda.make_chunk_dims(dd["q"], dd["v"], dd["cu_seqlens"])
        ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
        o1, h1 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                                   cu_seqlens=dd["cu_seqlens"], workspace=ws, check=True)
        status = kda.kda_debug_chunk_fwd_status(dims, ws)
        kda.kda_debug_set_time_split(0)
        o2, h2 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"],
                                   cu_seqlens=dd["cu_seqlens"], workspace=ws, check=True)
        status_plain = kda.kda_debug_chunk_fwd_status(dims, ws)
        torch.cuda.synchronize()
        d_o = (o1 - o2).abs().max().item() / o2.abs().max().item()
        d_h = (h1 - h2).abs().max().item() / h2.abs().max().item()
        print("time split %s: err_o %.2e err_hT %.2e; vs plain scan %.2e / %.2e; status %#x" % (case, eo, eh, d_o, d_h, status))
        assert d_o <= TOL_BF16 and d_h <= TOL_BF16
        assert status_plain == 0
        if case == "packed_ragged":
            assert status & GENERAL_WAY and status & ~(SHORT_WAY | GENERAL_WAY) == 0
        else:
            assert status == want
    finally:
        kda.kda_debug_set_time_split(1)


@pytest.mark.parametrize("B,T,H", [(6, 16384, 16), (10, 150, 8), (3, 64 * 60, 16), (1, 64 * 300, 5), (4, 4096, 16),
                                   (7, 777, 3)])
def test_bf16_workspace_of_the_advertised_size_is_one_time_segment(B, T, H):
    """kda_chunk_fwd_workspace_size is the size at which a call needs no time segments: the plan for exactly that
    many bytes must be a single segment, for pair counts whose flag area needs rounding and with or without the
    area of the time-split scan (plans only, nothing is launched)."""
    import paper_2510_26692_amd as kda
    dims = kda.kda.KdaDims(batch=B, seqlen=T, heads=H, dk=128, dv=128, chunk=64, num_seqs=B, in_dtype=1, out_dtype=0,
                           scale=1.0, max_seqlen=0)
    full = kda.kda_chunk_fwd_workspace_size(dims)
    plan = kda.kda_debug_chunk_fwd_plan(dims, full)
    assert plan[0] == (T + 63) // 64 and plan[1] == 1, plan
    assert kda.kda_debug_chunk_fwd_plan(dims, full - 256)[1] == 2


def test_bf16_two_host_threads_on_their_own_streams():
    """Two host threads, each with its own stream, workspace and inputs, call the prefill at the
    same time (the library keeps one helper stream per host thread and device).  Each result must
    equal, bit for bit, what the same inputs give when the thread runs alone."""
    import threading
    import paper_2510_26692_amd as kda
    xs = [si.make_prefill(2, 64 * 24 + 13, 4, 128, 128, "bf16", -2.0, 501 + i, 0.02) for i in range(2)]
    dev = [{k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()} for x in xs]

    def run(d, reps):
        out = None
        for _ in range(reps):
            out = kda.kda_chunk_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["beta"], h0=d["h0"], check=True)
        return out

    alone = [run(d, 1) for d in dev]
    torch.cuda.synchronize()
    results, errors = [None, None], []

    def worker(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                results[i] = run(dev[i], 20)
                torch.cuda.current_stream().synchronize()
        except Exception as e:                                   # surfaced below, in the test's thread
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i in range(2):
        assert torch.equal(results[i][0], alone[i][0]) and torch.equal(results[i][1], alone[i][1])


def test_bf16_many_caller_streams():
    """One host thread, 20 different streams in turn (more than the hardware has queues, and more than
    the library remembers), three calls on each without waiting in between: whichever stream of its
    own the library pairs a caller's stream with, every result equals the default stream's bit for bit
    and no wait gives up."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(2, 64 * 12 + 5, 4, 128, 128, "bf16", -2.0, 511, 0.02)
    d = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
    ref = kda.kda_chunk_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["beta"], h0=d["h0"], check=True)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(20)]
    dims = kda.kda.make_chunk_dims(d["q"], d["v"], None, 1.0, 0, torch.float32)
    outs = []
    for rep in range(3):
        for st in streams:
            with torch.cuda.stream(st):
                ws = torch.empty(kda.kda_chunk_fwd_workspace_size(dims), dtype=torch.uint8, device="cuda")
                o, hT = kda.kda_chunk_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["beta"], h0=d["h0"], workspace=ws)
                outs.append((o, hT, ws))
    torch.cuda.synchronize()
    for o, hT, ws in outs:
        kda.kda_chunk_fwd_check(dims, ws)
        assert torch.equal(o, ref[0]) and torch.equal(hT, ref[1])


@pytest.mark.parametrize("with_h0", [True, False])
def test_bf16_zero_tokens_returns_the_initial_state(with_h0):
    import paper_2510_26692_amd as kda
    B, H, d = 2, 3, 128
    z = lambda *shape: torch.empty(*shape, dtype=torch.bfloat16, device="cuda")
    h0 = si.make_state(B, H, d, d, 0.5, 601).cuda() if with_h0 else None
    hT = torch.full((B, H, d, d), 7.0, device="cuda")
    o, hT = kda.kda_chunk_fwd(z(B, 0, H, d), z(B, 0, H, d), z(B, 0, H, d), z(B, 0, H, d), z(B, 0, H), h0=h0, hT=hT)
    torch.cuda.synchronize()
    assert o.numel() == 0
    assert torch.equal(hT, h0 if with_h0 else torch.zeros_like(hT))


@pytest.mark.parametrize("mu,mode", [(-6.0, 8), (-2.0, 3)])
def test_bf16_time_split_scan_inside_time_segments(mu, mode):
    """A workspace of about half the full size: the call walks the time axis in three segments, and the
    sequential kernel of each segment is split into ranges; states are carried from segment to
    segment (a segment's final state goes to the array its initial state is read from).  Slow decay takes
    the general way in every segment; with fast decay and three ranges the segments take the short way (a last
    segment that ends before its ranges do would take the general one).  Checked against the oracle and
    against the single-segment call."""
    import paper_2510_26692_amd as kda
    x = si.make_prefill(2, 64 * 130 + 5, 1, 128, 128, "bf16", mu, 304, 0.05)
    dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
    dims = kda.kda.make_chunk_dims(dd["q"], dd["v"])
    full = kda.kda_chunk_fwd_workspace_size(dims)
    try:
        kda.kda_debug_set_time_split(mode)
        # the largest workspace, in steps of 5 % of the full one, that makes the call take three segments
        size = next(s_ for s_ in (int(full * f / 100) // 256 * 256 for f in range(95, 20, -5))
                    if kda.kda_debug_chunk_fwd_plan(dims, s_)[1] == 3)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        plan = kda.kda_debug_chunk_fwd_plan(dims, ws.numel())
        assert plan[1] == 3 and 3 <= plan[2] <= mode
        eo, eh = check_prefill(x, TOL_BF16, workspace=ws)
        o1, h1 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], workspace=ws,
                                   check=True)
        status = kda.kda_debug_chunk_fwd_status(dims, ws)
        o2, h2 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], check=True)
        kda.kda_debug_set_time_split(0)
        o3, h3 = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], workspace=ws,
                                   check=True)
        torch.cuda.synchronize()
    finally:
        kda.kda_debug_set_time_split(1)
    print("time split in segments (mu %.0f): err_o %.2e err_hT %.2e status %#x" % (mu, eo, eh, status))
    for o_, h_ in ((o2, h2), (o3, h3)):
        assert (o1 - o_).abs().max().item() <= TOL_BF16 * o_.abs().max().item()
        assert (h1 - h_).abs().max().item() <= TOL_BF16 * h_.abs().max().item()
    assert status == GENERAL_WAY if mu == -6.0 else status in (SHORT_WAY, SHORT_WAY | GENERAL_WAY)


@pytest.mark.parametrize("dtype,tol,d", [("f32", TOL_F32, 64), ("bf16", TOL_BF16, 128)])
@pytest.mark.parametrize("case", ["no_decay", "no_write", "full_write", "scalar_gate"])
def test_degenerate_gates(case, dtype, tol, d):
    """The special cases of Eq. (1): alpha = 1 (the delta rule without decay), beta = 0 (pure decay of
    the initial state: nothing is written), beta = 1 (every key is overwritten completely) and a
    decay shared by all channels of a head (the scalar-gate form)."""
    x = si.make_prefill(2, 3 * 64 + 17, 2, d, d, dtype, -2.0, 700 + len(case), 0.3)
    if case == "no_decay":
        x["log_alpha"] = torch.zeros_like(x["log_alpha"])
    elif case == "no_write":
        x["beta"] = torch.zeros_like(x["beta"])
    elif case == "full_write":
        x["beta"] = torch.ones_like(x["beta"])
    else:
        x["log_alpha"] = x["log_alpha"][..., :1].expand_as(x["log_alpha"]).contiguous()
    eo, eh = check_prefill(x, tol)
    print("degenerate %s %s: err_o %.2e err_hT %.2e" % (case, dtype, eo, eh))
    if case == "no_write":
        # closed form: h_T = Diag(prod alpha) h0, checked here against the GPU result directly
        import paper_2510_26692_amd as kda
        dd = {k_: (v_.cuda() if isinstance(v_, torch.Tensor) else v_) for k_, v_ in x.items()}
        _, hT = kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], h0=dd["h0"], check=True)
        G = x["log_alpha"].double().sum(dim=1)                       # [B,H,dk]
        ref = torch.exp(G)[..., None] * x["h0"].double()
        err = (hT.cpu().double() - ref).abs().max().item() / ref.abs().max().item()
        assert err <= tol, err


def test_bf16_thousands_of_short_packed_sequences():
    """3 000 packed sequences of 0 to 130 tokens (many shorter than a chunk, some empty): one grid
    row per sequence in kda_intra, one workgroup per (sequence, head) in kda_scan."""
    rng = np.random.default_rng(811)
    lens = rng.integers(0, 131, size=3000)
    lens[::97] = 0
    x = si.make_varlen(lens, 2, 128, 128, "bf16", -2.0, 812, 0.05)
    # (max_seqlen bounds the workspace: without it every sequence is sized as if it held all tokens)
    eo, eh = check_prefill(x, TOL_BF16, max_seqlen=int(lens.max()))
    print("bf16 3000 short sequences (%d tokens): err_o %.2e err_hT %.2e" % (int(lens.sum()), eo, eh))


@pytest.mark.parametrize("shape,dtype", [((1, 2, 128, 128), torch.float32), ((3, 2, 128, 128), torch.bfloat16), ((3, 2, 128), torch.float32)])
def test_an_array_too_small_for_the_final_states_is_refused(shape, dtype):
    import paper_2510_26692_amd as kda
    dd = to_device(si.make_prefill(3, 70, 2, 128, 128, "bf16", -2.0, 90, 0.05))
    with pytest.raises(ValueError):
        kda.kda_chunk_fwd(dd["q"], dd["k"], dd["v"], dd["log_alpha"], dd["beta"], hT=torch.empty(shape, dtype=dtype, device="cuda"))
