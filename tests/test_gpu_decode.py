"""GPU parity of kda_recurrent_step against the fp64 oracle (Eq. (1), one token)."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from helpers import rel_err, state_slices, worst_slice_err

pytestmark = pytest.mark.gpu

# fp32 arithmetic on both the state and the token vectors: the only differences
# from the fp64 oracle are fp32 rounding of ~dk products per output and the
# hardware exp2 (1 ulp), so errors sit near 1e-6; the gate is the stated one.
TOL_F32 = 1e-5
TOL_BF16 = 2e-3


def _run_steps(N, H, d, dtype, steps, seed, scale=1.0):
    import paper_2510_26692_amd as kda
    S0 = si.make_state(N, H, d, d, 0.02, seed)
    S_gpu = S0.cuda().clone()
    S_ref = S0.numpy().astype(np.float64)
    worst_o = 0.0
    for s in range(steps):
        tok = si.make_decode_tokens(N, H, d, d, dtype, -2.0, seed, s)
        g = {k_: v_.cuda() for k_, v_ in tok.items()}
        o = kda.kda_recurrent_step(g["q"], g["k"], g["v"], g["log_alpha"], g["beta"], S_gpu, scale=scale)
        o_ref, S_ref = oracle.kda_step(si.to_np32(tok["q"]), si.to_np32(tok["k"]), si.to_np32(tok["v"]),
                                       si.to_np32(tok["log_alpha"]), si.to_np32(tok["beta"]), S_ref,
                                       scale=scale)
        worst_o = max(worst_o, worst_slice_err(o.cpu().numpy(), o_ref, state_slices(N, H)))
    torch.cuda.synchronize()
    err_S = worst_slice_err(S_gpu.cpu().numpy(), S_ref, state_slices(N, H))
    return worst_o, err_S


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype,tol", [("f32", TOL_F32), ("bf16", TOL_BF16)])
def test_decode_small(d, dtype, tol):
    eo, eS = _run_steps(N=3, H=5, d=d, dtype=dtype, steps=7, seed=11, scale=0.7)
    print("decode d=%d %s: err_o %.2e err_S %.2e" % (d, dtype, eo, eS))
    assert eo <= tol and eS <= tol


def test_decode_config4_full_size_100_steps():
    """256 sequences x 32 heads, 128x128 fp32 states (512 MiB), 100 steps with fresh
    bf16 tokens; the state after the last step and the last o are checked."""
    import paper_2510_26692_amd as kda
    cfg = si.CONFIGS["cfg4_decode_bf16"]
    N, H, d, steps = cfg["N"], cfg["H"], cfg["dk"], cfg["steps"]
    S0 = si.make_state(N, H, d, d, cfg["state_std"], cfg["seed"])
    S_gpu = S0.cuda().clone()
    S_ref = S0.numpy().astype(np.float64)
    for s in range(steps):
        tok = si.make_decode_tokens(N, H, d, d, cfg["dtype"], cfg["mu"], cfg["seed"], s)
        g = {k_: v_.cuda() for k_, v_ in tok.items()}
        o = kda.kda_recurrent_step(g["q"], g["k"], g["v"], g["log_alpha"], g["beta"], S_gpu)
        o_ref, S_ref = oracle.kda_step(si.to_np32(tok["q"]), si.to_np32(tok["k"]), si.to_np32(tok["v"]),
                                       si.to_np32(tok["log_alpha"]), si.to_np32(tok["beta"]), S_ref)
    torch.cuda.synchronize()
    eS = worst_slice_err(S_gpu.cpu().numpy(), S_ref, state_slices(N, H))
    eo = worst_slice_err(o.cpu().numpy(), o_ref, state_slices(N, H))
    print("config 4: err_S %.2e err_o(last) %.2e" % (eS, eo))
    assert eS <= TOL_BF16 and eo <= TOL_BF16


def test_decode_rejects_bad_arguments():
    import paper_2510_26692_amd as kda
    q = torch.zeros(2, 2, 128, device="cuda")
    S = torch.zeros(2, 2, 128, 128, device="cuda")
    b = torch.zeros(2, 2, device="cuda")
    with pytest.raises(ValueError):
        kda.kda_recurrent_step(q, q, q, q, b, S[:, :, :64])
    q96 = torch.zeros(2, 2, 96, device="cuda")
    S96 = torch.zeros(2, 2, 96, 96, device="cuda")
    with pytest.raises(kda.KdaError) as ei:
        kda.kda_recurrent_step(q96, q96, q96, q96, b, S96)
    assert ei.value.status == 2


def _stack_tokens(N, H, d, dtype, Tq, seed):
    toks = [si.make_decode_tokens(N, H, d, d, dtype, -2.0, seed, t) for t in range(Tq)]
    return {k_: torch.stack([t_[k_] for t_ in toks], dim=1).contiguous() for k_ in toks[0]}


@pytest.mark.parametrize("Tq", [1, 3, 8])
@pytest.mark.parametrize("dtype,tol,d", [("f32", TOL_F32, 64), ("bf16", TOL_BF16, 128)])
def test_pooled_multi_token_decode(Tq, dtype, tol, d):
    """Sequences name states of a larger pool through a permuted index array with skipped entries;
    each takes Tq tokens through its state in one call.  Checked against the oracle: o, the named
    states, and that every other state of the pool is bit-for-bit untouched."""
    import paper_2510_26692_amd as kda
    N, H, P = 6, 4, 11
    pool0 = si.make_state(P, H, d, d, 0.02, 31)
    idx = torch.tensor([7, 2, -1, 10, 0, 5], dtype=torch.int32)
    tok = _stack_tokens(N, H, d, dtype, Tq, 31)
    g = {k_: v_.cuda() for k_, v_ in tok.items()}
    pool = pool0.cuda().clone()
    o_init = torch.full((N, Tq, H, d), 7.0, device="cuda")
    o = kda.kda_recurrent_steps_pooled(g["q"], g["k"], g["v"], g["log_alpha"], g["beta"], pool, idx.cuda(),
                                       scale=0.9, o=o_init)
    torch.cuda.synchronize()
    o_ref, pool_ref = oracle.kda_steps_pooled(si.to_np32(tok["q"]), si.to_np32(tok["k"]), si.to_np32(tok["v"]),
                                              si.to_np32(tok["log_alpha"]), si.to_np32(tok["beta"]),
                                              pool0.numpy().astype(np.float64), idx.numpy(), scale=0.9)
    o_np, pool_np = o.cpu().numpy(), pool.cpu().numpy()
    act = [n for n in range(N) if idx[n] >= 0]
    eo = max(rel_err(o_np[n, :, h], o_ref[n, :, h]) for n in act for h in range(H))
    eS = max(rel_err(pool_np[int(idx[n]), h], pool_ref[int(idx[n]), h]) for n in act for h in range(H))
    print("pooled decode Tq=%d %s: err_o %.2e err_S %.2e" % (Tq, dtype, eo, eS))
    assert eo <= tol and eS <= tol
    assert (o_np[2] == 7.0).all()                                   # skipped sequence: o untouched
    unused = [p_ for p_ in range(P) if p_ not in idx.tolist()]
    assert torch.equal(pool.cpu()[unused], pool0[unused])            # states nobody named


def test_pooled_decode_without_indices_equals_the_plain_step_and_rejects_bad_sizes():
    import paper_2510_26692_amd as kda
    N, H, d = 3, 2, 128
    S0 = si.make_state(N, H, d, d, 0.02, 41)
    tok = si.make_decode_tokens(N, H, d, d, "bf16", -2.0, 41, 0)
    g = {k_: v_.cuda() for k_, v_ in tok.items()}
    S1, S2 = S0.cuda().clone(), S0.cuda().clone()
    o1 = kda.kda_recurrent_step(g["q"], g["k"], g["v"], g["log_alpha"], g["beta"], S1)
    o2 = kda.kda_recurrent_steps_pooled(g["q"][:, None].contiguous(), g["k"][:, None].contiguous(),
                                        g["v"][:, None].contiguous(), g["log_alpha"][:, None].contiguous(),
                                        g["beta"][:, None].contiguous(), S2)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2[:, 0]) and torch.equal(S1, S2)
    big = _stack_tokens(N, H, d, "bf16", 9, 41)
    gb = {k_: v_.cuda() for k_, v_ in big.items()}
    with pytest.raises(kda.KdaError) as ei:
        kda.kda_recurrent_steps_pooled(gb["q"], gb["k"], gb["v"], gb["log_alpha"], gb["beta"], S2)
    assert ei.value.status == 1


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
def test_rows_of_skipped_sequences_are_zero_in_a_fresh_output(out_dtype):
    import paper_2510_26692_amd as kda
    N, H, d, Tq = 4, 3, 128, 5
    g = {k_: v_.cuda() for k_, v_ in _stack_tokens(N, H, d, "bf16", Tq, 74).items()}
    idx = torch.tensor([-1, 3, -2, 0], dtype=torch.int32, device="cuda")
    args = [g[n] for n in ("q", "k", "v", "log_alpha", "beta")]
    torch.full((N, Tq, H, d), 7.0, device="cuda")                   # (what a fresh output is likely to lie on)
    o = kda.kda_recurrent_steps_pooled(*args, si.make_state(5, H, d, d, 0.02, 75).cuda(), idx, out_dtype=out_dtype)
    given = torch.full((N, Tq, H, d), 7.0, dtype=out_dtype, device="cuda")
    kda.kda_recurrent_steps_pooled(*args, si.make_state(5, H, d, d, 0.02, 75).cuda(), idx, o=given)
    assert (o[[0, 2]] == 0).all() and (given[[0, 2]] == 7).all() and torch.equal(o[[1, 3]], given[[1, 3]])


def _decode_call(form, dtype, d, out_dtype, given, indices, Tq, seed):
    """(function of the binding, arguments, keywords) of a decode call on fresh tensors, the states last among the arguments."""
    import paper_2510_26692_amd as kda
    N, H, P = 5, 3, 7
    g = torch.Generator().manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rn = lambda *s: torch.randn(*s, generator=g).to(dt).cuda()
    lead = (N, H) if form == "step" else (N, Tq, H)
    q, k, v = rn(*lead, d) * 0.1, rn(*lead, d) * 0.1, rn(*lead, d)
    la = rn(*lead) if form == "scalar" else rn(*lead, d)
    la, beta = -la.abs(), rn(*lead).abs().clamp(max=1.0)
    S = 0.1 * torch.randn(N if form == "step" else P, H, d, d, generator=g).cuda()
    kw = dict(scale=0.7, out_dtype=out_dtype)
    if given:
        kw["o"] = torch.full(lead + (d,), 3.0, dtype=out_dtype or torch.float32, device="cuda")
    if form != "step" and indices:
        kw["state_indices"] = torch.tensor([6, -1, 0, 3, -7], dtype=torch.int32, device="cuda")
    if form.startswith("fused"):
        kw.update(prologue=form != "fused_gate", out_gate=rn(*lead, d) if "gate" in form else None)
        if form == "fused_all_gate":
            kw.update(a_scale=torch.rand(H, generator=g).cuda(), dt_bias=torch.randn(H, d, generator=g).cuda(),
                      norm_weight=torch.randn(d, generator=g).cuda(), l2norm_eps=1e-5, rms_eps=1e-4)
    call = {"step": kda.kda_recurrent_step, "plain": kda.kda_recurrent_steps_pooled, "scalar": kda.kda_recurrent_steps_pooled_scalar_gate}
    return call.get(form, kda.kda_recurrent_steps_fused), [q, k, v, la, beta, S], kw


@pytest.mark.parametrize("form", ["step", "plain", "scalar", "fused", "fused_gate", "fused_all_gate"])
@pytest.mark.parametrize("dtype,d,out_dtype", [("bf16", 128, None), ("bf16", 128, torch.bfloat16), ("bf16", 64, None), ("f32", 128, torch.float32)])
@pytest.mark.parametrize("given,indices", [(False, True), (True, True), (False, False)])
def test_native_marshalling_is_the_general_one(form, dtype, d, out_dtype, given, indices, monkeypatch):
    """Every form of the decode calls, marshalled natively and by the general path: the same outputs and states bit for bit,
    rows of skipped sequences zero in a fresh o and untouched in a given one."""
    import paper_2510_26692_amd as kda
    assert kda.kda._native is not None
    results = []
    for general in (False, True):
        call, args, kw = _decode_call(form, dtype, d, out_dtype, given, indices, 3, 71)
        if general:
            monkeypatch.setattr(kda.kda, "_native", None)
        o = call(*args, **kw)
        assert not given or o is kw["o"]
        results.append((o, args[-1]))
    (o0, S0), (o1, S1) = results
    assert o0.dtype == o1.dtype and torch.equal(o0, o1) and torch.equal(S0, S1)
    if form != "step" and indices:
        assert (o0[[1, 4]].float() == (3.0 if given else 0.0)).all()


@pytest.mark.parametrize("form", ["step", "plain", "fused_all_gate"])
def test_irregular_decode_calls_are_still_refused(form):
    import paper_2510_26692_amd as kda

    def refused(error, at=None, to=None, **more):
        call, args, kw = _decode_call(form, "bf16", 128, None, False, False, 2, 72)
        if at is not None:
            args[at] = to(args[at])
        with pytest.raises(error):
            call(*args, **{**kw, **more})
    wide = lambda t: torch.cat([t, t], dim=-1)[..., :t.shape[-1]]
    for at in range(6):
        refused(ValueError, at, lambda t: t.cpu())
        if at != 4:
            refused(ValueError, at, wide)
        refused(ValueError, at, lambda t: t.to(torch.float16))
    refused(ValueError, 5, lambda t: t[:, :-1].contiguous())
    refused(ValueError, o=torch.empty(3, device="cuda"))
    refused(ValueError, out_dtype=torch.float16)
    refused(ValueError, o=torch.empty(3, device="cuda"), out_dtype=torch.bfloat16)
    if form != "step":
        refused(ValueError, state_indices=torch.zeros(5, dtype=torch.int64, device="cuda"))
        refused(ValueError, state_indices=torch.zeros(4, dtype=torch.int32, device="cuda"))
        refused(ValueError, 1, lambda t: t[:, :, :-1].contiguous())
        refused(TypeError, nonsense=1)
        with pytest.raises(kda.KdaError):                           # nine tokens: refused by the library, on either way
            call, args, kw = _decode_call(form, "bf16", 128, None, False, False, 9, 73)
            call(*args, **kw)


@pytest.mark.parametrize("at", [1, 2, 3, 4])
@pytest.mark.parametrize("shorter", [lambda t: t[:-1].contiguous(), lambda t: t[:, :-1].contiguous()])
def test_a_step_with_too_short_an_input_is_refused(at, shorter):
    """k, v, log alpha and beta hold a row for every row of q, or nothing is launched: the kernel reads them all."""
    call, args, kw = _decode_call("step", "bf16", 128, None, False, False, 1, 74)
    args[at] = shorter(args[at])
    with pytest.raises(ValueError):
        call(*args, **kw)


@pytest.mark.parametrize("form", ["step", "plain", "fused_all_gate"])
def test_irregular_decode_calls_that_are_valid_are_still_taken(form):
    """What the native marshalling hands back and the general path accepts: the same outputs and states as the plain call's."""
    import numpy as np

    import paper_2510_26692_amd as kda

    class Tagged(torch.Tensor):
        pass

    class Recording:
        """The native functions, and for each call whether it was taken."""
        def __init__(self, native):
            self.taken = []

            def recorded(f):
                def g(*a):
                    r = f(*a)
                    self.taken.append(r is not None)
                    return r
                return g
            self.step, self.steps = recorded(native.step), recorded(native.steps)

    def results(change_args=lambda a: a, **change_kw):
        call, args, kw = _decode_call(form, "bf16", 128, None, False, form != "step", 2, 76)
        args = change_args(args)
        with pytest.MonkeyPatch.context() as m:
            recording = Recording(kda.kda._native)
            m.setattr(kda.kda, "_native", recording)
            o = call(*args, **{**kw, **change_kw})
        return o, args[5], recording.taken
    o, S, taken = results()
    assert taken == [True]
    irregular = [
        (lambda a: [t.as_subclass(Tagged) for t in a], {}),                           # a tensor subclass
        (lambda a: [torch.nn.Parameter(t, requires_grad=False) for t in a], {}),
        (lambda a: a, dict(scale=np.float32(0.7))),                                   # a number of another kind
        (lambda a: a, dict(scale=torch.tensor(0.7))),
    ]
    if form == "step":
        irregular.append((lambda a: a[:4] + [a[4][..., None]] + a[5:], {}))           # beta [N,H,1]
    every = []
    for change_args, change_kw in irregular:
        o1, S1, taken = results(change_args, **change_kw)
        every += taken
        assert torch.equal(o, o1) and torch.equal(S, S1)
    assert every.count(False) >= len(irregular) - 1                                   # (a Parameter is a plain tensor)


def test_c_entry_points_for_decode_agree():
    """kda_recurrent_steps_pooled, _pooled_scalar_gate and _fused against kda_recurrent_steps, which the binding calls: the same bits,
    rows of skipped sequences untouched."""
    import ctypes

    import paper_2510_26692_amd as kda
    lib, binding = kda.load_library(), kda.kda

    def run(entry, form, flags=None):
        call, (q, k, v, la, beta, S), kw = _decode_call(form, "bf16", 128, None, True, True, 3, 77)
        N, T, H, D = q.shape
        dims = binding.KdaDims(batch=N, seqlen=T, heads=H, dk=D, dv=D, chunk=64, num_seqs=N, in_dtype=1, out_dtype=0, scale=0.7, max_seqlen=0)
        ref = ctypes.byref
        stages = []
        if form.startswith("fused"):
            pro = binding._make_prologue(H, D, kw["l2norm_eps"], kw["a_scale"], kw["dt_bias"])
            epi = binding._make_epilogue(v, kw["out_gate"], kw["norm_weight"], kw["rms_eps"])
            stages = [ref(pro), ref(epi)]
        elif flags is not None:
            stages = [None, None]
        ptrs = [t.data_ptr() for t in (q, k, v, la, beta, S, kw["state_indices"], kw["o"])]
        more = [] if flags is None else [flags]
        assert entry(ref(dims), *stages, *ptrs, *more, torch.cuda.current_stream().cuda_stream) == 0, kda.kda_last_error()
        torch.cuda.synchronize()
        return kw["o"], S
    for form, entry, flags in (("plain", lib.kda_recurrent_steps_pooled, 0), ("scalar", lib.kda_recurrent_steps_pooled_scalar_gate, 1),
                               ("fused_all_gate", lib.kda_recurrent_steps_fused, 0)):
        (o0, S0), (o1, S1) = run(entry, form), run(lib.kda_recurrent_steps, form, flags)
        assert torch.equal(o0, o1) and torch.equal(S0, S1), form
        assert (o0[[1, 4]] == 3.0).all() and not (o0[[0, 2, 3]] == 3.0).any(), form
