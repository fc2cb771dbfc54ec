"""The work that a user of this package has it do: prefill, decode and backward passes of Kimi Delta
Attention through the public entry points, over the range of sizes, types and options they serve.

A case is a dict of plain values:

    op      "prefill" (kda_chunk_fwd and its variants), "decode" (one step or a few tokens over a pool of
            states), "backward" (kda_chunk_bwd)
    form    "plain"  q, k, v, log alpha and beta as the layer has them ready
            "layer"  raw projections in, gated output out (input prologue and output gate fused)
            "scalar" one decay per token and head
    rows    batch rows, sequences of a packed batch, or sequences of a decode step
    tokens  tokens per row; the upper bound of a packed sequence's length; tokens per sequence of a decode call
    shortest, lengths_seed   packed batches only: lengths are uniform in [shortest, tokens] from that seed
    heads, dim, dtype ("bf16" or "f32": inputs), out ("bf16" or "f32": o, and d_o in a backward pass)
    state   prefill, backward: initial states come in;  decode: sequences name their states through an index
    buffers True: the program keeps its output buffers and passes them in

Values follow the recipe of the tests and the benchmark: q and k of unit norm, v normal,
beta = sigmoid(normal), log alpha = -softplus(normal + mean) with mean -2 (slow decay).
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

import paper_2510_26692_amd as kda

DEV = "cuda"
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
DECAY_MEAN = -2.0
POOL_SPARE = 16                # states of a pool beyond the ones a call addresses


def _case(name, op, rows, tokens, heads, form="plain", shortest=0, lengths_seed=0, dim=128, dtype="bf16", out="f32",
          state=False, buffers=False):
    return dict(name=name, op=op, form=form, rows=rows, tokens=tokens, shortest=shortest, lengths_seed=lengths_seed,
                heads=heads, dim=dim, dtype=dtype, out=out, state=state, buffers=buffers)


def listed():
    return [
        # one user's chat turn being decoded: one sequence, one token, 32 heads (latency counts, 4 MB of states)
        _case("decode_one_sequence", "decode", 1, 1, 32),
        # a serving batch: 256 sequences, one token each, 512 MiB of states updated in place
        _case("decode_batch", "decode", 256, 1, 32, buffers=True),
        # speculative decoding: four draft tokens per sequence, states addressed in a pool, the layer's
        # prologue and gate fused, bf16 output for the projection that follows
        _case("decode_draft_layer", "decode", 48, 4, 32, form="layer", out="bf16", state=True),
        # a short prompt of ragged length: the first answer waits for it
        _case("prefill_short_prompt", "prefill", 1, 333, 32),
        # four 4096-token rows with initial states: the ordinary prefill (and a training step's forward pass)
        _case("prefill_rows", "prefill", 4, 4096, 16, state=True),
        # continuous batching: eight prompts of mixed lengths packed into one stream
        _case("prefill_packed", "prefill", 8, 8192, 32, shortest=512, lengths_seed=1),
        # the whole layer on a packed batch: raw projections in, gated bf16 output out
        _case("prefill_layer", "prefill", 6, 4096, 32, form="layer", shortest=256, lengths_seed=5, out="bf16"),
        # a long document: 2^17 tokens, one sequence, buffers kept by the program
        _case("prefill_long", "prefill", 1, 131072, 32, buffers=True),
        # fp32 inputs with small heads: the form in which the method is checked and small models are trained
        _case("prefill_f32", "prefill", 2, 1999, 8, dim=64, dtype="f32"),
        # the backward pass of the ordinary training step, gradients of the initial states included
        _case("backward_rows", "backward", 4, 4096, 16, out="bf16", state=True),
        # training on packed documents of mixed lengths, fp32 gradient of the output
        _case("backward_packed", "backward", 5, 3000, 16, shortest=100, lengths_seed=2),
        # one long sample per step: few (sequence, head) pairs, many chunks
        _case("backward_long", "backward", 1, 8192, 16, out="bf16"),
    ]


def _between(rng, low, high):
    """A whole number in [low, high], evenly spread over its logarithm, odd ones as likely as even ones."""
    return max(low, min(high, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def draw(rng):
    op = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "backward", "backward"])
    heads = rng.choice([2, 4, 8, 16, 32])
    dtype, dim = rng.choice([("bf16", 128), ("bf16", 128), ("bf16", 128), ("f32", 128), ("f32", 64)])
    out = rng.choice(["f32", "bf16"]) if (dtype, dim) == ("bf16", 128) else "f32"
    common = dict(dim=dim, dtype=dtype, out=out, state=rng.random() < 0.5, buffers=rng.random() < 0.5)
    if op == "decode":
        return _unnamed(_case("", op, _between(rng, 1, 256), rng.choice([1, 1, 1, 2, 3, 4, 8]), heads,
                              form=rng.choice(["plain", "plain", "layer", "scalar"]), **common))
    form = "plain"
    if op == "prefill" and (dtype, dim) == ("bf16", 128):          # the fused stages and the scalar decay are built for these
        form = rng.choice(["plain", "plain", "layer", "scalar"])
    rows = _between(rng, 1, 12)
    # tokens x heads of the whole call, at most those of the largest listed case of its kind
    most = 131072 * 32 if op == "prefill" and dtype == "bf16" else 4 * 4096 * 16
    tokens = _between(rng, 1, max(1, most // (rows * heads)))
    packed = rows > 1 and rng.random() < 0.5
    return _unnamed(_case("", op, rows, tokens, heads, form=form, shortest=rng.randint(1, tokens) if packed else 0,
                          lengths_seed=rng.randint(0, 999), **common))


def _unnamed(case):
    del case["name"]
    return case


def _lengths(case):
    """Tokens of each sequence."""
    if not case["shortest"]:
        return [case["tokens"]] * case["rows"]
    rng = np.random.default_rng(case["lengths_seed"])
    return [int(n) for n in rng.integers(case["shortest"], case["tokens"] + 1, case["rows"])]


def _tokens(gen, shape, dim, dtype, form):
    """q, k, v, decay, beta of `shape` = (rows, tokens, heads), made slice by slice so that no large fp32 copy is held."""
    rows, tokens, heads = shape
    x = {n: torch.empty(*shape, dim, dtype=dtype, device=DEV) for n in ("q", "k", "v")}
    x["decay"] = torch.empty(*shape, *(() if form == "scalar" else (dim,)), dtype=dtype, device=DEV)
    x["beta"] = torch.empty(*shape, dtype=dtype, device=DEV)
    step = max(1, (1 << 21) // (rows * heads))
    for t in range(0, tokens, step):
        part = slice(t, min(tokens, t + step))
        n = part.stop - part.start

        def normal(*more):
            return torch.randn(rows, n, heads, *more, generator=gen, device=DEV)
        gate = normal(*(() if form == "scalar" else (dim,))) + DECAY_MEAN
        if form == "layer":
            x["q"][:, part], x["k"][:, part] = 2.0 * normal(dim), 2.0 * normal(dim)
            x["decay"][:, part], x["beta"][:, part] = gate, normal()
        else:
            x["q"][:, part], x["k"][:, part] = F.normalize(normal(dim), dim=-1), F.normalize(normal(dim), dim=-1)
            x["decay"][:, part], x["beta"][:, part] = -F.softplus(gate), torch.sigmoid(normal())
        x["v"][:, part] = normal(dim)
    return x


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    op, form, heads, dim = case["op"], case["form"], case["heads"], case["dim"]
    dtype, out = TYPES[case["dtype"]], TYPES[case["out"]]
    rows, lengths = case["rows"], _lengths(case)
    packed = case["shortest"] > 0
    shape = (1, sum(lengths), heads) if packed else (rows, case["tokens"], heads)
    single = op == "decode" and case["tokens"] == 1 and form == "plain" and not case["state"]
    x = _tokens(gen, shape, dim, dtype, form)
    if single:
        x = {n: t[:, 0].contiguous() for n, t in x.items()}
    s = dict(case=case, x=x, single=single)
    kw = s["kw"] = {}
    if form == "layer":
        kw["a_scale"] = 0.5 + 1.5 * torch.rand(heads, generator=gen, device=DEV)
        kw["dt_bias"] = 0.5 * torch.randn(heads, dim, generator=gen, device=DEV)
        kw["out_gate"] = torch.randn(*shape, dim, generator=gen, device=DEV).to(dtype)
        kw["norm_weight"] = 1.0 + 0.1 * torch.randn(dim, generator=gen, device=DEV)
    if op == "decode":
        pool = rows + POOL_SPARE if case["state"] else rows
        s["states"] = 0.02 * torch.randn(pool, heads, dim, dim, generator=gen, device=DEV)
        if case["state"]:
            kw["state_indices"] = torch.randperm(pool, generator=gen, device=DEV)[:rows].to(torch.int32)
        kw["out_dtype"] = out
        if case["buffers"]:
            kw["o"] = torch.empty_like(x["v"], dtype=out)
        return s
    cu = None
    if packed:
        cu = torch.tensor([0] + lengths, device=DEV).cumsum(0).to(torch.int32)
        kw["cu_seqlens"], kw["max_seqlen"] = cu, max(lengths)
    if case["state"]:
        kw["h0"] = 0.02 * torch.randn(rows, heads, dim, dim, generator=gen, device=DEV)
    dims = kda.kda.make_chunk_dims(x["q"], x["v"], cu, 1.0, kw.get("max_seqlen", 0), out)
    if op == "prefill":
        kw["out_dtype"] = out
        need = kda.kda.kda_chunk_fwd_workspace_size(dims, output_gate=form == "layer")
        if case["buffers"]:
            kw["o"] = torch.empty_like(x["v"], dtype=out)
            kw["hT"] = torch.empty(rows, heads, dim, dim, device=DEV)
    else:
        s["d_o"] = torch.randn(*x["v"].shape, generator=gen, device=DEV).to(out)
        kw["want_dh0"] = case["state"]
        need = kda.kda_chunk_bwd_workspace_size(dims)
        if case["state"]:
            kw["dhT"] = 0.1 * torch.randn(rows, heads, dim, dim, generator=gen, device=DEV)
        if case["buffers"]:
            like = dict(dq="q", dk="k", dv="v", dlog_alpha="decay", dbeta="beta")
            kw["out"] = {g: torch.empty_like(x[n], dtype=torch.float32) for g, n in like.items()}
            kw["out"]["dh0"] = torch.empty_like(kw["h0"]) if case["state"] else None
    if need:
        kw["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    return s


def run(s):
    x, kw, op, form = s["x"], s["kw"], s["case"]["op"], s["case"]["form"]
    args = (x["q"], x["k"], x["v"], x["decay"], x["beta"])
    if op == "backward":
        return kda.kda_chunk_bwd(*args, s["d_o"], **kw)
    if op == "prefill":
        call = {"plain": kda.kda_chunk_fwd, "layer": kda.kda_chunk_fwd_fused, "scalar": kda.kda_chunk_fwd_scalar_gate}[form]
        return call(*args, **kw)
    if s["single"]:
        return kda.kda_recurrent_step(*args, s["states"], **kw), s["states"]
    call = {"plain": kda.kda_recurrent_steps_pooled, "layer": kda.kda_recurrent_steps_fused,
            "scalar": kda.kda_recurrent_steps_pooled_scalar_gate}[form]
    return call(*args, s["states"], **kw), s["states"]


def work(case):
    """Bytes: every input read once, every output written once, the states of the sequences among them.
    Operations per token and head: prefill 6 d^2 + 3 C d + C^2 with C = 64 (the chunkwise form's count);
    backward, per chunk, eight C d^2 products, eight half-filled C^2 d ones and three C^3 ones; decode, four
    operations per element of the state and reduction."""
    op, dim, heads = case["op"], case["dim"], case["heads"]
    size = {"bf16": 2, "f32": 4}
    si, so = size[case["dtype"]], size[case["out"]]
    units = sum(_lengths(case)) * heads                     # (token, head) pairs
    state = case["rows"] * heads * dim * dim * 4
    decay = 1 if case["form"] == "scalar" else dim
    inputs = (3 * dim + decay + 1 + (dim if case["form"] == "layer" else 0)) * si
    c = 64
    if op == "decode":
        return {"bytes": units * (inputs + dim * so) + 2 * state, "flops": units * 7 * dim * dim}
    if op == "prefill":
        return {"bytes": units * (inputs + dim * so) + state * (2 if case["state"] else 1),
                "flops": units * (6 * dim * dim + 3 * c * dim + c * c)}
    return {"bytes": units * (inputs + dim * so + (4 * dim + 1) * 4) + state * (3 if case["state"] else 0),
            "flops": units * (16 * dim * dim + 8 * c * dim + 6 * c * c)}


def tolerance(case):
    """2-norm errors, about four times what these paths show against the fp64 recurrence: fp16 operands of the
    bf16 prefill 4.5e-4; one rounding of o to bf16 1.7e-3; fp32 throughout 3e-7 (forward), 5.6e-7 (backward),
    1.1e-7 (decode, to which the fused stages add a few roundings)."""
    if case["op"] == "backward":
        return {"rel": 3e-6}
    if case["out"] == "bf16":
        return {"rel": 7e-3}
    if case["op"] == "decode":
        return {"rel": 2e-6 if case["form"] == "layer" else 5e-7}
    return {"rel": 2e-3 if case["dtype"] == "bf16" else 2e-6}
