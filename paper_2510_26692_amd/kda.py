"""ctypes binding for libkda.so (see include/kda.h for the contract).

Argument marshalling only.  Tensors are torch tensors used as device-memory
handles (``data_ptr()``), the stream is torch's current HIP stream.
"""
import ctypes
import os
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# KDA_LIBRARY_PATH lets a developer point the binding at another build of the same library.
_LIB_PATH = os.environ.get("KDA_LIBRARY_PATH") or os.path.join(_HERE, "libkda.so")
_lib = None
_native = None                            # decode calls marshalled natively (csrc/kda_host.cpp); None: not built, everything goes the general way

KDA_F32, KDA_BF16 = 0, 1
_DTYPE_CODE = {torch.float32: KDA_F32, torch.bfloat16: KDA_BF16}
_SCALAR_GATE, _ZERO_SKIPPED = 1, 2        # flags of kda_recurrent_steps
_STEPS_OPTIONS = {"scale", "o", "out_dtype"}


class KdaError(RuntimeError):
    """A libkda entry point returned a non-zero status."""

    def __init__(self, status, detail):
        super().__init__("libkda status %d (%s): %s" % (status, kda_status_string(status), detail))
        self.status = status
        self.detail = detail


class KdaDims(ctypes.Structure):
    """Mirror of ``kda_dims``."""
    _fields_ = [("batch", ctypes.c_int32), ("seqlen", ctypes.c_int64), ("heads", ctypes.c_int32),
                ("dk", ctypes.c_int32), ("dv", ctypes.c_int32), ("chunk", ctypes.c_int32),
                ("num_seqs", ctypes.c_int32), ("in_dtype", ctypes.c_int), ("out_dtype", ctypes.c_int),
                ("scale", ctypes.c_float), ("max_seqlen", ctypes.c_int64)]


class KdaPrologue(ctypes.Structure):
    """Mirror of ``kda_prologue``."""
    _fields_ = [("l2norm_eps", ctypes.c_float), ("a_scale", ctypes.c_void_p), ("dt_bias", ctypes.c_void_p)]


class KdaEpilogue(ctypes.Structure):
    """Mirror of ``kda_epilogue``."""
    _fields_ = [("rms_eps", ctypes.c_float), ("gate", ctypes.c_void_p), ("norm_weight", ctypes.c_void_p)]


def library_path():
    return _LIB_PATH


def load_library():
    """Load libkda.so; raises if it has not been built (no fallback exists)."""
    global _lib, _native
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise RuntimeError("libkda.so is not built: run `python -m paper_2510_26692_amd.build` "
                           "(there is no CPU or PyTorch fallback for the KDA kernels)")
    lib = ctypes.CDLL(_LIB_PATH)
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    dp = ctypes.POINTER(KdaDims)
    lib.kda_version.restype = ctypes.c_char_p
    lib.kda_last_error.restype = ctypes.c_char_p
    lib.kda_status_string.restype = ctypes.c_char_p
    lib.kda_status_string.argtypes = [ctypes.c_int]
    lib.kda_chunk_fwd_workspace_size.restype = sz
    lib.kda_chunk_fwd_workspace_size.argtypes = [dp]
    lib.kda_chunk_fwd_min_workspace_size.restype = sz
    lib.kda_chunk_fwd_min_workspace_size.argtypes = [dp]
    lib.kda_chunk_fwd.restype = ctypes.c_int
    lib.kda_chunk_fwd.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.kda_chunk_fwd_check.restype = ctypes.c_int
    lib.kda_chunk_fwd_check.argtypes = [dp, vp, sz, vp]
    lib.kda_chunk_bwd_workspace_size.restype = sz
    lib.kda_chunk_bwd_workspace_size.argtypes = [dp]
    lib.kda_chunk_bwd.restype = ctypes.c_int
    lib.kda_chunk_bwd.argtypes = [dp] + [vp] * 15 + [vp, sz, vp]
    lib.kda_clear_unowned_rows.restype = ctypes.c_int
    lib.kda_clear_unowned_rows.argtypes = [vp, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.POINTER(vp),
                                           ctypes.POINTER(sz), vp]
    lib.kda_static_scratch_size.restype = ctypes.c_size_t
    lib.kda_static_scratch_size.argtypes = []
    lib.kda_chunk_fwd_static_scratch.restype = ctypes.c_int
    lib.kda_chunk_fwd_static_scratch.argtypes = [ctypes.POINTER(KdaDims)] + [ctypes.c_void_p] * 10
    lib.kda_debug_set_producers.restype = None
    lib.kda_debug_set_producers.argtypes = [ctypes.c_int]
    lib.kda_debug_set_wait_limit.restype = None
    lib.kda_debug_set_wait_limit.argtypes = [ctypes.c_ulonglong]
    lib.kda_debug_chunk_fwd_plan.restype = ctypes.c_int
    lib.kda_debug_chunk_fwd_plan.argtypes = [ctypes.POINTER(KdaDims), ctypes.c_size_t, ctypes.c_int,
                                             ctypes.POINTER(ctypes.c_int64)]
    lib.kda_debug_prefill_grid.restype = ctypes.c_int
    lib.kda_debug_prefill_grid.argtypes = [ctypes.POINTER(KdaDims), ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int64)]
    lib.kda_debug_chunk_fwd_status.restype = ctypes.c_int
    lib.kda_debug_chunk_fwd_status.argtypes = [ctypes.POINTER(KdaDims), vp, sz, vp, ctypes.POINTER(ctypes.c_uint)]
    lib.kda_debug_stream_probe.restype = ctypes.c_int
    lib.kda_debug_stream_probe.argtypes = [ctypes.c_int, vp, sz, vp]
    lib.kda_debug_prefill_traffic_probe.restype = ctypes.c_int
    lib.kda_debug_prefill_traffic_probe.argtypes = [vp, sz, ctypes.POINTER(ctypes.c_size_t), vp]
    lib.kda_debug_mfma_probe.restype = ctypes.c_int
    lib.kda_debug_mfma_probe.argtypes = [vp, ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_double), vp]
    lib.kda_debug_set_time_split.restype = None
    lib.kda_debug_set_time_split.argtypes = [ctypes.c_int]
    lib.kda_recurrent_step.restype = ctypes.c_int
    lib.kda_recurrent_step.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.kda_recurrent_steps_pooled.restype = ctypes.c_int
    lib.kda_recurrent_steps_pooled.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    pp, ep = ctypes.POINTER(KdaPrologue), ctypes.POINTER(KdaEpilogue)
    lib.kda_chunk_fwd_fused.restype = ctypes.c_int
    lib.kda_chunk_fwd_fused.argtypes = [dp, pp, ep, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.kda_chunk_fwd_fused_workspace_size.restype = sz
    lib.kda_chunk_fwd_fused_workspace_size.argtypes = [dp, ep]
    lib.kda_chunk_fwd_fused_min_workspace_size.restype = sz
    lib.kda_chunk_fwd_fused_min_workspace_size.argtypes = [dp, ep]
    lib.kda_chunk_fwd_scalar_gate.restype = ctypes.c_int
    lib.kda_chunk_fwd_scalar_gate.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.kda_recurrent_steps_pooled_scalar_gate.restype = ctypes.c_int
    lib.kda_recurrent_steps_pooled_scalar_gate.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.kda_recurrent_steps_fused.restype = ctypes.c_int
    lib.kda_recurrent_steps_fused.argtypes = [dp, pp, ep, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.kda_recurrent_steps.restype = ctypes.c_int
    lib.kda_recurrent_steps.argtypes = [dp, pp, ep, vp, vp, vp, vp, vp, vp, vp, vp, ctypes.c_uint32, vp]
    try:
        from . import _kda_host
        _kda_host.bind(*[ctypes.cast(f, vp).value for f in (lib.kda_recurrent_step, lib.kda_recurrent_steps)], _raw_stream)
        _native = _kda_host
    except ImportError as e:                # (missing, or built for another torch or interpreter: right all the same, but no secret)
        warnings.warn("decode calls are marshalled in Python, at about twice the host time: %s (build it with "
                      "python -m paper_2510_26692_amd.build)" % e, RuntimeWarning, stacklevel=2)
    _lib = lib
    return lib


def kda_version():
    return load_library().kda_version().decode()


def kda_last_error():
    return load_library().kda_last_error().decode()


def kda_debug_set_producers(enabled):
    """Fault injection (kda_debug.h): 0 makes the per-chunk workgroups of later prefill calls do nothing."""
    load_library().kda_debug_set_producers(int(bool(enabled)))


def kda_debug_set_wait_limit(ticks):
    """Ticks of the 100 MHz device clock a sequential workgroup waits for one slot (default 200 000 000)."""
    load_library().kda_debug_set_wait_limit(int(ticks))


def kda_debug_chunk_fwd_plan(dims, workspace_bytes, output_gate=False):
    """(chunk indices per time segment, time segments, ranges of the time-split scan, chunks in the first
    range, chunks in each other range) for a kda_chunk_fwd call with this workspace size."""
    out = (ctypes.c_int64 * 5)()
    st = load_library().kda_debug_chunk_fwd_plan(ctypes.byref(dims), ctypes.c_size_t(int(workspace_bytes)),
                                                 int(bool(output_gate)), out)
    if st != 0:
        raise KdaError(st, kda_last_error())
    return tuple(int(x) for x in out)


def kda_debug_prefill_grid(dims, packed, compute_units=256):
    """(pairs per batch, chunks a per-chunk workgroup works through, workgroups) of a bf16 prefill's first launch (kda_debug.h)."""
    out = (ctypes.c_int64 * 3)()
    st = load_library().kda_debug_prefill_grid(ctypes.byref(dims), int(bool(packed)), int(compute_units), out)
    if st != 0:
        raise KdaError(st, kda_last_error())
    return tuple(int(x) for x in out)


def kda_debug_chunk_fwd_status(dims, workspace):
    """The raw status word the bf16 prefill call that used `workspace` with `dims` left behind (waits for the
    current stream): bits 1, 2, 4 failures, 256 / 512 the way the time-split scan took (kda_debug.h)."""
    word = ctypes.c_uint(0)
    st = load_library().kda_debug_chunk_fwd_status(ctypes.byref(dims), _ptr(workspace),
                                                   ctypes.c_size_t(workspace.numel() * workspace.element_size()),
                                                   _stream_ptr(workspace.device), ctypes.byref(word))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return int(word.value)


def kda_debug_stream_probe(mode, buffer):
    """One streaming pass over the fp32 device tensor `buffer` (a multiple of 65536 bytes, overwritten) on the
    current stream: mode 0 reads, 1 writes, 2 reads, modifies and writes in place.  Returns the bytes of the buffer."""
    _check_dev(buffer)
    assert buffer.dtype == torch.float32 and buffer.is_contiguous()
    nbytes = buffer.numel() * 4
    st = load_library().kda_debug_stream_probe(int(mode), _ptr(buffer), ctypes.c_size_t(nbytes), _stream_ptr(buffer.device))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return nbytes


def kda_debug_prefill_traffic_probe(buffer):
    """One launch of the prefill traffic probe over the uint8 device tensor `buffer` (a multiple of 172032 bytes,
    overwritten) on the current stream; returns (items, bytes moved)."""
    _check_dev(buffer)
    nbytes = buffer.numel() * buffer.element_size()
    moved = ctypes.c_size_t(0)
    st = load_library().kda_debug_prefill_traffic_probe(_ptr(buffer), ctypes.c_size_t(nbytes), ctypes.byref(moved),
                                                        _stream_ptr(buffer.device))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return nbytes // 172032, int(moved.value)


def kda_debug_mfma_probe(sink, workgroups, iters):
    """One launch of the matrix-core probe on the current stream; returns its floating-point operations."""
    _check_dev(sink)
    flops = ctypes.c_double(0.0)
    st = load_library().kda_debug_mfma_probe(_ptr(sink), int(workgroups), int(iters), ctypes.byref(flops), _stream_ptr(sink.device))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return flops.value


def kda_debug_set_time_split(mode):
    """0 = off, 1 = on (the library estimates whether and how far to split), 2..32 = that many ranges
    (at most) whatever the estimate says."""
    load_library().kda_debug_set_time_split(int(mode))


def kda_status_string(status):
    return load_library().kda_status_string(int(status)).decode()


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _check_dev(*tensors):
    dev = None
    for t in tensors:
        if t is None:
            continue
        if not t.is_cuda:
            raise ValueError("libkda takes device tensors only")
        if not t.is_contiguous():
            raise ValueError("libkda takes contiguous tensors only")
        dev = dev or t.device
        if t.device != dev:
            raise ValueError("all tensors must live on one device")
    return dev


def _raw_stream(index):
    return torch.cuda.current_stream(index).cuda_stream


# (the same number without a Stream object around it: 0.1 instead of 2 us)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", _raw_stream)


def _stream_ptr(dev):
    return ctypes.c_void_p(_raw_stream(dev.index))


def _result(done):
    """What the native way returned: the tensor, or the status of a call the library refused."""
    if type(done) is int:
        raise KdaError(done, kda_last_error())
    return done


def _mostly_unowned(cu_seqlens, tokens, max_seqlen):
    """Whether max_seqlen tells that most rows of a packed call belong to no sequence.  Fresh outputs are then filled with zeros
    whole, at the rate of a plain fill (200000 rows x 32 heads, 2048 of them owned: 0.48 against 0.50 ms)."""
    return 0 < 2 * max_seqlen * (cu_seqlens.numel() - 1) < tokens


def _clear_unowned(cu_seqlens, tensors):
    """Zeros in the rows [0, cu_seqlens[0]) and [cu_seqlens[-1], T) of freshly allocated [1,T,...] tensors (the calls write
    all other rows)."""
    tensors = [t for t in tensors if t.numel()]
    if not tensors:
        return
    n, tokens = len(tensors), tensors[0].shape[1]
    ptrs = (ctypes.c_void_p * n)(*[t.data_ptr() for t in tensors])
    rows = (ctypes.c_size_t * n)(*[t.numel() // tokens * t.element_size() for t in tensors])
    st = load_library().kda_clear_unowned_rows(_ptr(cu_seqlens), cu_seqlens.numel() - 1, tokens, n, ptrs, rows,
                                               _stream_ptr(cu_seqlens.device))
    if st != 0:
        raise KdaError(st, kda_last_error())


def _out_dtype(o, out_dtype):
    """torch dtype of o: that of a tensor passed in, else `out_dtype`, else fp32."""
    dt = o.dtype if o is not None else (out_dtype or torch.float32)
    if out_dtype is not None and dt != out_dtype:
        raise ValueError("o has dtype %s but out_dtype is %s" % (dt, out_dtype))
    if dt not in _DTYPE_CODE:
        raise ValueError("unsupported output dtype %s" % dt)
    return dt


def make_chunk_dims(q, v, cu_seqlens=None, scale=1.0, max_seqlen=0, out_dtype=torch.float32):
    B, T, H, dk = q.shape
    dv = v.shape[-1]
    N = B if cu_seqlens is None else cu_seqlens.numel() - 1
    return KdaDims(batch=B, seqlen=T, heads=H, dk=dk, dv=dv, chunk=64, num_seqs=N,
                   in_dtype=_DTYPE_CODE[q.dtype], out_dtype=_DTYPE_CODE[out_dtype], scale=float(scale),
                   max_seqlen=int(max_seqlen))


def kda_chunk_fwd_workspace_size(dims, output_gate=False):
    """Bytes for a single-segment call; output_gate=True: for kda_chunk_fwd_fused with an output gate."""
    if not output_gate:
        return int(load_library().kda_chunk_fwd_workspace_size(ctypes.byref(dims)))
    return int(load_library().kda_chunk_fwd_fused_workspace_size(ctypes.byref(dims), ctypes.byref(KdaEpilogue())))


def kda_chunk_fwd_min_workspace_size(dims, output_gate=False):
    if not output_gate:
        return int(load_library().kda_chunk_fwd_min_workspace_size(ctypes.byref(dims)))
    return int(load_library().kda_chunk_fwd_fused_min_workspace_size(ctypes.byref(dims), ctypes.byref(KdaEpilogue())))


def kda_chunk_fwd_check(dims, workspace):
    """Waits for the current stream and raises KdaError if the kda_chunk_fwd call that used
    `workspace` with `dims` reported a failed wait (see kda_chunk_fwd_check in kda.h)."""
    if workspace is None:
        return
    st = load_library().kda_chunk_fwd_check(ctypes.byref(dims), _ptr(workspace),
                                            ctypes.c_size_t(workspace.numel() * workspace.element_size()),
                                            _stream_ptr(workspace.device))
    if st != 0:
        raise KdaError(st, kda_last_error())


def _make_prologue(H, dk, l2norm_eps, a_scale, dt_bias):
    for t, shape, name in ((a_scale, (H,), "a_scale"), (dt_bias, (H, dk), "dt_bias")):
        if t is not None and (t.dtype != torch.float32 or tuple(t.shape) != shape or not t.is_cuda
                              or not t.is_contiguous()):
            raise ValueError("%s must be a contiguous fp32 device tensor of shape %r" % (name, shape))
    return KdaPrologue(l2norm_eps=float(l2norm_eps),
                       a_scale=None if a_scale is None else a_scale.data_ptr(),
                       dt_bias=None if dt_bias is None else dt_bias.data_ptr())


def _make_epilogue(v, out_gate, norm_weight, rms_eps):
    if out_gate is None:
        return None
    if out_gate.shape != v.shape or out_gate.dtype != v.dtype or not out_gate.is_cuda or not out_gate.is_contiguous():
        raise ValueError("out_gate must be a contiguous device tensor with the shape and dtype of v")
    if norm_weight is not None and (norm_weight.dtype != torch.float32 or tuple(norm_weight.shape) != (v.shape[-1],)
                                    or not norm_weight.is_cuda or not norm_weight.is_contiguous()):
        raise ValueError("norm_weight must be a contiguous fp32 device tensor of shape (dv,)")
    return KdaEpilogue(rms_eps=float(rms_eps), gate=out_gate.data_ptr(),
                       norm_weight=None if norm_weight is None else norm_weight.data_ptr())


def kda_chunk_fwd_fused(q, k, v, gate, beta, prologue=True, l2norm_eps=1e-6, a_scale=None, dt_bias=None,
                        out_gate=None, norm_weight=None, rms_eps=1e-6, **kw):
    """kda_chunk_fwd with the fused stages of kda.h.  prologue=True: q, k, beta and gate are raw
    projections (L2Norm, Sigmoid and log_alpha = -a_scale[h] softplus(gate + dt_bias[h]) run inside
    the kernel; a_scale fp32 [H], dt_bias fp32 [H,dk] on the device, or None); prologue=False: they
    are taken as kda_chunk_fwd takes them (gate = log_alpha).  out_gate (shape and dtype of v) turns
    on the output gate o <- Sigmoid(out_gate) * RMSNorm(o) * norm_weight (fp32 [dv] or None).
    Other arguments and the result as for kda_chunk_fwd."""
    pro = _make_prologue(q.shape[2], q.shape[3], l2norm_eps, a_scale, dt_bias) if prologue else None
    return kda_chunk_fwd(q, k, v, gate, beta, _fused=(pro, _make_epilogue(v, out_gate, norm_weight, rms_eps)), **kw)


def kda_chunk_fwd(q, k, v, log_alpha, beta, h0=None, cu_seqlens=None, scale=1.0, o=None,
                  hT=None, want_hT=True, workspace=None, max_seqlen=0, check=False, out_dtype=None,
                  _fused=None, _scalar_gate=False):
    """Chunkwise prefill.  q,k,log_alpha [B,T,H,dk]; v [B,T,H,dv]; beta [B,T,H];
    h0 [N,H,dk,dv] fp32 or None; cu_seqlens int32 [N+1] on device or None.
    Returns (o [B,T,H,dv], hT fp32 [N,H,dk,dv] or None); o is fp32 unless out_dtype (or the `o`
    passed in) is torch.bfloat16, which bf16 inputs allow.  `o`, `hT` and
    `workspace` (a uint8 device tensor) may be passed in to avoid allocation.
    check=True synchronises and runs kda_chunk_fwd_check before returning."""
    lib = load_library()
    dev = _check_dev(q, k, v, log_alpha, beta, h0, cu_seqlens, o, hT, workspace)
    if not (q.dtype == k.dtype == v.dtype == log_alpha.dtype == beta.dtype):
        raise ValueError("q, k, v, log_alpha, beta must share one dtype")
    if q.dtype not in _DTYPE_CODE:
        raise ValueError("unsupported input dtype %s" % q.dtype)
    B, T, H, dk = q.shape
    dv = v.shape[-1]
    if k.shape != q.shape or log_alpha.shape != ((B, T, H) if _scalar_gate else q.shape) \
            or v.shape != (B, T, H, dv) or beta.shape != (B, T, H):
        raise ValueError("inconsistent input shapes")
    odt = _out_dtype(o, out_dtype)
    dims = make_chunk_dims(q, v, cu_seqlens, scale, max_seqlen, odt)
    N = dims.num_seqs
    if o is not None and o.shape != (B, T, H, dv):
        raise ValueError("o must have shape [B,T,H,dv]")
    if h0 is not None and (h0.dtype != torch.float32 or h0.shape != (N, H, dk, dv)):
        raise ValueError("h0 must be fp32 [N,H,dk,dv]")
    if cu_seqlens is not None and cu_seqlens.dtype != torch.int32:
        raise ValueError("cu_seqlens must be int32")
    clear = False
    if o is None:
        # (up to 8 MiB the fill costs less than the clearing call: 12 tokens x 2 heads, bf16, 24.5 against 26.3 us in all)
        packed = cu_seqlens is not None
        filled = packed and (T * H * dv * odt.itemsize <= 8 << 20 or _mostly_unowned(cu_seqlens, T, max_seqlen))
        o = (torch.zeros if filled else torch.empty)(B, T, H, dv, dtype=odt, device=dev)
        clear = packed and not filled
    if hT is not None and hT.numel() * hT.element_size() < N * H * dk * dv * 4:
        raise ValueError("hT must be fp32 [N,H,dk,dv]")
    if hT is None and want_hT:
        hT = torch.empty(N, H, dk, dv, dtype=torch.float32, device=dev)
    if workspace is None:
        need = kda_chunk_fwd_workspace_size(dims, output_gate=_fused is not None and _fused[1] is not None)
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=dev) if need else None
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    tail = (_ptr(q), _ptr(k), _ptr(v), _ptr(log_alpha), _ptr(beta), _ptr(h0), _ptr(cu_seqlens), _ptr(o),
            _ptr(hT), _ptr(workspace), ctypes.c_size_t(ws_bytes), _stream_ptr(dev))
    if _scalar_gate:
        st = lib.kda_chunk_fwd_scalar_gate(ctypes.byref(dims), *tail)
    elif _fused is None:
        st = lib.kda_chunk_fwd(ctypes.byref(dims), *tail)
    else:
        st = lib.kda_chunk_fwd_fused(ctypes.byref(dims), *[None if f is None else ctypes.byref(f) for f in _fused],
                                     *tail)
    if st != 0:
        raise KdaError(st, kda_last_error())
    if clear:                               # (behind the call, whose launch need not wait for this one's)
        _clear_unowned(cu_seqlens, [o])
    if check:
        kda_chunk_fwd_check(dims, workspace)
    return o, hT


def kda_static_scratch_size():
    return int(load_library().kda_static_scratch_size())


def kda_chunk_fwd_static_scratch(q, k, v, log_alpha, beta, o, hT=None, h0=None, cu_seqlens=None, scale=1.0, max_seqlen=0):
    """kda_chunk_fwd on the library's static scratch array: nothing is allocated, so `o` (and `hT`, if the
    final states are wanted) must be passed in.  Returns (o, hT)."""
    lib = load_library()
    dev = _check_dev(q, k, v, log_alpha, beta, h0, cu_seqlens, o, hT)
    B, T, H, dk = q.shape
    dv = v.shape[-1]
    if not (q.dtype == k.dtype == v.dtype == log_alpha.dtype == beta.dtype) or q.dtype not in _DTYPE_CODE:
        raise ValueError("q, k, v, log_alpha, beta must share a supported dtype")
    if k.shape != q.shape or log_alpha.shape != q.shape or v.shape != (B, T, H, dv) or beta.shape != (B, T, H) \
            or o.shape != (B, T, H, dv) or o.dtype not in _DTYPE_CODE:
        raise ValueError("inconsistent shapes")
    dims = make_chunk_dims(q, v, cu_seqlens, scale, max_seqlen, o.dtype)
    N = dims.num_seqs
    for name, t in (("hT", hT), ("h0", h0)):
        if t is not None and (t.dtype != torch.float32 or t.shape != (N, H, dk, dv)):
            raise ValueError("%s must be fp32 [N,H,dk,dv]" % name)
    st = lib.kda_chunk_fwd_static_scratch(ctypes.byref(dims), _ptr(q), _ptr(k), _ptr(v), _ptr(log_alpha), _ptr(beta),
                                          _ptr(h0), _ptr(cu_seqlens), _ptr(o), _ptr(hT), _stream_ptr(dev))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return o, hT


def kda_chunk_bwd_workspace_size(dims):
    return int(load_library().kda_chunk_bwd_workspace_size(ctypes.byref(dims)))


def kda_chunk_bwd(q, k, v, log_alpha, beta, do, dhT=None, h0=None, cu_seqlens=None, scale=1.0,
                  want_dh0=True, workspace=None, max_seqlen=0, out=None):
    """Backward pass of kda_chunk_fwd.  Inputs as there; do [B,T,H,dv] fp32, or bf16 with bf16 inputs;
    dhT fp32 [N,H,dk,dv] or None.  Returns a dict of fp32 tensors dq, dk, dlog_alpha [B,T,H,dk], dv [B,T,H,dv], dbeta [B,T,H]
    and dh0 [N,H,dk,dv] (None unless want_dh0); rows of tokens that belong to no sequence are zero
    (this wrapper clears them in the gradients it allocates; the library leaves such rows untouched).  `out`:
    the dict an earlier call returned, to be written in place instead of allocating."""
    lib = load_library()
    dev = _check_dev(q, k, v, log_alpha, beta, do, dhT, h0, cu_seqlens, workspace)
    if not (q.dtype == k.dtype == v.dtype == log_alpha.dtype == beta.dtype) or q.dtype not in _DTYPE_CODE:
        raise ValueError("q, k, v, log_alpha, beta must share a supported dtype")
    B, T, H, dk = q.shape
    dv = v.shape[-1]
    if k.shape != q.shape or log_alpha.shape != q.shape or v.shape != (B, T, H, dv) or beta.shape != (B, T, H):
        raise ValueError("inconsistent input shapes")
    if do.dtype not in _DTYPE_CODE or do.shape != (B, T, H, dv):
        raise ValueError("do must be fp32 or bf16 [B,T,H,dv]")
    dims = make_chunk_dims(q, v, cu_seqlens, scale, max_seqlen, do.dtype)        # do has the dtype o had
    N = dims.num_seqs
    for name, t in (("dhT", dhT), ("h0", h0)):
        if t is not None and (t.dtype != torch.float32 or t.shape != (N, H, dk, dv)):
            raise ValueError("%s must be fp32 [N,H,dk,dv]" % name)
    if cu_seqlens is not None and cu_seqlens.dtype != torch.int32:
        raise ValueError("cu_seqlens must be int32")
    f32 = dict(dtype=torch.float32, device=dev)
    clear = None
    shapes = {"dq": (B, T, H, dk), "dk": (B, T, H, dk), "dv": (B, T, H, dv), "dlog_alpha": (B, T, H, dk),
              "dbeta": (B, T, H), "dh0": (N, H, dk, dv)}
    if out is None:
        # (five fills are five launches, which gradients of up to 64 MiB do not repay: 8192 rows x 16 heads x 64, 64 against 72 us in all)
        packed = cu_seqlens is not None
        filled = packed and T * H * dk * 4 > 64 << 20 and _mostly_unowned(cu_seqlens, T, max_seqlen)
        out = {n_: (torch.zeros if filled else torch.empty)(*sh, **f32) for n_, sh in shapes.items() if n_ != "dh0"}
        if packed and not filled:
            clear = list(out.values())
        out["dh0"] = torch.empty(*shapes["dh0"], **f32) if want_dh0 else None
    else:                                   # the dict of an earlier call with the same shapes, written in place
        for n_, sh in shapes.items():
            t = out.get(n_)
            if t is None and n_ == "dh0":
                continue
            if t is None or t.dtype != torch.float32 or tuple(t.shape) != sh or not t.is_contiguous():
                raise ValueError("out[%r] must be a contiguous fp32 tensor of shape %r" % (n_, sh))
        _check_dev(q, *[t for t in out.values() if t is not None])
    if workspace is None:
        need = kda_chunk_bwd_workspace_size(dims)
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=dev) if need else None
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    st = lib.kda_chunk_bwd(ctypes.byref(dims), _ptr(q), _ptr(k), _ptr(v), _ptr(log_alpha), _ptr(beta), _ptr(h0),
                           _ptr(cu_seqlens), _ptr(do), _ptr(dhT), _ptr(out["dq"]), _ptr(out["dk"]),
                           _ptr(out["dv"]), _ptr(out["dlog_alpha"]), _ptr(out["dbeta"]), _ptr(out["dh0"]),
                           _ptr(workspace), ctypes.c_size_t(ws_bytes), _stream_ptr(dev))
    if st != 0:
        raise KdaError(st, kda_last_error())
    if clear:                               # (behind the call, as in kda_chunk_fwd)
        _clear_unowned(cu_seqlens, clear)
    return out


def kda_chunk_fwd_scalar_gate(q, k, v, log_alpha_head, beta, **kw):
    """kda_chunk_fwd with one decay per (token, head): log_alpha_head [B,T,H] (the scalar-gate case
    of Eq. (1)); other arguments and the result as for kda_chunk_fwd."""
    return kda_chunk_fwd(q, k, v, log_alpha_head, beta, _scalar_gate=True, **kw)


def kda_recurrent_step(q, k, v, log_alpha, beta, S, scale=1.0, o=None, out_dtype=None):
    """One decode step.  q,k,log_alpha [N,H,dk]; v [N,H,dv]; beta [N,H];
    S fp32 [N,H,dk,dv], updated in place.  Returns o [N,H,dv] (fp32, or bf16 on request as in
    kda_chunk_fwd)."""
    lib = load_library()
    if _native is not None:
        done = _native.step(q, k, v, log_alpha, beta, S, scale, o, out_dtype)
        if done is not None:
            return _result(done)
    dev = _check_dev(q, k, v, log_alpha, beta, S, o)
    N, H, dk = q.shape
    dv = v.shape[-1]
    if S.dtype != torch.float32 or S.shape != (N, H, dk, dv):
        raise ValueError("S must be fp32 [N,H,dk,dv]")
    if q.dtype not in _DTYPE_CODE or not (q.dtype == k.dtype == v.dtype == log_alpha.dtype == beta.dtype):
        raise ValueError("q, k, v, log_alpha, beta must share a supported dtype")
    if min(k.numel(), log_alpha.numel()) < N * H * dk or v.numel() < N * H * dv or beta.numel() < N * H:
        raise ValueError("inconsistent input shapes")
    odt = _out_dtype(o, out_dtype)
    if o is None:
        o = torch.empty(N, H, dv, dtype=odt, device=dev)
    elif o.shape != (N, H, dv):
        raise ValueError("o must have shape [N,H,dv]")
    dims = KdaDims(batch=N, seqlen=1, heads=H, dk=dk, dv=dv, chunk=64, num_seqs=N,
                   in_dtype=_DTYPE_CODE[q.dtype], out_dtype=_DTYPE_CODE[odt], scale=float(scale), max_seqlen=0)
    st = lib.kda_recurrent_step(ctypes.byref(dims), _ptr(q), _ptr(k), _ptr(v), _ptr(log_alpha),
                                _ptr(beta), _ptr(S), _ptr(o), _stream_ptr(dev))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return o


def kda_recurrent_steps_fused(q, k, v, gate, beta, S_pool, state_indices=None, prologue=True, l2norm_eps=1e-6,
                              a_scale=None, dt_bias=None, out_gate=None, norm_weight=None, rms_eps=1e-6, **kw):
    """kda_recurrent_steps_pooled with the fused stages (see kda_chunk_fwd_fused)."""
    load_library()
    if _native is not None and kw.keys() <= _STEPS_OPTIONS:
        done = _native.steps(q, k, v, gate, beta, S_pool, state_indices, kw.get("scale", 1.0), kw.get("o"), kw.get("out_dtype"),
                             2 if prologue else 3, l2norm_eps, a_scale, dt_bias, out_gate, norm_weight, rms_eps)
        if done is not None:
            return _result(done)
    pro = _make_prologue(q.shape[2], q.shape[3], l2norm_eps, a_scale, dt_bias) if prologue else None
    return kda_recurrent_steps_pooled(q, k, v, gate, beta, S_pool, state_indices,
                                      _fused=(pro, _make_epilogue(v, out_gate, norm_weight, rms_eps)), **kw)


def kda_recurrent_steps_pooled_scalar_gate(q, k, v, log_alpha_head, beta, S_pool, state_indices=None, **kw):
    """kda_recurrent_steps_pooled with one decay per (token, head): log_alpha_head [N,Tq,H]."""
    return kda_recurrent_steps_pooled(q, k, v, log_alpha_head, beta, S_pool, state_indices, _scalar_gate=True, **kw)


def kda_recurrent_steps_pooled(q, k, v, log_alpha, beta, S_pool, state_indices=None, scale=1.0, o=None,
                               out_dtype=None, _fused=None, _scalar_gate=False):
    """Decode over a state pool.  q,k,log_alpha [N,Tq,H,dk]; v [N,Tq,H,dv]; beta [N,Tq,H];
    S_pool fp32 [P,H,dk,dv], the addressed states updated in place; state_indices int32 [N] on the
    device (negative = skip) or None for 0..N-1.  Returns o [N,Tq,H,dv] (fp32, or bf16 on request as in
    kda_chunk_fwd)."""
    lib = load_library()
    if _native is not None and _fused is None:
        done = _native.steps(q, k, v, log_alpha, beta, S_pool, state_indices, scale, o, out_dtype, int(bool(_scalar_gate)), 0.0, None, None,
                             None, None, 0.0)
        if done is not None:
            return _result(done)
    dev = _check_dev(q, k, v, log_alpha, beta, S_pool, state_indices, o)
    N, Tq, H, dk = q.shape
    dv = v.shape[-1]
    if S_pool.dtype != torch.float32 or S_pool.dim() != 4 or S_pool.shape[1:] != (H, dk, dv):
        raise ValueError("S_pool must be fp32 [P,H,dk,dv]")
    if q.dtype not in _DTYPE_CODE or not (q.dtype == k.dtype == v.dtype == log_alpha.dtype == beta.dtype):
        raise ValueError("q, k, v, log_alpha, beta must share a supported dtype")
    if k.shape != q.shape or log_alpha.shape != ((N, Tq, H) if _scalar_gate else q.shape) \
            or v.shape != (N, Tq, H, dv) or beta.shape != (N, Tq, H):
        raise ValueError("inconsistent input shapes")
    if state_indices is None:
        if S_pool.shape[0] < N:
            raise ValueError("S_pool holds fewer states than there are sequences")
    elif state_indices.dtype != torch.int32 or state_indices.shape != (N,):
        raise ValueError("state_indices must be int32 [N]")
    odt = _out_dtype(o, out_dtype)
    flags = _SCALAR_GATE if _scalar_gate else 0
    if o is None:                           # (with indices: rows of skipped sequences are zero)
        o = torch.empty(N, Tq, H, dv, dtype=odt, device=dev)
        flags |= _ZERO_SKIPPED
    elif o.shape != (N, Tq, H, dv):
        raise ValueError("o must have shape [N,Tq,H,dv]")
    dims = KdaDims(batch=N, seqlen=Tq, heads=H, dk=dk, dv=dv, chunk=64, num_seqs=N,
                   in_dtype=_DTYPE_CODE[q.dtype], out_dtype=_DTYPE_CODE[odt], scale=float(scale), max_seqlen=0)
    pro, epi = _fused or (None, None)
    st = lib.kda_recurrent_steps(ctypes.byref(dims), None if pro is None else ctypes.byref(pro), None if epi is None else ctypes.byref(epi),
                                 _ptr(q), _ptr(k), _ptr(v), _ptr(log_alpha), _ptr(beta), _ptr(S_pool), _ptr(state_indices), _ptr(o),
                                 flags, _stream_ptr(dev))
    if st != 0:
        raise KdaError(st, kda_last_error())
    return o
