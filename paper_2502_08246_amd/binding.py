"""Binding of libsaap.so (declared in include/saap.h) to torch tensors.

Argument marshalling only: shapes are read off the tensors, pointers and the current HIP
stream are handed to the C entry points, status codes become exceptions.  Outputs are
allocated with torch (device memory) unless the caller passes them in.

The calls a program makes for every prompt, token or training step (NATIVE) are C++ functions on
torch tensors (csrc/native.cpp): marshalled here a call held the host for 10 to 15 us, as long as its
kernels take.  The others go through ctypes.
"""
from __future__ import annotations

import ctypes
import importlib
import os

import torch

F32, BF16 = 0, 1
GROUP_SUM, INDEPENDENT = 0, 1
PROBS, LOGITS = 0, 1
OP_ASSIGN_KEYS, OP_BUILD_BUCKET_INDEX, OP_CLASSIFY_QUERIES, OP_SELECT_BUCKETS = 0, 1, 2, 3
OP_SPARSE_DECODE_ATTENTION, OP_DENSE_DECODE_ATTENTION, OP_APPEND_KEYS, OP_WINDOW_PUSH = 4, 5, 6, 7
OP_BUCKET_ATTENTION_MASS, OP_QUERY_MODEL_LOSS_GRADS, OP_BUCKET_ATTENTION_MASS_BATCH = 8, 9, 10
OP_PLANNED_DECODE_ATTENTION, OP_PREFILL_SPARSE_ATTENTION, OP_UPDATE_CENTROIDS_FROM_IDS = 11, 12, 13
WS_HEADER_BYTES = 65536

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libsaap.so")
_NATIVE_PATH = os.path.join(_HERE, "_native.so")
_lib = None
_native = None

NATIVE = (
    "assign_keys", "build_bucket_index", "build_windowed_index", "quantize_kv",
    "classify_queries", "select_buckets", "select_buckets_from_logits", "build_visit_plan", "select_buckets_planned",
    "sparse_decode_attention", "sparse_decode_attention_fp8", "windowed_decode_attention", "windowed_decode_attention_fp8",
    "dense_decode_attention", "dense_decode_attention_fp8", "select_attend", "select_attend_fp8",
    "planned_decode_attention", "planned_decode_attention_fp8", "prefill_sparse_attention",
    "append_keys", "append_keys_fp8", "window_push", "window_push_fp8", "adam_update",
)

EXPORTS = (
    "saap_workspace_bytes", "saap_workspace_reset", "saap_status_string", "saap_device_compute_units",
    "saap_assign_keys", "saap_build_bucket_index", "saap_append_keys", "saap_classify_queries",
    "saap_select_buckets", "saap_sparse_decode_attention", "saap_dense_decode_attention", "saap_stream_read_probe", "saap_mfma_rate_probe",
    "saap_build_windowed_index", "saap_window_push", "saap_windowed_decode_attention",
    "saap_append_keys_fp8", "saap_window_push_fp8",
    "saap_select_buckets_from_logits", "saap_update_centroids", "saap_recompact_index",
    "saap_quantize_kv", "saap_sparse_decode_attention_fp8", "saap_dense_decode_attention_fp8",
    "saap_windowed_decode_attention_fp8",
    "saap_bucket_attention_mass", "saap_query_model_loss_grads", "saap_adam_update",
    "saap_bucket_attention_mass_batch", "saap_query_model_bn_loss_grads", "saap_fold_batch_norm",
    "saap_build_visit_plan", "saap_select_buckets_planned", "saap_planned_decode_attention",
    "saap_planned_decode_attention_fp8", "saap_visit_plan_bytes", "saap_sparse_decode_attention_noalloc",
    "saap_prefill_sparse_attention", "saap_classify_select", "saap_select_attend", "saap_select_attend_fp8", "saap_select_attend_windowed",
    "saap_build_bucket_index_zeroed", "saap_build_windowed_index_zeroed",
    "saap_update_centroids_from_ids",
)


class SaapError(RuntimeError):
    def __init__(self, call: str, status: int):
        self.status = status
        super().__init__(f"{call} failed: {status_string(status)} ({status})")


class _Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("S", "Hq", "Hkv", "N", "B", "nprobe", "d", "hidden", "dtype", "mode")]


def library_path() -> str:
    return _LIB_PATH


def load_library():
    """Load the built library; build it first (python -m paper_2502_08246_amd.build) if absent."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            from . import build as _build
            _build.build()
        lib = ctypes.CDLL(_LIB_PATH)
        lib.saap_workspace_bytes.restype = ctypes.c_size_t
        lib.saap_workspace_bytes.argtypes = [ctypes.c_int32, ctypes.POINTER(_Shape)]
        lib.saap_status_string.restype = ctypes.c_char_p
        lib.saap_status_string.argtypes = [ctypes.c_int32]
        for name in EXPORTS[4:] + ("saap_workspace_reset", "saap_device_compute_units"):
            getattr(lib, name).restype = ctypes.c_int32
        lib.saap_visit_plan_bytes.restype = ctypes.c_size_t
        lib.saap_visit_plan_bytes.argtypes = [ctypes.c_int32] * 5
        _lib = lib
    return _lib


def status_string(status: int) -> str:
    return load_library().saap_status_string(int(status)).decode()


def _check(call: str, status: int) -> None:
    if status != 0:
        raise SaapError(call, status)


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise TypeError(f"unsupported dtype {t.dtype}")


def _ptr(t):
    if t is None:
        return ctypes.c_void_p(0)
    if not t.is_cuda:
        raise ValueError("SAAP tensors must live in GPU memory; there is no CPU path")
    if not t.is_contiguous():
        raise ValueError("SAAP tensors must be contiguous")
    return ctypes.c_void_p(t.data_ptr())


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _i32(v):
    return ctypes.c_int32(int(v))


def workspace_bytes(op: int, **shape) -> int:
    sh = _Shape(**{k: int(v) for k, v in shape.items()})
    return int(load_library().saap_workspace_bytes(op, ctypes.byref(sh)))


def native():
    """The native call layer (csrc/native.cpp), built first if absent."""
    global _native
    if _native is None:
        load_library()
        if not os.path.exists(_NATIVE_PATH):
            from . import build as _build
            _build.build_native()
        _native = importlib.import_module("._native", __package__)
    return _native


def workspace(nbytes: int, device, asked_for: bool = True) -> torch.Tensor:
    """The shared workspace buffer of the device's current stream, at least nbytes long.

    Every stream has its own, zero-filled when it is made (which is what the header of arrival counters needs) and
    replaced by a larger one on demand: calls on different streams may run at the same time and never meet in one.  Pass
    it to calls on the stream it was asked for on.  One that a program has asked for is never freed.

    A HIP graph holds the RAW ADDRESS of the buffer that its calls were given: a capture takes over the buffer that the
    eager calls before it have made, all graphs of a device share that one (replay them one after the other, or capture
    with ws=), no eager call uses it again and it is never freed.  Growing while the current stream is capturing is
    refused (allocating there would also break the capture): run the call once eagerly first, or pass ws= explicitly."""
    device = torch.device(device)
    if device.type != "cuda":
        raise ValueError("SAAP workspaces live in GPU memory; there is no CPU path")
    return native().workspace(int(nbytes), torch.cuda.current_device() if device.index is None else device.index,
                              asked_for)


def _ws(op, device, ws, **shape):
    need = workspace_bytes(op, **shape)
    if need == 0:
        raise SaapError("saap_workspace_bytes", -1)
    if ws is None:
        ws = workspace(need, device, asked_for=False)
    return ws, ctypes.c_size_t(ws.numel())


def workspace_reset(ws: torch.Tensor) -> None:
    """Zeroes the header of a caller-provided workspace (needed once before its first use, or after a
    call was abandoned midway)."""
    st = load_library().saap_workspace_reset(_ptr(ws), ctypes.c_size_t(ws.numel()), _stream())
    _check("saap_workspace_reset", st)


def stream_read_probe(src: torch.Tensor, sink: torch.Tensor) -> None:
    """Measurement aid: one pass of non-temporal 16-byte loads over `src` (see saap_stream_read_probe)."""
    st = load_library().saap_stream_read_probe(_ptr(src), ctypes.c_size_t(src.numel() * src.element_size()), _ptr(sink),
                                               ctypes.c_size_t(sink.numel() * sink.element_size()), _stream())
    _check("saap_stream_read_probe", st)


def mfma_rate_probe(operands: torch.Tensor, iters: int, sink: torch.Tensor, wgs_per_cu: int = 2) -> float:
    """Measurement aid: enqueues the bare matrix-instruction loop on `operands` (bf16 values) and returns the
    floating-point operations of the launch (see saap_mfma_rate_probe)."""
    flop = ctypes.c_double(0.0)
    st = load_library().saap_mfma_rate_probe(_ptr(operands), ctypes.c_size_t(operands.numel() * operands.element_size()),
                                             ctypes.c_int32(iters), ctypes.c_int32(wgs_per_cu), _ptr(sink), ctypes.byref(flop),
                                             _stream())
    _check("saap_mfma_rate_probe", st)
    return flop.value


def classify_select(xq, W1, b1, W2, b2, Hkv, nprobe, off=None, ln=None, resident_run=-1, want_plan=False, logits=None,
                    probs=None, out=None, plan=None, ws=None):
    """classify_queries (logits) + the group selection in one call. -> (logits [S,Hq,B], selected [S,Hkv,nprobe], plan
    or None).  want_plan (or plan=) also writes the lists' visit plan, which needs off and ln."""
    S, Hq, d = xq.shape
    Hw, hidden, _ = W1.shape
    B = W2.shape[1]
    if W2.shape != (Hw, B, hidden) or W1.dtype != xq.dtype or W2.dtype != xq.dtype:
        raise ValueError("W1 [Hw,hidden,d] and W2 [Hw,B,hidden] must match xq's dtype")
    dev = xq.device
    logits = logits if logits is not None else torch.empty(S, Hq, B, dtype=torch.float32, device=dev)
    sel = out if out is not None else torch.empty(S, Hkv, nprobe, dtype=torch.int32, device=dev)
    if want_plan or plan is not None:
        if off is None or ln is None:
            raise ValueError("a visit plan needs off and ln")
        plan = _plan_buffer(plan, S, Hq, Hkv, nprobe + (1 if resident_run >= 0 else 0), GROUP_SUM, dev)
    ws, wsb = _ws(OP_CLASSIFY_QUERIES, dev, ws, S=S, Hq=Hq, hidden=hidden)
    st = load_library().saap_classify_select(
        _ptr(xq), _ptr(W1), _ptr(b1), _ptr(W2), _ptr(b2), _i32(Hw), _ptr(logits), _ptr(probs), _ptr(sel), _ptr(off),
        _ptr(ln), _i32(resident_run), _ptr(plan), _i32(S), _i32(Hq), _i32(Hkv), _i32(d), _i32(hidden), _i32(B),
        _i32(nprobe), _i32(_dtype_code(xq)), _ptr(ws), wsb, _stream())
    _check("saap_classify_select", st)
    return logits, sel, plan


def visit_plan_ints(S, Hq, Hkv, nruns, mode=GROUP_SUM) -> int:
    """int32 elements of the visit plan of S*Hkv (GROUP_SUM) or S*Hq (INDEPENDENT) lists of nruns runs."""
    nbytes = int(load_library().saap_visit_plan_bytes(int(S), int(Hq), int(Hkv), int(nruns), int(mode)))
    if nbytes == 0:
        raise SaapError("saap_visit_plan_bytes", -1)
    return nbytes // 4


def _plan_buffer(plan, S, Hq, Hkv, nruns, mode, device):
    n = visit_plan_ints(S, Hq, Hkv, nruns, mode)
    if plan is None:
        plan = torch.empty(n, dtype=torch.int32, device=device)
    elif plan.dtype != torch.int32 or plan.numel() < n:
        raise ValueError(f"plan must be int32 with at least {n} elements")
    return plan


def sparse_decode_attention_noalloc(q, Ks, Vs, off, ln, selected, scale, out, lse, mode=GROUP_SUM):
    """sparse_decode_attention without a workspace argument: the library's built-in scratch array serves.  The
    caller passes every output; nothing is allocated here or in the library."""
    S, Hq, d = q.shape
    _, Hkv, Ncap, _ = Ks.shape
    B = ln.shape[2]
    nprobe = selected.shape[2]
    st = load_library().saap_sparse_decode_attention_noalloc(
        _ptr(q), _ptr(Ks), _ptr(Vs), _ptr(off), _ptr(ln), _ptr(selected) if nprobe > 0 else ctypes.c_void_p(0),
        _i32(nprobe), _i32(mode), ctypes.c_float(scale), _ptr(out), _i32(_dtype_code(out)), _ptr(lse), _i32(S),
        _i32(Hq), _i32(Hkv), _i32(Ncap), _i32(B), _i32(d), _i32(_dtype_code(q)), _stream())
    _check("saap_sparse_decode_attention_noalloc", st)
    return out, lse


def bucket_attention_mass(q, Ks, off, ln, scale, out=None, lse=None, ws=None):
    """q [S,Hq,d]; Ks [S,Hkv,Ncap,d]; off, ln from build_bucket_index -> mass fp32 [S,Hq,B], lse fp32 [S,Hq]."""
    S, Hq, d = q.shape
    _, Hkv, Ncap, _ = Ks.shape
    B = ln.shape[2]
    dev = q.device
    mass = out if out is not None else torch.empty(S, Hq, B, dtype=torch.float32, device=dev)
    lse = lse if lse is not None else torch.empty(S, Hq, dtype=torch.float32, device=dev)
    ws, wsb = _ws(OP_BUCKET_ATTENTION_MASS, dev, ws, S=S, Hq=Hq, Hkv=Hkv, B=B)
    st = load_library().saap_bucket_attention_mass(
        _ptr(q), _ptr(Ks), _ptr(off), _ptr(ln), ctypes.c_float(scale), _ptr(mass), _ptr(lse), _i32(S), _i32(Hq),
        _i32(Hkv), _i32(Ncap), _i32(B), _i32(d), _i32(_dtype_code(q)), _ptr(ws), wsb, _stream())
    _check("saap_bucket_attention_mass", st)
    return mass, lse


def bucket_attention_mass_batch(q, Ks, off, ln, scale, out=None, lse=None, ws=None):
    """q [S,Hkv,R,d] bf16 (R queries per KV head); Ks [S,Hkv,Ncap,d] -> mass fp32 [S,Hkv,R,B], lse fp32 [S,Hkv,R]."""
    S, Hkv, R, d = q.shape
    Ncap = Ks.shape[2]
    B = ln.shape[2]
    dev = q.device
    mass = out if out is not None else torch.empty(S, Hkv, R, B, dtype=torch.float32, device=dev)
    lse = lse if lse is not None else torch.empty(S, Hkv, R, dtype=torch.float32, device=dev)
    ws, wsb = _ws(OP_BUCKET_ATTENTION_MASS_BATCH, dev, ws, S=S, Hkv=Hkv, N=R, B=B)
    st = load_library().saap_bucket_attention_mass_batch(
        _ptr(q), _ptr(Ks), _ptr(off), _ptr(ln), ctypes.c_float(scale), _ptr(mass), _ptr(lse), _i32(S), _i32(Hkv),
        _i32(R), _i32(Ncap), _i32(B), _i32(d), _i32(_dtype_code(q)), _ptr(ws), wsb, _stream())
    _check("saap_bucket_attention_mass_batch", st)
    return mass, lse


class _MlpF32(ctypes.Structure):
    _fields_ = [("W1", ctypes.c_void_p), ("b1", ctypes.c_void_p), ("W2", ctypes.c_void_p), ("b2", ctypes.c_void_p)]


def _mlp_struct(tensors):
    for t in tensors:
        if t.dtype != torch.float32:
            raise TypeError("the query model is trained in fp32")
    return _MlpF32(*(_ptr(t) for t in tensors))


def query_model_loss_grads(x, target, params, grads=None, loss=None, ws=None):
    """x [Hw,R,d] (bf16 or fp32), target fp32 [Hw,R,B], params = (W1 [Hw,hidden,d], b1 [Hw,hidden], W2 [Hw,B,hidden],
    b2 [Hw,B]) fp32 -> loss fp32 [Hw], grads (tuple shaped like params)."""
    Hw, R, d = x.shape
    W1, b1, W2, b2 = params
    hidden, B = W1.shape[1], W2.shape[1]
    if W1.shape != (Hw, hidden, d) or b1.shape != (Hw, hidden) or W2.shape != (Hw, B, hidden) or b2.shape != (Hw, B):
        raise ValueError("parameter shapes do not fit x")
    if target.shape != (Hw, R, B) or target.dtype != torch.float32:
        raise ValueError("target must be fp32 [Hw,R,B]")
    dev = x.device
    grads = grads if grads is not None else tuple(torch.empty_like(p) for p in params)
    loss = loss if loss is not None else torch.empty(Hw, dtype=torch.float32, device=dev)
    ws, wsb = _ws(OP_QUERY_MODEL_LOSS_GRADS, dev, ws, Hkv=Hw, N=R, d=d, hidden=hidden, B=B)
    ps, gs = _mlp_struct(params), _mlp_struct(grads)
    st = load_library().saap_query_model_loss_grads(
        _ptr(x), _ptr(target), ctypes.byref(ps), ctypes.byref(gs), _ptr(loss), _i32(Hw), _i32(R), _i32(d), _i32(hidden),
        _i32(B), _i32(_dtype_code(x)), _ptr(ws), wsb, _stream())
    _check("saap_query_model_loss_grads", st)
    return loss, grads


class _BatchNormF32(ctypes.Structure):
    _fields_ = [("gamma", ctypes.c_void_p), ("beta", ctypes.c_void_p), ("grad_gamma", ctypes.c_void_p),
                ("grad_beta", ctypes.c_void_p), ("running_mean", ctypes.c_void_p), ("running_var", ctypes.c_void_p),
                ("momentum", ctypes.c_float), ("eps", ctypes.c_float)]


def query_model_bn_loss_grads(x, target, params, gamma, beta, running_mean=None, running_var=None, momentum=0.1, eps=1e-5,
                              grads=None, grad_gamma=None, grad_beta=None, loss=None, ws=None):
    """query_model_loss_grads for the model with batch normalisation of the hidden layer; gamma, beta [Hw,hidden]
    fp32; running_mean / running_var (both or neither) are updated in place.
    -> loss [Hw], grads (dW1, db1, dW2, db2), grad_gamma, grad_beta."""
    Hw, R, d = x.shape
    W1, b1, W2, b2 = params
    hidden, B = W1.shape[1], W2.shape[1]
    if W1.shape != (Hw, hidden, d) or b1.shape != (Hw, hidden) or W2.shape != (Hw, B, hidden) or b2.shape != (Hw, B):
        raise ValueError("parameter shapes do not fit x")
    if target.shape != (Hw, R, B) or target.dtype != torch.float32:
        raise ValueError("target must be fp32 [Hw,R,B]")
    for t in (gamma, beta, running_mean, running_var):
        if t is not None and (t.shape != (Hw, hidden) or t.dtype != torch.float32):
            raise ValueError("gamma, beta and the running statistics must be fp32 [Hw,hidden]")
    dev = x.device
    grads = grads if grads is not None else tuple(torch.empty_like(p) for p in params)
    grad_gamma = grad_gamma if grad_gamma is not None else torch.empty_like(gamma)
    grad_beta = grad_beta if grad_beta is not None else torch.empty_like(beta)
    loss = loss if loss is not None else torch.empty(Hw, dtype=torch.float32, device=dev)
    ws, wsb = _ws(OP_QUERY_MODEL_LOSS_GRADS, dev, ws, Hkv=Hw, N=R, d=d, hidden=hidden, B=B)
    ps, gs = _mlp_struct(params), _mlp_struct(grads)
    bn = _BatchNormF32(_ptr(gamma), _ptr(beta), _ptr(grad_gamma), _ptr(grad_beta), _ptr(running_mean), _ptr(running_var),
                       momentum, eps)
    st = load_library().saap_query_model_bn_loss_grads(
        _ptr(x), _ptr(target), ctypes.byref(ps), ctypes.byref(gs), ctypes.byref(bn), _ptr(loss), _i32(Hw), _i32(R),
        _i32(d), _i32(hidden), _i32(B), _i32(_dtype_code(x)), _ptr(ws), wsb, _stream())
    _check("saap_query_model_bn_loss_grads", st)
    return loss, grads, grad_gamma, grad_beta


def fold_batch_norm(W1, b1, gamma, beta, running_mean, running_var, eps=1e-5, out_dtype=torch.bfloat16):
    """-> (W1' [Hw,hidden,d] out_dtype, b1' fp32): the inference form of the normalised first layer."""
    Hw, hidden, d = W1.shape
    for t in (W1, b1, gamma, beta, running_mean, running_var):
        if t.dtype != torch.float32:
            raise TypeError("fold_batch_norm takes fp32 tensors")
    W1o = torch.empty(Hw, hidden, d, dtype=out_dtype, device=W1.device)
    b1o = torch.empty(Hw, hidden, dtype=torch.float32, device=W1.device)
    st = load_library().saap_fold_batch_norm(_ptr(W1), _ptr(b1), _ptr(gamma), _ptr(beta), _ptr(running_mean),
                                             _ptr(running_var), ctypes.c_float(eps), _ptr(W1o), _ptr(b1o), _i32(Hw),
                                             _i32(hidden), _i32(d), _i32(_dtype_code(W1o)), _stream())
    _check("saap_fold_batch_norm", st)
    return W1o, b1o


def recompact_index(off, ln, idx, Ks, Vs, slack_new, Ncap_new, resident=False, overflow_flag=None):
    """Fresh slack behind every bucket without re-assignment. -> (off_new, idx_new, Ks_new, Vs_new, overflow_flag);
    ln stays valid."""
    S, Hkv, Ncap, d = Ks.shape
    runs = ln.shape[2]
    B = runs - (1 if resident else 0)
    dev = Ks.device
    off_new = torch.empty_like(off)
    idx_new = torch.empty(S, Hkv, Ncap_new, dtype=torch.int32, device=dev)
    Kn = torch.zeros(S, Hkv, Ncap_new, d, dtype=Ks.dtype, device=dev)
    Vn = torch.zeros(S, Hkv, Ncap_new, d, dtype=Ks.dtype, device=dev)
    if overflow_flag is None:
        overflow_flag = torch.zeros(4, dtype=torch.int32, device=dev)
    st = load_library().saap_recompact_index(_ptr(off), _ptr(ln), _ptr(idx), _ptr(Ks), _ptr(Vs), _ptr(off_new),
                                             _ptr(idx_new), _ptr(Kn), _ptr(Vn), _ptr(overflow_flag), _i32(S), _i32(Hkv),
                                             _i32(Ncap), _i32(Ncap_new), _i32(B), _i32(1 if resident else 0), _i32(d),
                                             _i32(_dtype_code(Ks)), _i32(slack_new), _stream())
    _check("saap_recompact_index", st)
    return off_new, idx_new, Kn, Vn, overflow_flag


def update_centroids(x_sorted, off, ln, centroids_old, normalize=True, out=None):
    """x_sorted [S,Hkv,Ncap,d] (features grouped by build_bucket_index), off, ln -> new centroids [Hkv,B,d]."""
    S, Hkv, Ncap, d = x_sorted.shape
    B = ln.shape[2]
    new = out if out is not None else torch.empty_like(centroids_old)
    st = load_library().saap_update_centroids(_ptr(x_sorted), _ptr(off), _ptr(ln), _ptr(centroids_old), _ptr(new),
                                              _i32(S), _i32(Hkv), _i32(Ncap), _i32(B), _i32(d),
                                              _i32(_dtype_code(x_sorted)), _i32(1 if normalize else 0), _stream())
    _check("saap_update_centroids", st)
    return new


def update_centroids_from_ids(x, bucket_ids, centroids_old, normalize=True, out=None, ws=None):
    """x [S,Hkv,N,d] and its bucket_ids int32 [S,Hkv,N] (assign_keys) -> new centroids [Hkv,B,d]."""
    S, Hkv, N, d = x.shape
    B = centroids_old.shape[1]
    if bucket_ids.shape != (S, Hkv, N) or bucket_ids.dtype != torch.int32 or centroids_old.dtype != x.dtype:
        raise ValueError("bucket_ids must be int32 [S,Hkv,N] and the centroids in the dtype of x")
    new = out if out is not None else torch.empty_like(centroids_old)
    ws, wsb = _ws(OP_UPDATE_CENTROIDS_FROM_IDS, x.device, ws, S=S, Hkv=Hkv, N=N, B=B)
    st = load_library().saap_update_centroids_from_ids(
        _ptr(x), _ptr(bucket_ids), _ptr(centroids_old), _ptr(new), _i32(S), _i32(Hkv), _i32(N), _i32(B), _i32(d),
        _i32(_dtype_code(x)), _i32(1 if normalize else 0), _ptr(ws), wsb, _stream())
    _check("saap_update_centroids_from_ids", st)
    return new


def lloyd_iterations(x, centroids, iters, normalize=True):
    """`iters` iterations of (spherical) k-means on the device, composed of the library's calls: assign_keys and
    update_centroids_from_ids.  x [S,Hkv,N,d], centroids [Hkv,B,d] (the initial ones; not modified) -> new centroids."""
    c = centroids
    for _ in range(iters):
        c = update_centroids_from_ids(x, assign_keys(x, c), c, normalize)
    return c


def _built_on_first_use(name):
    def call(*args, **kwargs):
        return getattr(native(), name)(*args, **kwargs)

    call.__name__ = call.__qualname__ = name
    return call


try:
    from . import _native
except ImportError:     # not built yet: the first call builds it, or says why it cannot be loaded
    globals().update({_n: _built_on_first_use(_n) for _n in NATIVE})
else:
    globals().update({_n: getattr(_native, _n) for _n in NATIVE})
