"""Python binding of include/lsq.h.  Argument marshalling only: the calls themselves go through csrc/calls.cpp (a CPython
extension, `_calls`), `load()` gives the same entry points as ctypes functions.

Every wrapper takes torch tensors that already live on the GPU, passes their
device pointers, the sizes and the current HIP stream to the C entry point of
the same name, and returns the output tensors.  Optional `out=`-style arguments
let a caller (the benchmark) reuse buffers so that a call allocates nothing.
"""
from __future__ import annotations

import ctypes as C
import os
import sysconfig

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "liblsq.so")
_CALLS_PATH = os.path.join(_HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
_lib = None

LSQ_F16, LSQ_BF16, LSQ_F32 = 0, 1, 2
LSQ_OP_LAYERNORM_BWD, LSQ_OP_BIAS_DROPOUT_RESIDUAL_BWD, LSQ_OP_BIAS_ACT_DROPOUT_BWD = 0, 1, 2
LSQ_OP_SPLIT_HEADS_BWD = 3
LSQ_OP_EMBEDDING_BWD = 4
LSQ_OP_BDR_LAYERNORM_BWD = 5
LSQ_ACT = {"relu": 0, "gelu": 1, "gelu_tanh": 2}
_DT = {torch.float16: LSQ_F16, torch.bfloat16: LSQ_BF16, torch.float32: LSQ_F32}

EXPORTS = [
    "lsq_workspace_bytes", "lsq_status_string", "lsq_layernorm_fwd", "lsq_layernorm_bwd", "lsq_layernorm_bwd_noalloc",
    "lsq_bias_dropout_residual_fwd", "lsq_bias_dropout_residual_bwd", "lsq_softmax_fwd", "lsq_softmax_bwd",
    "lsq_ls_xent_fwd", "lsq_ls_xent_bwd", "lsq_ls_xent_fwd_bwd", "lsq_adam_step",
    "lsq_bias_act_dropout_fwd", "lsq_bias_act_dropout_bwd", "lsq_adam_step_lp", "lsq_sgd_step",
    "lsq_split_heads_fwd", "lsq_split_heads_bwd", "lsq_merge_heads_fwd", "lsq_merge_heads_bwd",
    "lsq_embedding_fwd", "lsq_embedding_bwd",
    "lsq_bdr_layernorm_fwd", "lsq_bdr_layernorm_bwd",
    "lsq_adam_state_bytes", "lsq_adam_state_pack", "lsq_adam_state_unpack", "lsq_adam_step_blocked",
    "lsq_trainer_state_bytes", "lsq_trainer_state_pack", "lsq_trainer_state_unpack", "lsq_sgd_step_blocked",
    "lsq_adam_step_lp_blocked",
    "lsq_pad_offsets", "lsq_pad_remove", "lsq_pad_restore", "lsq_softmax_varlen_fwd", "lsq_softmax_varlen_bwd",
    "lsq_calib_stream", "lsq_softmax_candidates", "lsq_softmax_tune",
]


class LsqError(RuntimeError):
    pass


def lib_path() -> str:
    return _LIB_PATH


def load():
    """Load liblsq.so (built by `python -m paper_2110_05722_amd.build`).  Raises if absent."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise LsqError(f"{_LIB_PATH} is missing: build it with `python -m paper_2110_05722_amd.build` "
                       "(there is no fallback path)")
    lib = C.CDLL(_LIB_PATH)
    vp, i32, i64, u64, f32, sz = C.c_void_p, C.c_int32, C.c_int64, C.c_uint64, C.c_float, C.c_size_t
    sig = {
        "lsq_workspace_bytes": (sz, [i32, i64, i32]),
        "lsq_status_string": (C.c_char_p, [C.c_int]),
        "lsq_layernorm_fwd": (C.c_int, [vp, vp, vp, vp, vp, vp, i64, i32, f32, C.c_int, vp]),
        "lsq_layernorm_bwd": (C.c_int, [vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, i64, i32, C.c_int, vp]),
        "lsq_layernorm_bwd_noalloc": (C.c_int, [vp, vp, vp, vp, vp, vp, vp, vp, vp, i64, i32, C.c_int, vp]),
        "lsq_calib_stream": (C.c_int, [i32, vp, vp, i64, vp]),
        "lsq_softmax_candidates": (i32, [i32]),
        "lsq_softmax_tune": (C.c_int, [vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64,
                                       C.c_int, i32, i32, vp]),
        "lsq_bias_dropout_residual_fwd": (C.c_int, [vp, vp, vp, vp, i64, i32, f32, u64, u64, C.c_int, vp]),
        "lsq_bias_dropout_residual_bwd": (C.c_int, [vp, vp, vp, i64, i32, f32, u64, u64, vp, sz, C.c_int, vp]),
        "lsq_softmax_fwd": (C.c_int, [vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64, C.c_int, vp]),
        "lsq_softmax_bwd": (C.c_int, [vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64, C.c_int, vp]),
        "lsq_ls_xent_fwd": (C.c_int, [vp, vp, vp, vp, vp, vp, i64, i32, f32, i32, C.c_int, vp]),
        "lsq_ls_xent_bwd": (C.c_int, [vp, vp, vp, vp, i64, i32, f32, i32, f32, C.c_int, vp]),
        "lsq_ls_xent_fwd_bwd": (C.c_int, [vp, vp, vp, vp, vp, vp, vp, i64, i32, f32, i32, f32, C.c_int, vp]),
        "lsq_adam_step": (C.c_int, [vp, vp, vp, vp, vp, i64, f32, f32, f32, f32, f32, i32, i32, i32, f32,
                                    C.c_int, C.c_int, vp]),
        "lsq_bias_act_dropout_fwd": (C.c_int, [vp, vp, vp, i64, i32, i32, f32, u64, u64, C.c_int, vp]),
        "lsq_bias_act_dropout_bwd": (C.c_int, [vp, vp, vp, vp, vp, i64, i32, i32, f32, u64, u64, vp, sz, C.c_int, vp]),
        "lsq_adam_step_lp": (C.c_int, [vp, vp, vp, vp, i64, f32, f32, f32, f32, f32, i32, i32, i32, f32, C.c_int, vp]),
        "lsq_sgd_step": (C.c_int, [vp, vp, vp, vp, i64, f32, f32, f32, i32, f32, C.c_int, C.c_int, vp]),
        "lsq_split_heads_fwd": (C.c_int, [vp, vp, vp, vp, vp, i32, i32, i32, i32, i32, C.c_int, vp]),
        "lsq_split_heads_bwd": (C.c_int, [vp, vp, vp, vp, vp, i32, i32, i32, i32, i32, vp, sz, C.c_int, vp]),
        "lsq_merge_heads_fwd": (C.c_int, [vp, vp, i32, i32, i32, i32, C.c_int, vp]),
        "lsq_merge_heads_bwd": (C.c_int, [vp, vp, i32, i32, i32, i32, C.c_int, vp]),
        "lsq_embedding_fwd": (C.c_int, [vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64, C.c_int, vp]),
        "lsq_embedding_bwd": (C.c_int, [vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64, vp, sz, C.c_int, vp]),
        "lsq_bdr_layernorm_fwd": (C.c_int, [vp, vp, vp, vp, vp, vp, vp, vp, vp, i64, i32, f32, u64, u64, f32, C.c_int, vp]),
        "lsq_bdr_layernorm_bwd": (C.c_int, [vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, i64, i32, f32, u64, u64,
                                             C.c_int, vp]),
        "lsq_adam_state_bytes": (sz, [i64]),
        "lsq_adam_state_pack": (C.c_int, [vp, vp, vp, vp, i64, vp]),
        "lsq_adam_state_unpack": (C.c_int, [vp, vp, vp, vp, i64, vp]),
        "lsq_adam_step_blocked": (C.c_int, [vp, vp, vp, i64, f32, f32, f32, f32, f32, i32, i32, i32, f32, C.c_int, C.c_int, vp]),
        "lsq_trainer_state_bytes": (sz, [i64, i32]),
        "lsq_trainer_state_pack": (C.c_int, [vp, vp, vp, vp, i64, i32, vp]),
        "lsq_trainer_state_unpack": (C.c_int, [vp, vp, vp, vp, i64, i32, vp]),
        "lsq_sgd_step_blocked": (C.c_int, [vp, vp, vp, i64, f32, f32, f32, i32, f32, C.c_int, C.c_int, vp]),
        "lsq_adam_step_lp_blocked": (C.c_int, [vp, vp, vp, i64, f32, f32, f32, f32, f32, i32, i32, i32, f32, C.c_int, vp]),
        "lsq_pad_offsets": (C.c_int, [vp, vp, i32, i32, vp]),
        "lsq_pad_remove": (C.c_int, [vp, vp, vp, i32, i32, i32, i64, C.c_int, vp]),
        "lsq_pad_restore": (C.c_int, [vp, vp, vp, i32, i32, i32, i64, C.c_int, vp]),
        "lsq_softmax_varlen_fwd": (C.c_int, [vp, vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64, C.c_int, vp]),
        "lsq_softmax_varlen_bwd": (C.c_int, [vp, vp, vp, vp, vp, i32, i32, i32, i32, i32, f32, f32, u64, u64, C.c_int, vp]),
    }
    for name, (res, args) in sig.items():
        fn = getattr(lib, name)
        fn.restype = res
        fn.argtypes = args
    _lib = lib
    return lib


def lsq_status_string(code: int) -> str:
    return load().lsq_status_string(code).decode()


def lsq_workspace_bytes(op: int, rows: int, cols: int) -> int:
    return int(load().lsq_workspace_bytes(op, rows, cols))


def _check(code: int, name: str):
    if code != 0:
        raise LsqError(f"{name} failed: {lsq_status_string(code)}")


def _ptr(t):
    """Device address of a tensor (an int: ctypes converts it for a c_void_p argument as fast as a ready-made object)."""
    if t is None:
        return None
    if not t.is_cuda:
        raise LsqError("tensors must live on the GPU (there is no CPU path)")
    if not t.is_contiguous():
        raise LsqError("tensors must be contiguous")
    return t.data_ptr()


def _dt(t) -> int:
    try:
        return _DT[t.dtype]
    except KeyError:
        raise LsqError(f"unsupported dtype {t.dtype}") from None


# torch's raw stream and device queries are not public: where a build has them under other names, the public call serves
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
_raw_device = getattr(torch._C, "_cuda_getDevice", None)


def _stream():
    """The current device's current stream, as an int.  torch.cuda.current_stream() builds a Stream object for it, 2.75 us of
    a 13 us call; the raw query takes 0.19.  It wants an initialised runtime, which the public call sees to."""
    if _raw_stream is None or _raw_device is None or not torch.cuda.is_initialized():
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_raw_device())


def _need(name: str, t, numel: int, dtype=None):
    """The library takes bare pointers: a tensor shorter than what the kernel will touch is refused here."""
    if t is None:
        return
    if t.numel() < numel:
        raise LsqError(f"{name} holds {t.numel()} elements, the call needs {numel}")
    if dtype is not None and t.dtype != dtype:
        raise LsqError(f"{name} is {t.dtype}, expected {dtype}")


class _Native:
    """csrc/calls.cpp, loaded by the first call: argument checks and conversions, output tensors, the C entry points themselves.
    What it does not take (tensor subclasses, an active function mode) comes back to _ptr, _need and the two below."""

    def __getattr__(self, name):
        global _native
        load()
        if not os.path.exists(_CALLS_PATH):
            raise LsqError(f"{_CALLS_PATH} is missing: build it with `python -m paper_2110_05722_amd.build` "
                           "(there is no fallback path)")
        try:
            from . import _calls
        except ImportError as e:
            raise LsqError(f"{_CALLS_PATH} does not load here ({e}): build it again") from e
        if _calls.torch_version != str(torch.__version__):
            raise LsqError(f"{_CALLS_PATH} was built for torch {_calls.torch_version}, this is {torch.__version__}: build it again")
        _calls.setup(LsqError, C.ArgumentError, lambda: _stream(), _ptr, _need, _empty, lambda t: torch.empty_like(t))
        _native = _calls
        return getattr(_calls, name)


_native = _Native()


def _empty(like, dtype, *size):
    return torch.empty(size, dtype=like.dtype if dtype is None else dtype, device=like.device)


def _workspace(op: int, rows: int, cols: int, like, ws):
    if ws is not None:
        return ws
    return _native.empty(like, torch.uint8, max(_native.workspace_bytes(op, rows, cols), 16))


# ---------------------------------------------------------------------------
def lsq_layernorm_fwd(x, gamma, beta, eps: float = 1e-5, y=None, mean=None, rstd=None):
    """x: [rows, hidden] -> (y, mean[rows] fp32, rstd[rows] fp32)."""
    rows, hidden = x.shape
    y = _native.empty_like(x) if y is None else y
    mean = _native.empty(x, torch.float32, rows) if mean is None else mean
    rstd = _native.empty(x, torch.float32, rows) if rstd is None else rstd
    _native.need("y", y, rows * hidden, x.dtype, "gamma", gamma, hidden, x.dtype, "beta", beta, hidden, x.dtype,
                  "mean", mean, rows, torch.float32, "rstd", rstd, rows, torch.float32)
    _native.lsq_layernorm_fwd(y, mean, rstd, x, gamma, beta, rows, hidden, eps, x.dtype)
    return y, mean, rstd


def lsq_layernorm_bwd(dy, x, gamma, mean, rstd, dres_in=None, dx=None, dgamma=None, dbeta=None, workspace=None):
    """-> (dx, dgamma[hidden] fp32, dbeta[hidden] fp32)."""
    rows, hidden = x.shape
    dx = _native.empty_like(x) if dx is None else dx
    dgamma = _native.empty(x, torch.float32, hidden) if dgamma is None else dgamma
    dbeta = _native.empty(x, torch.float32, hidden) if dbeta is None else dbeta
    ws = _workspace(LSQ_OP_LAYERNORM_BWD, rows, hidden, x, workspace)
    _native.need("dy", dy, rows * hidden, x.dtype, "dx", dx, rows * hidden, x.dtype,
                  "dres_in", dres_in, rows * hidden, x.dtype, "gamma", gamma, hidden, x.dtype,
                  "mean", mean, rows, torch.float32, "rstd", rstd, rows, torch.float32,
                  "dgamma", dgamma, hidden, torch.float32, "dbeta", dbeta, hidden, torch.float32)
    _native.lsq_layernorm_bwd(dx, dgamma, dbeta, dy, x, gamma, mean, rstd, dres_in, ws, ws.numel() * ws.element_size(), rows,
                               hidden, x.dtype)
    return dx, dgamma, dbeta


def lsq_layernorm_bwd_noalloc(dy, x, gamma, mean, rstd, dx, dgamma, dbeta, dres_in=None):
    """LayerNorm backward into caller-supplied outputs, scratch held by the library: the call allocates nothing."""
    rows, hidden = x.shape
    _native.need("dy", dy, rows * hidden, x.dtype, "dx", dx, rows * hidden, x.dtype,
                  "dres_in", dres_in, rows * hidden, x.dtype, "gamma", gamma, hidden, x.dtype,
                  "mean", mean, rows, torch.float32, "rstd", rstd, rows, torch.float32,
                  "dgamma", dgamma, hidden, torch.float32, "dbeta", dbeta, hidden, torch.float32)
    _native.lsq_layernorm_bwd_noalloc(dx, dgamma, dbeta, dy, x, gamma, mean, rstd, dres_in, rows, hidden, x.dtype)
    return dx, dgamma, dbeta


def lsq_bias_dropout_residual_fwd(x, bias, residual, p: float, seed: int, offset: int, out=None):
    rows, hidden = x.shape
    out = _native.empty_like(x) if out is None else out
    _native.need("out", out, rows * hidden, x.dtype, "residual", residual, rows * hidden, x.dtype,
                  "bias", bias, hidden, x.dtype)
    _native.lsq_bias_dropout_residual_fwd(out, x, bias, residual, rows, hidden, p, seed, offset, x.dtype)
    return out


def lsq_bias_dropout_residual_bwd(dy, p: float, seed: int, offset: int, want_dbias: bool = True, dx=None, dbias=None,
                                  workspace=None):
    """-> (dx, dbias[hidden] fp32 or None)."""
    rows, hidden = dy.shape
    dx = _native.empty_like(dy) if dx is None else dx
    if want_dbias and dbias is None:
        dbias = _native.empty(dy, torch.float32, hidden)
    ws = _workspace(LSQ_OP_BIAS_DROPOUT_RESIDUAL_BWD, rows, hidden, dy, workspace)
    _native.need("dx", dx, rows * hidden, dy.dtype, "dbias", dbias, hidden, torch.float32)
    _native.lsq_bias_dropout_residual_bwd(dx, dbias if want_dbias else None, dy, rows, hidden, p, seed, offset, ws,
                                           ws.numel() * ws.element_size(), dy.dtype)
    return dx, (dbias if want_dbias else None)


def lsq_softmax_fwd(x, key_len=None, causal: bool = False, scale: float = 1.0, p_attn: float = 0.0, seed: int = 0,
                    offset: int = 0, y=None, y_drop=None):
    """x: [batch, heads, q_len, k_len]; key_len: int32[batch] or None -> (y, y_drop or None)."""
    B, N, Lq, Lk = x.shape
    y = _native.empty_like(x) if y is None else y
    if p_attn > 0 and y_drop is None:
        y_drop = _native.empty_like(x)
    _native.need("y", y, x.numel(), x.dtype, "y_drop", y_drop, x.numel(), x.dtype, "key_len", key_len, B, torch.int32)
    _native.lsq_softmax_fwd(y, y_drop if p_attn > 0 else None, x, key_len, B, N, Lq, Lk, int(causal), scale, p_attn, seed,
                             offset, x.dtype)
    return y, (y_drop if p_attn > 0 else None)


def lsq_softmax_bwd(dy, y, key_len=None, causal: bool = False, scale: float = 1.0, p_attn: float = 0.0, seed: int = 0,
                    offset: int = 0, dx=None):
    B, N, Lq, Lk = y.shape
    dx = _native.empty_like(y) if dx is None else dx
    _native.need("dx", dx, y.numel(), y.dtype, "dy", dy, y.numel(), y.dtype, "key_len", key_len, B, torch.int32)
    _native.lsq_softmax_bwd(dx, dy, y, key_len, B, N, Lq, Lk, int(causal), scale, p_attn, seed, offset, y.dtype)
    return dx


def lsq_ls_xent_fwd(logits, target, alpha: float, ignore_index: int = -100, want_sums: bool = True,
                    want_nll: bool = True, loss=None, nll=None, lse=None, sums=None):
    """logits: [tokens, vocab]; target: int32[tokens] -> (loss[tokens], nll[tokens] or None, lse[tokens],
    sums[3] or None), all fp32."""
    T, V = logits.shape
    loss = _native.empty(logits, torch.float32, T) if loss is None else loss
    lse = _native.empty(logits, torch.float32, T) if lse is None else lse
    if want_nll and nll is None:
        nll = _native.empty(logits, torch.float32, T)
    if want_sums and sums is None:
        sums = _native.empty(logits, torch.float32, 3)
    _native.need("target", target, T, torch.int32, "loss", loss, T, torch.float32, "nll", nll, T, torch.float32,
                  "lse", lse, T, torch.float32, "sums", sums, 3, torch.float32)
    _native.lsq_ls_xent_fwd(loss, nll if want_nll else None, lse, sums if want_sums else None, logits, target, T, V, alpha,
                             ignore_index, logits.dtype)
    return loss, (nll if want_nll else None), lse, (sums if want_sums else None)


def lsq_ls_xent_bwd(logits, lse, target, alpha: float, ignore_index: int = -100, grad_scale: float = 1.0,
                    dlogits=None):
    T, V = logits.shape
    dlogits = _native.empty_like(logits) if dlogits is None else dlogits
    _native.need("target", target, T, torch.int32, "lse", lse, T, torch.float32, "dlogits", dlogits, T * V, logits.dtype)
    _native.lsq_ls_xent_bwd(dlogits, logits, lse, target, T, V, alpha, ignore_index, grad_scale, logits.dtype)
    return dlogits


def lsq_ls_xent_fwd_bwd(logits, target, alpha: float, ignore_index: int = -100, grad_scale: float = 1.0,
                        want_sums: bool = True, want_nll: bool = True, loss=None, nll=None, lse=None, sums=None,
                        dlogits=None):
    """Forward and backward in one pass -> (loss, nll or None, lse, sums or None, dlogits).  dlogits may be
    `logits` itself (in place)."""
    T, V = logits.shape
    loss = _native.empty(logits, torch.float32, T) if loss is None else loss
    lse = _native.empty(logits, torch.float32, T) if lse is None else lse
    if want_nll and nll is None:
        nll = _native.empty(logits, torch.float32, T)
    if want_sums and sums is None:
        sums = _native.empty(logits, torch.float32, 3)
    dlogits = _native.empty_like(logits) if dlogits is None else dlogits
    _native.need("target", target, T, torch.int32, "loss", loss, T, torch.float32, "nll", nll, T, torch.float32,
                  "lse", lse, T, torch.float32, "sums", sums, 3, torch.float32, "dlogits", dlogits, T * V, logits.dtype)
    _native.lsq_ls_xent_fwd_bwd(loss, nll if want_nll else None, lse, sums if want_sums else None, dlogits, logits, target, T,
                                 V, alpha, ignore_index, grad_scale, logits.dtype)
    return loss, (nll if want_nll else None), lse, (sums if want_sums else None), dlogits


def lsq_adam_step(p, m, v, g, p_lp=None, *, lr: float, beta1: float, beta2: float, eps: float, step: int,
                  weight_decay: float = 0.0, adamw: bool = False, bias_correction: bool = True,
                  inv_grad_scale: float = 1.0):
    """In place on fp32 p, m, v (flat); g low precision (or fp32); p_lp optional low-precision copy out."""
    for t in (p, m, v):
        if t.dtype != torch.float32:
            raise LsqError("p, m, v must be fp32")
    n = p.numel()
    _native.need("m", m, n, None, "v", v, n, None, "g", g, n, None, "p_lp", p_lp, n, None)
    _native.lsq_adam_step(p, m, v, g, p_lp, n, lr, beta1, beta2, eps, weight_decay, step, int(adamw), int(bias_correction),
                           inv_grad_scale, g.dtype, p_lp.dtype if p_lp is not None else LSQ_F16)
    return p, m, v, p_lp


def lsq_bias_act_dropout_fwd(x, bias, act: str, p: float, seed: int, offset: int, out=None):
    """out = Dropout_p(act(x + bias)); act in {"relu", "gelu", "gelu_tanh"}."""
    rows, hidden = x.shape
    out = _native.empty_like(x) if out is None else out
    _native.need("out", out, rows * hidden, x.dtype, "bias", bias, hidden, x.dtype)
    _native.lsq_bias_act_dropout_fwd(out, x, bias, rows, hidden, LSQ_ACT[act], p, seed, offset, x.dtype)
    return out


def lsq_bias_act_dropout_bwd(dy, x, bias, act: str, p: float, seed: int, offset: int, want_dbias: bool = True, dx=None,
                             dbias=None, workspace=None):
    """-> (dx, dbias[hidden] fp32 or None)."""
    rows, hidden = x.shape
    dx = _native.empty_like(x) if dx is None else dx
    if want_dbias and dbias is None:
        dbias = _native.empty(x, torch.float32, hidden)
    ws = _workspace(LSQ_OP_BIAS_ACT_DROPOUT_BWD, rows, hidden, x, workspace)
    _native.need("dy", dy, rows * hidden, x.dtype, "dx", dx, rows * hidden, x.dtype, "bias", bias, hidden, x.dtype,
                  "dbias", dbias, hidden, torch.float32)
    _native.lsq_bias_act_dropout_bwd(dx, dbias if want_dbias else None, dy, x, bias, rows, hidden, LSQ_ACT[act], p, seed,
                                      offset, ws, ws.numel() * ws.element_size(), x.dtype)
    return dx, (dbias if want_dbias else None)


def lsq_adam_step_lp(p_lp, m, v, g, *, lr: float, beta1: float, beta2: float, eps: float, step: int,
                     weight_decay: float = 0.0, adamw: bool = False, bias_correction: bool = True,
                     inv_grad_scale: float = 1.0):
    """In place on the low-precision p_lp and fp32 m, v (flat); g in the same low precision."""
    if g.dtype != p_lp.dtype:
        raise LsqError("g and p_lp must share one low-precision dtype")
    _native.need("m", m, p_lp.numel(), torch.float32, "v", v, p_lp.numel(), torch.float32, "g", g, p_lp.numel(), None)
    _native.lsq_adam_step_lp(p_lp, m, v, g, p_lp.numel(), lr, beta1, beta2, eps, weight_decay, step, int(adamw),
                              int(bias_correction), inv_grad_scale, p_lp.dtype)
    return p_lp, m, v


def lsq_sgd_step(p, momentum_buf, g, p_lp=None, *, lr: float, momentum: float = 0.0, weight_decay: float = 0.0,
                 nesterov: bool = False, inv_grad_scale: float = 1.0):
    """In place on fp32 p (and momentum_buf if momentum > 0); p_lp optional low-precision copy out."""
    if p.dtype != torch.float32:
        raise LsqError("p must be fp32")
    _native.need("momentum_buf", momentum_buf, p.numel(), torch.float32, "g", g, p.numel(), None,
                  "p_lp", p_lp, p.numel(), None)
    _native.lsq_sgd_step(p, momentum_buf, g, p_lp, p.numel(), lr, momentum, weight_decay, int(nesterov), inv_grad_scale,
                          g.dtype, p_lp.dtype if p_lp is not None else LSQ_F16)
    return p, momentum_buf, p_lp


def lsq_split_heads_fwd(x, bias, batch: int, length: int, heads: int, head_dim: int, parts: int, outs=None):
    """x: [batch*len, parts*heads*head_dim] (+ bias) -> list of `parts` tensors [batch, heads, len, head_dim]."""
    if outs is None:
        outs = [_native.empty(x, None, batch, heads, length, head_dim) for _ in range(parts)]
    hidden = heads * head_dim
    _native.need("x", x, batch * length * parts * hidden, None, "bias", bias, parts * hidden, x.dtype)
    if len(outs) < parts:
        raise LsqError(f"{parts} parts need {parts} output tensors")
    for o in outs[:parts]:
        _native.need("out", o, batch * length * hidden, x.dtype)
    o3 = [*outs[:parts], None, None, None]
    _native.lsq_split_heads_fwd(o3[0], o3[1], o3[2], x, bias, batch, length, heads, head_dim, parts, x.dtype)
    return outs


def lsq_split_heads_bwd(grads, batch: int, length: int, heads: int, head_dim: int, want_dbias: bool = True, din=None,
                        dbias=None, workspace=None):
    """grads: list of `parts` tensors [batch, heads, len, head_dim] -> (din [batch*len, parts*hidden], dbias or None)."""
    parts = len(grads)
    cols = parts * heads * head_dim
    g0 = grads[0]
    din = _native.empty(g0, None, batch * length, cols) if din is None else din
    if want_dbias and dbias is None:
        dbias = _native.empty(g0, torch.float32, cols)
    ws = _workspace(LSQ_OP_SPLIT_HEADS_BWD, batch * length, cols, g0, workspace)
    if not 1 <= parts <= 3:
        raise LsqError("1 to 3 parts")
    for g in grads:
        _native.need("grad", g, batch * length * heads * head_dim, g0.dtype)
    _native.need("din", din, batch * length * cols, g0.dtype, "dbias", dbias, cols, torch.float32)
    g3 = [*grads, None, None, None]
    _native.lsq_split_heads_bwd(din, dbias if want_dbias else None, g3[0], g3[1], g3[2], batch, length, heads, head_dim,
                                 parts, ws, ws.numel() * ws.element_size(), g0.dtype)
    return din, (dbias if want_dbias else None)


def lsq_merge_heads_fwd(x, out=None):
    """x: [batch, heads, len, head_dim] -> [batch*len, heads*head_dim]."""
    B, N, Ln, D = x.shape
    out = _native.empty(x, None, B * Ln, N * D) if out is None else out
    _native.need("out", out, x.numel(), x.dtype)
    _native.lsq_merge_heads_fwd(out, x, B, Ln, N, D, x.dtype)
    return out


def lsq_merge_heads_bwd(dy, batch: int, length: int, heads: int, head_dim: int, dx=None):
    """dy: [batch*len, heads*head_dim] -> [batch, heads, len, head_dim]."""
    dx = _native.empty(dy, None, batch, heads, length, head_dim) if dx is None else dx
    _native.need("dy", dy, batch * heads * length * head_dim, None, "dx", dx, batch * heads * length * head_dim, dy.dtype)
    _native.lsq_merge_heads_bwd(dx, dy, batch, length, heads, head_dim, dy.dtype)
    return dx


def lsq_embedding_fwd(tokens, emb, pos, pad_idx: int, scale: float, p: float, seed: int, offset: int, out=None):
    """tokens: int32 [batch, len]; emb: [vocab, hidden]; pos: [>= len, hidden] -> out [batch*len, hidden]."""
    if tokens.dtype != torch.int32:
        raise LsqError("tokens must be int32")
    B, Ln = tokens.shape
    V, H = emb.shape
    out = _native.empty(emb, None, B * Ln, H) if out is None else out
    _native.need("out", out, B * Ln * H, emb.dtype, "pos", pos, Ln * H, emb.dtype)
    if pos.shape[-1] != H:
        raise LsqError("pos must be [>= len, hidden]")
    _native.lsq_embedding_fwd(out, tokens, emb, pos, B, Ln, H, V, pad_idx, scale, p, seed, offset, emb.dtype)
    return out


def lsq_embedding_bwd(demb, dpos, dy, tokens, pad_idx: int, scale: float, p: float, seed: int, offset: int,
                      workspace=None):
    """Accumulates into demb [vocab, hidden] and (if not None) dpos [len, hidden]."""
    if tokens.dtype != torch.int32:
        raise LsqError("tokens must be int32")
    B, Ln = tokens.shape
    V, H = demb.shape
    ws = _workspace(LSQ_OP_EMBEDDING_BWD, B * Ln, H, dy, workspace)
    _native.need("dy", dy, B * Ln * H, demb.dtype, "dpos", dpos, Ln * H, demb.dtype)
    _native.lsq_embedding_bwd(demb, dpos, dy, tokens, B, Ln, H, V, pad_idx, scale, p, seed, offset, ws,
                               ws.numel() * ws.element_size(), demb.dtype)
    return demb, dpos


def lsq_bdr_layernorm_fwd(x, bias, residual, gamma, beta, p: float, seed: int, offset: int, eps: float = 1e-5,
                          h=None, y=None, mean=None, rstd=None):
    """h = residual + Dropout(x + bias); y = LayerNorm(h), one pass -> (h, y, mean, rstd)."""
    rows, hidden = x.shape
    h = _native.empty_like(x) if h is None else h
    y = _native.empty_like(x) if y is None else y
    mean = _native.empty(x, torch.float32, rows) if mean is None else mean
    rstd = _native.empty(x, torch.float32, rows) if rstd is None else rstd
    _native.need("h", h, rows * hidden, x.dtype, "y", y, rows * hidden, x.dtype, "residual", residual, rows * hidden, x.dtype,
                  "bias", bias, hidden, x.dtype, "gamma", gamma, hidden, x.dtype, "beta", beta, hidden, x.dtype,
                  "mean", mean, rows, torch.float32, "rstd", rstd, rows, torch.float32)
    _native.lsq_bdr_layernorm_fwd(h, y, mean, rstd, x, bias, residual, gamma, beta, rows, hidden, p, seed, offset, eps,
                                   x.dtype)
    return h, y, mean, rstd


def lsq_bdr_layernorm_bwd(dy, h, gamma, mean, rstd, p: float, seed: int, offset: int, dres_in=None, dh=None, dx=None,
                          dgamma=None, dbeta=None, dbias=None, workspace=None):
    """Backward of lsq_bdr_layernorm_fwd -> (dh, dx, dgamma, dbeta, dbias)."""
    rows, hidden = h.shape
    dh = _native.empty_like(h) if dh is None else dh
    dx = _native.empty_like(h) if dx is None else dx
    mk = lambda t: _native.empty(h, torch.float32, hidden) if t is None else t
    dgamma, dbeta, dbias = mk(dgamma), mk(dbeta), mk(dbias)
    ws = _workspace(LSQ_OP_BDR_LAYERNORM_BWD, rows, hidden, h, workspace)
    _native.need("dy", dy, rows * hidden, h.dtype, "dh", dh, rows * hidden, h.dtype, "dx", dx, rows * hidden, h.dtype,
                  "dres_in", dres_in, rows * hidden, h.dtype, "gamma", gamma, hidden, h.dtype,
                  "mean", mean, rows, torch.float32, "rstd", rstd, rows, torch.float32,
                  "dgamma", dgamma, hidden, torch.float32, "dbeta", dbeta, hidden, torch.float32,
                  "dbias", dbias, hidden, torch.float32)
    _native.lsq_bdr_layernorm_bwd(dh, dx, dgamma, dbeta, dbias, dy, h, gamma, mean, rstd, dres_in, ws,
                                   ws.numel() * ws.element_size(), rows, hidden, p, seed, offset, h.dtype)
    return dh, dx, dgamma, dbeta, dbias


LSQ_ADAM_BLOCK = 8192


def lsq_adam_state_bytes(n: int) -> int:
    return int(load().lsq_adam_state_bytes(n))


def lsq_adam_state_pack(p, m=None, v=None, state=None):
    """fp32 p (and m, v; None = zeros) -> blocked optimizer state (fp32, lsq_adam_state_bytes(n) bytes)."""
    n = p.numel()
    need = lsq_adam_state_bytes(n) // 4
    state = _native.empty(p, torch.float32, need) if state is None else state
    _native.need("state", state, need, torch.float32, "p", p, n, torch.float32, "m", m, n, torch.float32,
                  "v", v, n, torch.float32)
    _native.lsq_adam_state_pack(state, p, m, v, n)
    return state


def lsq_adam_state_unpack(state, n: int, p=None, m=None, v=None, want=("p", "m", "v")):
    """Blocked optimizer state -> (p, m, v) fp32[n]; entries not in `want` (and not passed) come back as None."""
    p = _native.empty(state, torch.float32, n) if p is None and "p" in want else p
    m = _native.empty(state, torch.float32, n) if m is None and "m" in want else m
    v = _native.empty(state, torch.float32, n) if v is None and "v" in want else v
    _native.need("state", state, lsq_adam_state_bytes(n) // 4, torch.float32, "p", p, n, torch.float32,
                  "m", m, n, torch.float32, "v", v, n, torch.float32)
    _native.lsq_adam_state_unpack(p, m, v, state, n)
    return p, m, v


def lsq_adam_step_blocked(state, g, p_lp=None, *, lr: float, beta1: float, beta2: float, eps: float, step: int,
                          weight_decay: float = 0.0, adamw: bool = False, bias_correction: bool = True,
                          inv_grad_scale: float = 1.0):
    """lsq_adam_step on the blocked state (in place); g [n] low precision or fp32; p_lp optional copy out."""
    n = g.numel()
    _native.need("state", state, lsq_adam_state_bytes(n) // 4, torch.float32, "p_lp", p_lp, n, None)
    _native.lsq_adam_step_blocked(state, g, p_lp, n, lr, beta1, beta2, eps, weight_decay, step, int(adamw),
                                   int(bias_correction), inv_grad_scale, g.dtype, p_lp.dtype if p_lp is not None else LSQ_F16)
    return state, p_lp


def lsq_trainer_state_bytes(n: int, arrays: int) -> int:
    return int(load().lsq_trainer_state_bytes(n, arrays))


def lsq_trainer_state_pack(arrays_in, state=None):
    """List of 1..3 fp32 tensors [n] (entries after the first may be None = zeros) -> blocked state."""
    k = len(arrays_in)
    a0 = arrays_in[0]
    n = a0.numel()
    need = lsq_trainer_state_bytes(n, k) // 4
    state = _native.empty(a0, torch.float32, need) if state is None else state
    _native.need("state", state, need, torch.float32)
    for t in arrays_in:
        _native.need("array", t, n, torch.float32)
    a3 = [*arrays_in, None, None, None]
    _native.lsq_trainer_state_pack(state, a3[0], a3[1], a3[2], n, k)
    return state


def lsq_trainer_state_unpack(state, n: int, arrays: int):
    """Blocked state -> list of `arrays` fp32 tensors [n]."""
    _native.need("state", state, lsq_trainer_state_bytes(n, arrays) // 4, torch.float32)
    outs = [_native.empty(state, torch.float32, n) for _ in range(arrays)]
    a3 = [*outs, None, None, None]
    _native.lsq_trainer_state_unpack(a3[0], a3[1], a3[2], state, n, arrays)
    return outs


def lsq_sgd_step_blocked(state, g, p_lp=None, *, lr: float, momentum: float = 0.0, weight_decay: float = 0.0,
                         nesterov: bool = False, inv_grad_scale: float = 1.0):
    """lsq_sgd_step on the [p | momentum buffer] blocked state (in place)."""
    n = g.numel()
    _native.need("state", state, lsq_trainer_state_bytes(n, 2) // 4, torch.float32, "p_lp", p_lp, n, None)
    _native.lsq_sgd_step_blocked(state, g, p_lp, n, lr, momentum, weight_decay, int(nesterov), inv_grad_scale, g.dtype,
                                  p_lp.dtype if p_lp is not None else LSQ_F16)
    return state, p_lp


def lsq_adam_step_lp_blocked(p_lp, state, g, *, lr: float, beta1: float, beta2: float, eps: float, step: int,
                             weight_decay: float = 0.0, adamw: bool = False, bias_correction: bool = True,
                             inv_grad_scale: float = 1.0):
    """lsq_adam_step_lp with the moments in the [m | v] blocked state (p_lp and the state in place)."""
    if g.dtype != p_lp.dtype:
        raise LsqError("g and p_lp must share one low-precision dtype")
    n = p_lp.numel()
    _native.need("state", state, lsq_trainer_state_bytes(n, 2) // 4, torch.float32, "g", g, n, None)
    _native.lsq_adam_step_lp_blocked(p_lp, state, g, n, lr, beta1, beta2, eps, weight_decay, step, int(adamw),
                                      int(bias_correction), inv_grad_scale, p_lp.dtype)
    return p_lp, state


def lsq_pad_offsets(key_len, batch: int, max_len: int, offsets=None):
    """key_len: int32[batch] (or None: all full) -> offsets int32[batch+1] on the device."""
    if offsets is None:
        dev = key_len.device if key_len is not None else torch.device("cuda", torch.cuda.current_device())
        offsets = torch.empty(batch + 1, dtype=torch.int32, device=dev)
    _native.need("key_len", key_len, batch, torch.int32, "offsets", offsets, batch + 1, torch.int32)
    _native.lsq_pad_offsets(offsets, key_len, batch, max_len)
    return offsets


def lsq_pad_remove(padded, offsets, packed_rows: int, packed=None):
    """padded: [batch, max_len, hidden] -> packed [packed_rows, hidden] (rows from sum(len) on are not written)."""
    B, L, H = padded.shape
    packed = _native.empty(padded, None, packed_rows, H) if packed is None else packed
    _native.need("offsets", offsets, B + 1, torch.int32)
    if packed.dim() != 2 or packed.shape[1] != H or packed.dtype != padded.dtype:
        raise LsqError("packed must be [rows, hidden] of the padded tensor's dtype")
    _native.lsq_pad_remove(packed if packed.numel() else None, padded if padded.numel() else None, offsets, B, L, H,
                            packed.shape[0], padded.dtype)
    return packed


def lsq_pad_restore(packed, offsets, batch: int, max_len: int, padded=None):
    """packed: [rows, hidden] -> padded [batch, max_len, hidden], zeros on the padding."""
    H = packed.shape[1]
    padded = _native.empty(packed, None, batch, max_len, H) if padded is None else padded
    _native.need("offsets", offsets, batch + 1, torch.int32, "padded", padded, batch * max_len * H, packed.dtype)
    _native.lsq_pad_restore(padded if padded.numel() else None, packed if packed.numel() else None, offsets, batch, max_len,
                             H, packed.shape[0], packed.dtype)
    return padded


def lsq_softmax_varlen_fwd(x, key_len=None, query_len=None, causal: bool = False, scale: float = 1.0,
                           p_attn: float = 0.0, seed: int = 0, offset: int = 0, y=None, y_drop=None):
    """lsq_softmax_fwd with query_len: int32[batch]; rows of padded queries are not read and come out as zeros."""
    B, N, Lq, Lk = x.shape
    y = _native.empty_like(x) if y is None else y
    if p_attn > 0 and y_drop is None:
        y_drop = _native.empty_like(x)
    _native.need("y", y, x.numel(), x.dtype, "y_drop", y_drop, x.numel(), x.dtype, "key_len", key_len, B, torch.int32,
                  "query_len", query_len, B, torch.int32)
    _native.lsq_softmax_varlen_fwd(y, y_drop if p_attn > 0 else None, x, key_len, query_len, B, N, Lq, Lk, int(causal), scale,
                                    p_attn, seed, offset, x.dtype)
    return y, (y_drop if p_attn > 0 else None)


def lsq_softmax_varlen_bwd(dy, y, key_len=None, query_len=None, causal: bool = False, scale: float = 1.0,
                           p_attn: float = 0.0, seed: int = 0, offset: int = 0, dx=None):
    B, N, Lq, Lk = y.shape
    dx = _native.empty_like(y) if dx is None else dx
    _native.need("dx", dx, y.numel(), y.dtype, "dy", dy, y.numel(), y.dtype, "key_len", key_len, B, torch.int32,
                  "query_len", query_len, B, torch.int32)
    _native.lsq_softmax_varlen_bwd(dx, dy, y, key_len, query_len, B, N, Lq, Lk, int(causal), scale, p_attn, seed, offset,
                                    y.dtype)
    return dx


def lsq_calib_stream(kind: str, dst, src=None, nbytes: int = 0):
    """A plain memory stream (measurement aid): kind = "copy" | "read" | "write" | "empty"."""
    k = {"copy": 0, "read": 1, "write": 2, "empty": 3}[kind]
    _native.need("dst", dst, 0, None, "src", src, 0, None)       # tensors, not addresses
    _native.lsq_calib_stream(k, dst, src, nbytes)


def lsq_softmax_candidates(k_len: int) -> int:
    return int(load().lsq_softmax_candidates(k_len))


def lsq_softmax_tune(x, dy, key_len=None, query_len=None, causal: bool = False, scale: float = 1.0, p_attn: float = 0.0,
                     seed: int = 0, offset: int = 0, force: int = -1, reps: int = 20, y=None, y_drop=None, dx=None):
    """Search (force = -1), set (force >= 0) or forget (force = -2) the launch shape of the softmax for problems like
    this one -> (best_fwd, best_bwd, us[2][4])."""
    B, N, Lq, Lk = x.shape
    y = _native.empty_like(x) if y is None else y
    dx = _native.empty_like(x) if dx is None else dx
    if p_attn > 0 and y_drop is None:
        y_drop = _native.empty_like(x)
    bf, bb = C.c_int32(0), C.c_int32(0)
    us = (C.c_float * 8)()
    _check(load().lsq_softmax_tune(C.byref(bf), C.byref(bb), us, _ptr(y), _ptr(y_drop) if p_attn > 0 else None, _ptr(dx), _ptr(x),
                                   _ptr(dy), _ptr(key_len), _ptr(query_len), B, N, Lq, Lk, int(causal), scale, p_attn, seed, offset,
                                   _dt(x), force, reps, _stream()), "lsq_softmax_tune")
    return bf.value, bb.value, [[us[d * 4 + c] for c in range(4)] for d in range(2)]
