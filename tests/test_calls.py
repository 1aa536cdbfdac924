"""The native half of the binding (csrc/calls.cpp) against the general Python forms that it stands in for, on the CPU: what they
accept it accepts, what they refuse it refuses with the same error."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2110_05722_amd as L
from paper_2110_05722_amd import binding

A = 4096          # aligned, never dereferenced: every call below fails before a launch


class Sub(torch.Tensor):
    pass


def outcome(f):
    try:
        r = f()
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)
    return r


TENSORS = {"f16": torch.zeros(12, dtype=torch.float16), "f32": torch.zeros(3, 4), "param": torch.nn.Parameter(torch.zeros(12)),
           "sub": torch.zeros(12).as_subclass(Sub), "strided": torch.zeros(4, 6).t(), "none": None, "not one": 3.0, "empty": torch.zeros(0),
           "wide stride": torch.zeros(12, 50)[:1, :12], "odd stride of one": torch.zeros(12).as_strided((1, 12), (50, 1)),
           "flat": torch.zeros(12).expand(3, 12), "pixels": torch.zeros(2, 3, 4, 5).to(memory_format=torch.channels_last), "scalar": torch.zeros(()),
           "none in": torch.zeros(3, 0, 2)}


@pytest.mark.parametrize("numel", [0, 12, 13, -1, 1 << 70, np.int64(12)])
@pytest.mark.parametrize("dtype", [None, torch.float16, torch.float32])
@pytest.mark.parametrize("name", TENSORS)
def test_need_says_what_the_python_form_says(name, dtype, numel):
    t = TENSORS[name]
    assert outcome(lambda: binding._native.need("t", t, numel, dtype)) == outcome(lambda: binding._need("t", t, numel, dtype))
    # the same as the second of two
    good = ("g", TENSORS["f32"], 12, torch.float32)
    assert outcome(lambda: binding._native.need(*good, "t", t, numel, dtype)) == outcome(lambda: binding._need("t", t, numel, dtype))


@pytest.mark.parametrize("sizes", [(), (0,), (7,), (2, 3), (2, 0, 3, 4), (-1,), (np.int64(5), 2), (1, 1, 1, 1, 1, 1), (2.0,)])
@pytest.mark.parametrize("name", ["f16", "param", "sub", "strided"])
def test_empty_is_torch_empty(name, sizes):
    like = TENSORS[name]
    for dtype in (None, torch.uint8):
        a, b = outcome(lambda: binding._native.empty(like, dtype, *sizes)), outcome(lambda: binding._empty(like, dtype, *sizes))
        if torch.is_tensor(b):
            assert (type(a), a.shape, a.dtype, a.device, a.stride(), a.requires_grad) == (type(b), b.shape, b.dtype, b.device, b.stride(), b.requires_grad)
        else:
            assert a == b


@pytest.mark.parametrize("name", [n for n in TENSORS if n != "none"])
def test_empty_like_is_torch_empty_like(name):
    t = TENSORS[name]
    a, b = outcome(lambda: binding._native.empty_like(t)), outcome(lambda: torch.empty_like(t))
    if torch.is_tensor(b):
        assert (type(a), a.shape, a.dtype, a.stride(), a.requires_grad) == (type(b), b.shape, b.dtype, b.stride(), b.requires_grad)
    else:
        assert a == b


def test_a_function_mode_sees_the_allocations():
    class Seen(torch.overrides.TorchFunctionMode):
        names = []

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.names.append(func.__name__)
            return func(*args, **(kwargs or {}))

    with Seen() as seen:
        binding._native.empty(TENSORS["f32"], None, 3)
        binding._native.empty_like(TENSORS["f32"])
    assert "empty" in seen.names and "empty_like" in seen.names


# (arguments of lsq_layernorm_fwd without the stream, ctypes status or what is raised)
LN = [A, A, A, A, A, A, 4, 8, 1e-5, 0]


def _ln(i, v):
    a = list(LN)
    a[i] = v
    return a


@pytest.mark.parametrize("args", [_ln(7, 0), _ln(8, -1.0), _ln(3, A + 2), _ln(9, 5), _ln(3, None), _ln(6, 4.0), _ln(6, "4"), _ln(8, "x"),
                                  _ln(6, None), _ln(7, (1 << 32) + 0), _ln(7, np.int32(0)), _ln(6, torch.tensor(-1)), _ln(7, False), _ln(8, -1)])
def test_numbers_convert_as_ctypes_converts_them(monkeypatch, args):
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    want = outcome(lambda: L.load().lsq_layernorm_fwd(*args, 0))
    got = outcome(lambda: binding._native.lsq_layernorm_fwd(*args))
    if isinstance(want, int):
        assert got == (L.LsqError, f"lsq_layernorm_fwd failed: {L.lsq_status_string(want)}") and want != 0
    else:
        assert got[0] is want[0] is C.ArgumentError


def test_tensors_and_dtypes_are_refused_in_order(monkeypatch):
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    f = binding._native.lsq_layernorm_fwd
    for t in (TENSORS["f32"], TENSORS["sub"], TENSORS["param"]):
        assert outcome(lambda: f(*_ln(3, t)[:9], torch.float64)) == (L.LsqError, "tensors must live on the GPU (there is no CPU path)")
    assert outcome(lambda: f(*LN[:9], torch.float64)) == (L.LsqError, "unsupported dtype torch.float64")
    assert outcome(lambda: f(*_ln(7, 0)[:9], torch.bfloat16)) == (L.LsqError, "lsq_layernorm_fwd failed: LSQ_INVALID_ARG")
    assert outcome(lambda: f(*LN[:-1]))[0] is TypeError
    # the stream is asked for last: what is wrong with the arguments is said first
    monkeypatch.setattr(binding, "_stream", lambda: 1 / 0)
    assert outcome(lambda: f(*_ln(3, TENSORS["f32"])))[0] is L.LsqError
    assert outcome(lambda: f(*_ln(7, 0)))[0] is ZeroDivisionError


def test_every_entry_point_with_a_stream_has_its_native_call():
    assert binding._native.need() is None            # loads the extension
    for name in binding.EXPORTS:
        takes_stream = name not in ("lsq_workspace_bytes", "lsq_status_string", "lsq_adam_state_bytes", "lsq_trainer_state_bytes",
                                    "lsq_softmax_candidates", "lsq_softmax_tune")
        assert hasattr(binding._native, name) == takes_stream, name


@pytest.mark.gpu
def test_on_the_gpu_parameters_and_subclasses_are_tensors_like_any_other():
    x = torch.randn(9, 64, device="cuda")
    g, b = torch.rand(64, device="cuda"), torch.rand(64, device="cuda")
    want = L.lsq_layernorm_fwd(x, g, b)
    for gg, xx in ((torch.nn.Parameter(g), x), (g.as_subclass(Sub), x.as_subclass(Sub))):
        got = L.lsq_layernorm_fwd(xx, gg, b)
        assert all(torch.equal(torch.Tensor(p), q) for p, q in zip(got, want)) and type(got[0]) is type(torch.empty_like(xx))
    with pytest.raises(L.LsqError, match="must be contiguous"):
        L.lsq_layernorm_fwd(torch.randn(64, 9, device="cuda").t(), g, b)
    with pytest.raises(L.LsqError, match="unsupported dtype torch.float64"):
        L.lsq_layernorm_fwd(x.double(), g.double(), b.double())


def test_an_extension_of_another_torch_or_python_is_refused(monkeypatch):
    """It is built against torch's own headers: what another interpreter or torch would load is refused, before anything in it is used."""
    import sysconfig
    assert binding._CALLS_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert binding._native.need() is None
    loaded = binding._native
    monkeypatch.setattr(binding, "_native", binding._Native())
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "1.0.0")
        with pytest.raises(L.LsqError, match="built for torch .* this is 1.0.0"):
            binding._native.need()
    with monkeypatch.context() as m:
        m.setattr(binding, "_CALLS_PATH", binding._CALLS_PATH + ".absent")
        with pytest.raises(L.LsqError, match="is missing"):
            binding._native.need()
    assert binding._native.need() is None and binding._native is loaded


def test_addresses_are_not_tensors():
    """No wrapper takes a bare address in a tensor's place (None in a position that may be empty is another matter)."""
    for args in (("copy", A, None, 16), ("read", None, A, 16), ("write", True, None, 16)):
        assert outcome(lambda: L.lsq_calib_stream(*args))[0] is AttributeError
    t = torch.zeros(4, 8)
    for call in (lambda: L.lsq_layernorm_fwd(t, A, t[0]), lambda: L.lsq_bias_dropout_residual_fwd(t, None, A, 0.0, 1, 1), lambda: L.lsq_merge_heads_fwd(A),
                 lambda: L.lsq_adam_step(A, t, t, t, lr=1e-3, beta1=0.9, beta2=0.9, eps=1e-8, step=1), lambda: L.lsq_embedding_fwd(A, t, t, 0, 1.0, 0.0, 1, 1),
                 lambda: L.lsq_pad_remove(t.view(1, 4, 8), A, 2), lambda: L.lsq_ls_xent_fwd(t, A, 0.1), lambda: L.lsq_softmax_fwd(t.view(1, 1, 4, 8), key_len=A)):
        assert outcome(call)[0] is AttributeError
