"""The binding's native calls against its Python path: the same results (an
explicit stream argument takes the Python path), the same objects where `out`
is given, and the same errors for arguments that are not the common form.
A failed launch is raised and the call not made a second time, and the
interpreter lock is released around the library."""
import ctypes

import pytest
import torch

import paper_2608_26581_amd as rfq
from paper_2608_26581_amd import rfq as binding

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


def _same(a, b):
    a, b = [x if isinstance(x, tuple) else (x,) for x in (a, b)]
    assert len(a) == len(b)
    for s, t in zip(a, b):
        assert (s is None) == (t is None)
        if s is not None:
            assert s.dtype == t.dtype and s.shape == t.shape and s.device == t.device
            assert torch.equal(s.view(torch.uint8), t.view(torch.uint8))


@pytest.mark.parametrize("M", [1, 40])
@pytest.mark.parametrize("residual", [True, False])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_native_calls_match_the_python_path(M, residual, dtype):
    N, K = 96, 2048
    s = torch.cuda.current_stream()
    gen = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((M, K), generator=gen, device="cuda").to(dtype)
    w = torch.randn((N, K), generator=gen, device="cuda")
    wq, hw = rfq.rfq_quantize_weight(w), rfq.rfq_hif4_quantize(w, residual=False)[:2]
    print("native calls M=%d %s" % (M, dtype), flush=True)

    def both(f, *args, **kw):
        a = f(*args, **kw)
        _same(a, f(*args, stream=s, **kw))
        return a

    q = both(rfq.rfq_quantize_act, x, residual=residual)
    h = both(rfq.rfq_hif4_quantize, x, residual=residual)
    both(rfq.rfq_gemm_stream, x, *wq, residual=residual, out_dtype=dtype)
    for split in (False, True):
        both(rfq.rfq_gemm, *q, *wq, out_dtype=dtype, split=split)
        both(rfq.rfq_hif4_gemm, *h, *hw, out_dtype=dtype, split=split)
    both(rfq.rfq_gemm_swiglu_quantize, *q, wq[0][:64], wq[1][:64], residual=residual)
    if residual:
        for rule in (0, 1):
            phi = both(rfq.rfq_fallback_map, q[2], q[1], rule, 127)
            both(rfq.rfq_gemm_phi, *q, *wq, phi, out_dtype=dtype)
        both(rfq.rfq_gemm_phi, *q, *wq, None, out_dtype=dtype)
    out = torch.empty((M, N), dtype=dtype, device="cuda")
    assert rfq.rfq_gemm(*q, *wq, out=out) is out
    _same(out, rfq.rfq_gemm(*q, *wq, out_dtype=dtype))
    # A subclass goes through the Python path.
    _same(rfq.rfq_gemm(q[0].as_subclass(Sub), *q[1:], *wq, out_dtype=dtype), out)


def test_native_calls_refuse_what_the_python_path_refuses():
    x = torch.randn(8, 512, device="cuda")
    q, w = rfq.rfq_quantize_act(x), rfq.rfq_quantize_weight(torch.randn(32, 512, device="cuda"))
    for bad, err in (((q[0].cpu(), *q[1:], *w), ValueError), ((*q[:3], None, *w), ValueError),
                     ((*q, w[0], w[1][:, :8]), ValueError), ((*q, w[0].int(), w[1]), TypeError),
                     ((q[0][:, ::2], *q[1:], *w), ValueError)):
        with pytest.raises(err):
            rfq.rfq_gemm(*bad)
    with pytest.raises(TypeError):
        rfq.rfq_gemm(*q, *w, out_dtype=torch.float16)
    with pytest.raises(ValueError):
        rfq.rfq_gemm(*q, *w, out=torch.empty(8, 31, device="cuda"))
    with pytest.raises(rfq.RfqError):
        rfq.rfq_gemm_stream(x[:, :480].contiguous(), w[0][:, :240].contiguous(),
                            w[1][:, :15].contiguous())
    with pytest.raises(rfq.RfqError):
        rfq.rfq_quantize_act(x[:, :40].contiguous())
    with pytest.raises(TypeError):
        rfq.rfq_quantize_act(x.half())


def _operands():
    x = torch.randn(40, 2048, device="cuda")
    w = torch.randn(96, 2048, device="cuda")
    return (x, rfq.rfq_quantize_act(x), rfq.rfq_quantize_weight(w), rfq.rfq_hif4_quantize(x),
            rfq.rfq_hif4_quantize(w, residual=False)[:2])


def _common_forms(wrap=lambda t: t, **kw):
    """name in the native module -> a call of the binding in that form, with
    every tensor passed through wrap."""
    x, q, w, h, hw = _operands()
    phi = rfq.rfq_fallback_map(q[2], q[1], 0)
    x, phi = wrap(x), wrap(phi)
    q, w, h, hw = (tuple(map(wrap, t)) for t in (q, w, h, hw))
    return {
        "quantize_act": lambda: rfq.rfq_quantize_act(x, **kw),
        "hif4_quantize": lambda: rfq.rfq_hif4_quantize(x, **kw),
        "gemm": lambda: rfq.rfq_gemm(*q, *w, **kw),
        "gemm, split": lambda: rfq.rfq_gemm(*q, *w, split=True, **kw),
        "hif4_gemm": lambda: rfq.rfq_hif4_gemm(*h, *hw, **kw),
        "hif4_gemm, split": lambda: rfq.rfq_hif4_gemm(*h, *hw, split=True, **kw),
        "gemm_stream": lambda: rfq.rfq_gemm_stream(x, *w, **kw),
        "gemm_phi": lambda: rfq.rfq_gemm_phi(*q, *w, phi, **kw),
        "fallback_map": lambda: rfq.rfq_fallback_map(q[2], q[1], 0, **kw),
        "gemm_swiglu_quantize": lambda: rfq.rfq_gemm_swiglu_quantize(*q, w[0][:64], w[1][:64], **kw),
    }


def _native_result(monkeypatch, call):
    """What the native call returns to the binding."""
    class Done(Exception):
        pass

    got = []

    def native(func, *args):
        got.append(getattr(binding._calls, func)(*args))
        raise Done

    with monkeypatch.context() as m:
        m.setattr(binding, "_native", native)
        with pytest.raises(Done):
            call()
    return got[0]


def test_the_common_forms_are_served_natively(monkeypatch):
    """Every common form gets its result from the native call, also on another
    stream: with nothing native the binding would still answer, in Python."""
    torch.manual_seed(7)
    forms = _common_forms()
    torch.manual_seed(7)
    python = _common_forms(stream=torch.cuda.current_stream())
    side = torch.cuda.Stream()
    for name, call in forms.items():
        r = _native_result(monkeypatch, call)
        assert r is not None, name
        _same(r, python[name]())
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            s = _native_result(monkeypatch, call)
        torch.cuda.current_stream().wait_stream(side)
        _same(s, r)


@pytest.mark.parametrize("wrap", [lambda t: t.as_subclass(Sub), lambda t: t.cpu(),
                                  lambda t: t[:, :-1], lambda t: t.float() if t.dtype in (
                                      torch.uint8, torch.int32) else t.half()],
                         ids=["subclass", "cpu", "narrowed", "dtype"])
def test_other_forms_are_left_to_the_python_path(monkeypatch, wrap):
    for name, call in _common_forms(wrap).items():
        assert _native_result(monkeypatch, call) is None, name


def _bind_stub(stub):
    """Points the native calls at stub, except for the workspace sizes."""
    lib = binding.load()
    address = ctypes.cast(stub, ctypes.c_void_p).value
    binding._calls.bind(*(
        ctypes.cast(getattr(lib, f), ctypes.c_void_p).value if f.endswith("_bytes") else address
        for f in binding._NATIVE_ENTRIES))


def test_a_failed_launch_is_raised_and_the_call_not_repeated(monkeypatch):
    launches = []
    stub = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: launches.append(1) or 6)   # RFQ_ERR_LAUNCH
    forms, lib = _common_forms(), binding.load()

    class StatusNamesOnly:
        rfq_status_str = lib.rfq_status_str
        rfq_gemm_workspace_bytes = lib.rfq_gemm_workspace_bytes
        rfq_hif4_gemm_workspace_bytes = lib.rfq_hif4_gemm_workspace_bytes

        def __getattr__(self, name):
            raise AssertionError("%s called after the failed launch" % name)

    monkeypatch.setattr(binding, "_lib", StatusNamesOnly())
    _bind_stub(stub)
    try:
        for name, call in forms.items():
            launches.clear()
            with pytest.raises(rfq.RfqError, match="RFQ_ERR_LAUNCH") as e:
                call()
            assert e.value.status == 6 and len(launches) == 1, name
    finally:
        binding._bind_calls(lib)


def test_the_interpreter_lock_is_released_around_the_library(monkeypatch):
    """The library's entry points stand for PyGILState_Check here: it returns 1
    (an argument error to the native call, which then gives None) where the
    thread holds the lock and 0 (done: the result) where it does not."""
    forms, lib = _common_forms(), binding.load()
    _bind_stub(ctypes.pythonapi.PyGILState_Check)
    try:
        for name, call in forms.items():
            assert _native_result(monkeypatch, call) is not None, name
    finally:
        binding._bind_calls(lib)
