"""The binding's native calls against its Python path: the same results (an
explicit stream argument takes the Python path), the same objects where `out`
is given, and the same errors for arguments that are not the common form."""
import pytest
import torch

import paper_2608_26581_amd as rfq

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
