"""The general product kernel, which serves scale tensors that are not 16-byte
aligned (and code tensors past the other kernels' sizes): with and without the
residual, both output types, fallback maps and the scale bytes' range, every
operand's scales one byte past an aligned address."""
import numpy as np
import pytest
import torch

import paper_2608_26581_amd as rfq
from gpu_util import assert_gemm_close, dev, host, host_bf16_as_f32
from oracle_pins import SWEEP_SCALE_BYTES, scale_sweep_blocks

pytestmark = pytest.mark.gpu

# One block; K below, at and past a stage of 256, ragged; a single tile row and
# ragged tiles; K a multiple of 256 (scales 8 bytes at a time when aligned).
SHAPES = [(1, 5, 32), (64, 96, 640), (129, 257, 512), (200, 328, 1056), (300, 130, 2592)]


def _shifted(t):
    if t is None:
        return None
    raw = torch.empty(t.numel() + 1, dtype=torch.uint8, device="cuda")
    v = raw[1:].view(t.shape)
    v.copy_(t)
    return v


def _operands(M, N, K):
    rng = np.random.default_rng(M + N + K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, ::max(7, K // 5)] *= 50
    w = rng.normal(0, 0.02, (N, K)).astype(np.float32)
    q, w = rfq.rfq_quantize_act(dev(x)), rfq.rfq_quantize_weight(dev(w))
    return (q[0], _shifted(q[1]), q[2], _shifted(q[3])), (w[0], _shifted(w[1]))


def _values(z):
    return host_bf16_as_f32(z) if z.dtype == torch.bfloat16 else host(z)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("residual", [True, False])
def test_product(orc, M, N, K, dtype, residual):
    q, w = _operands(M, N, K)
    q = q if residual else (*q[:2], None, None)
    print("general kernel: M=%d N=%d K=%d %s residual=%s" % (M, N, K, dtype, residual), flush=True)
    z = rfq.rfq_gemm(*q, *w, out_dtype=dtype)
    zr, bound = orc.gemm(*[None if t is None else host(t) for t in (*q, *w)])
    assert_gemm_close(_values(z), zr, bound, dtype == torch.bfloat16, "product")
    # With a workspace too: these operands run unsplit.
    assert torch.equal(rfq.rfq_gemm(*q, *w, out_dtype=dtype, split=True), z)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_maps(orc, M, N, K, dtype):
    q, w = _operands(M, N, K)
    shape = ((M + 63) // 64, (K + 255) // 256)
    rng = np.random.default_rng(K)
    print("general kernel, maps: M=%d N=%d K=%d %s" % (M, N, K, dtype), flush=True)
    for phi in [(rng.random(shape) < p).astype(np.uint8) for p in (0.25, 0.75)] + [
            rng.integers(0, 256, shape).astype(np.uint8)]:
        z = rfq.rfq_gemm_phi(*q, *w, dev(phi), out_dtype=dtype)
        zr, bound = orc.gemm_phi(*[host(t) for t in (*q, *w)], phi)
        assert_gemm_close(_values(z), zr, bound, dtype == torch.bfloat16, "map")
    for fill, ops in ((1, q), (0, (*q[:2], None, None))):
        phi = torch.full(shape, fill, dtype=torch.uint8, device="cuda")
        assert torch.equal(rfq.rfq_gemm_phi(*q, *w, phi, out_dtype=dtype),
                           rfq.rfq_gemm(*ops, *w, out_dtype=dtype))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_scale_bytes(orc, dtype):
    """Products of blocks whose scale bytes span the range (see the sweep through
    the converters): rows that stay far from fp32's underflow and overflow."""
    x = scale_sweep_blocks(dtype == torch.bfloat16)
    q = rfq.rfq_quantize_act(torch.from_numpy(x.astype(np.float32)).cuda().to(dtype))
    q = (q[0], _shifted(q[1]), q[2], _shifted(q[3]))
    row_bytes = np.array(list(SWEEP_SCALE_BYTES) + [0])
    rng = np.random.default_rng(31)
    for j in (100, 0, -100):
        wv = (rng.standard_normal((96, x.shape[1])) * 2.0 ** j).astype(np.float32)
        w = rfq.rfq_quantize_weight(dev(wv))
        w = (w[0], _shifted(w[1]))
        print("general kernel, scale bytes: j=%d %s" % (j, dtype), flush=True)
        for out_dtype in (torch.float32, torch.bfloat16):
            z = rfq.rfq_gemm(*q, *w, out_dtype=out_dtype)
            zr, bound = orc.gemm(*[host(t) for t in (*q, *w)])
            ok = np.abs(row_bytes - 127 + j) <= 100
            assert_gemm_close(_values(z)[ok], zr[ok], bound[ok], out_dtype == torch.bfloat16,
                              "scale bytes j=%d" % j)
