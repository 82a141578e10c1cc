"""Where a product's store width or kernel changes with its sizes: the results on
both sides of the line."""
import numpy as np
import pytest
import torch

import paper_2608_26581_amd as rfq
from gpu_util import assert_gemm_close, host

pytestmark = pytest.mark.gpu


def _mx(M, N, K, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed + M + N + K)
    x = torch.randn((M, K), generator=gen, device="cuda")
    x[:, ::37] *= 40
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    return rfq.rfq_quantize_act(x), rfq.rfq_quantize_weight(w)


def _guarded(M, N, dtype):
    """An [M][N] tensor and a check that the 256 bytes on either side of it
    stayed as they were."""
    n = M * N * (2 if dtype == torch.bfloat16 else 4)
    raw = torch.full((n + 512,), 0x5A, dtype=torch.uint8, device="cuda")
    return raw[256:256 + n].view(dtype).view(M, N), lambda: bool(
        (raw[:256] == 0x5A).all() and (raw[256 + n:] == 0x5A).all())


# Columns 4 past a multiple of 8: bf16 rows start at 8 bytes and are stored 8
# bytes at a time.  128 x 128 tiles (at most one per CU, and more), 256 x 128,
# 256 x 256; a last column tile of 4 columns, and of all but 4.
@pytest.mark.parametrize("M,N,K", [(129, 132, 96), (130, 252, 512), (2100, 2180, 512),
                                   (300, 12300, 1024), (2900, 2820, 64), (2900, 2812, 608)])
@pytest.mark.parametrize("residual", [True, False])
def test_bf16_rows_of_4_past_a_multiple_of_8(M, N, K, residual):
    q, w = _mx(M, N, K)
    q = q if residual else (q[0], q[1], None, None)
    print("bf16 rows at 8 bytes: M=%d N=%d K=%d" % (M, N, K), flush=True)
    z, intact = _guarded(M, N, torch.bfloat16)
    rfq.rfq_gemm(*q, *w, out=z)
    # The same sums in fp32, rounded by torch.
    assert torch.equal(z, rfq.rfq_gemm(*q, *w).bfloat16())
    assert intact()


# fp32 rows of whole and of broken 16-byte chunks, on each tile shape.
@pytest.mark.parametrize("M,N,K", [(129, 132, 96), (129, 131, 96), (130, 253, 512), (2100, 2180, 512),
                                   (2100, 2179, 512), (300, 12300, 1024), (300, 12301, 2048),
                                   (2900, 2820, 64), (2900, 2822, 608)])
@pytest.mark.parametrize("residual", [True, False])
def test_fp32_rows(M, N, K, residual):
    q, w = _mx(M, N, K)
    q = q if residual else (q[0], q[1], None, None)
    print("fp32 rows: M=%d N=%d K=%d" % (M, N, K), flush=True)
    z, intact = _guarded(M, N, torch.float32)
    rfq.rfq_gemm(*q, *w, out=z)
    # The same sums, which the bf16 store rounds.
    assert torch.equal(z.bfloat16(), rfq.rfq_gemm(*q, *w, out_dtype=torch.bfloat16))
    assert intact()


# 256 x 128 tiles from K = 1024 (SwiGLU epilogue: 2048, plain 1536; rows of Z
# that do not start at 16 bytes: 2048; up to 192 rows: 512), 128 x 128 below.
@pytest.mark.parametrize("M,N,K", [(300, 12300, 992), (300, 12300, 1024), (520, 7200, 512),
                                   (300, 12301, 1024), (300, 12301, 2016), (300, 12301, 2048),
                                   (192, 16500, 480), (192, 16500, 512), (193, 16500, 512),
                                   (256, 16501, 1024)])
def test_tall_tiles_from_their_shortest_k(orc, M, N, K):
    q, w = _mx(M, N, K)
    print("tall tiles: M=%d N=%d K=%d" % (M, N, K), flush=True)
    z = host(rfq.rfq_gemm(*q, *w))
    rows = np.unique(np.r_[0:4, 255:258, M - 3:M, 130:M:29].clip(0, M - 1))
    zr, bound = orc.gemm(*[host(t)[rows] for t in q], host(w[0]), host(w[1]))
    assert_gemm_close(z[rows], zr, bound, False, "product")
    ones = torch.ones(((M + 63) // 64, (K + 255) // 256), dtype=torch.uint8, device="cuda")
    assert np.array_equal(host(rfq.rfq_gemm_phi(*q, *w, ones)), z)
    zb, intact = _guarded(M, N, torch.bfloat16)
    rfq.rfq_gemm(*q, *w, out=zb)
    assert torch.equal(zb, torch.from_numpy(z).cuda().bfloat16()) and intact()
    assert torch.equal(rfq.rfq_gemm_phi(*q, *w, ones, out_dtype=torch.bfloat16), zb)


@pytest.mark.parametrize("K,residual", [(1536, True), (2048, True), (1024, False), (1536, False)])
def test_tall_swiglu_tiles_from_their_shortest_k(K, residual):
    """The same codes as the chain of product and SwiGLU quantizer."""
    M, Nh = 300, 6144
    q, w = _mx(M, 2 * Nh, K)
    q = q if residual else (q[0], q[1], None, None)
    print("tall SwiGLU tiles: K=%d" % K, flush=True)
    got = rfq.rfq_gemm_swiglu_quantize(*q, *w)
    gu = rfq.rfq_gemm(*q, *w, out_dtype=torch.bfloat16).view(M, Nh // 32, 2, 32)
    g, u = (gu[:, :, i].reshape(M, Nh).contiguous() for i in (0, 1))
    want = rfq.rfq_swiglu_quantize_act(g, u)
    for a, b in zip(got[:4], want[:4]):
        assert torch.equal(a, b)


# K of up to eight stages: one stage in registers or two (with the residual two
# from K = 544 and 65 tiles, K = 1056), and from 1024 tiles 128 x 128 ones up to K = 256.
@pytest.mark.parametrize("M,N,K", [(497, 704, 480), (497, 704, 512), (2048, 1024, 512),
                                   (2049, 1024, 512), (1024, 1024, 544), (1025, 1024, 544),
                                   (300, 500, 1024), (300, 500, 1056), (4000, 4130, 256), (4205, 4204, 256),
                                   (4205, 4204, 288), (8200, 2050, 32)])
@pytest.mark.parametrize("residual", [True, False])
def test_short_k_tiles(M, N, K, residual):
    """The bits of the same rows in blocks of 256, whose tiles are few."""
    q, w = _mx(M, N, K)
    q = q if residual else (q[0], q[1], None, None)
    print("short K: M=%d N=%d K=%d" % (M, N, K), flush=True)
    phi = (torch.arange((M + 63) // 64, device="cuda") % 3 != 0).to(torch.uint8)
    phi = phi[:, None].expand(-1, (K + 255) // 256).contiguous()
    calls = [lambda q, phi, **kw: rfq.rfq_gemm(*q, *w, **kw)]
    if residual:
        calls.append(lambda q, phi, **kw: rfq.rfq_gemm_phi(*q, *w, phi, **kw))
    for call in calls:
        for dt in (torch.float32, torch.bfloat16):
            z, intact = _guarded(M, N, dt)
            call(q, phi, out=z)
            for r in range(0, M, 256):
                qr = [None if t is None else t[r:r + 256].clone() for t in q]
                assert torch.equal(z[r:r + 256], call(qr, phi[r // 64:r // 64 + 4].clone(),
                                                      out_dtype=dt))
            assert intact()


# Ragged K, 33 to 64 rows: the few-row kernel below N = 16384, 128-wide tiles from
# there (to K = 2048).
@pytest.mark.parametrize("M,N,K", [(32, 16390, 96), (33, 16380, 96), (33, 16384, 96),
                                   (64, 16390, 416), (50, 16388, 2016), (50, 16388, 2080)])
@pytest.mark.parametrize("residual", [True, False])
def test_few_rows_wide_at_ragged_k(orc, M, N, K, residual):
    q, w = _mx(M, N, K)
    q = q if residual else (q[0], q[1], None, None)
    print("few rows, ragged K: M=%d N=%d K=%d" % (M, N, K), flush=True)
    z, intact = _guarded(M, N, torch.float32)
    rfq.rfq_gemm(*q, *w, out=z)
    rows = np.unique(np.r_[0:3, 30:33, M - 2:M].clip(0, M - 1))
    zr, bound = orc.gemm(*[None if t is None else host(t)[rows] for t in q], host(w[0]),
                         host(w[1]))
    assert_gemm_close(host(z)[rows], zr, bound, False, "product")
    assert intact()
    zb = rfq.rfq_gemm(*q, *w, out_dtype=torch.bfloat16, split=True)
    assert torch.equal(zb, z.bfloat16())
    if residual:
        ones = torch.ones((1, (K + 255) // 256), dtype=torch.uint8, device="cuda")
        assert torch.equal(rfq.rfq_gemm_phi(*q, *w, ones), z)


# Splits above 128 rows at short K: parts of 512 and of 1024 columns, the
# residual split and the plain product not, and ragged K.
@pytest.mark.parametrize("M,N,K", [(213, 512, 3584), (256, 576, 4096), (150, 200, 2848),
                                   (1130, 200, 4096), (256, 1344, 3072), (285, 1410, 3072),
                                   (167, 384, 1536), (331, 41, 1152), (521, 192, 1920)])
@pytest.mark.parametrize("residual", [True, False])
def test_split_at_short_k(orc, M, N, K, residual):
    q, w = _mx(M, N, K)
    q = q if residual else (q[0], q[1], None, None)
    print("split at short K: M=%d N=%d K=%d" % (M, N, K), flush=True)
    z, intact = _guarded(M, N, torch.float32)
    rfq.rfq_gemm(*q, *w, out=z, split=True)
    rows = np.unique(np.r_[0:4, M - 3:M, 0:M:17])
    zr, bound = orc.gemm(*[None if t is None else host(t)[rows] for t in q], host(w[0]),
                         host(w[1]))
    assert_gemm_close(host(z)[rows], zr, bound, False, "split")
    assert intact()


def _hif4(M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    x = torch.randn((M, K), generator=gen, device="cuda")
    x[:, ::37] *= 40
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    return rfq.rfq_hif4_quantize(x), rfq.rfq_hif4_quantize(w, residual=False)[:2]


# 128-wide tiles: 258, 260 and 510 of them (two workgroups of the plain product
# per CU on codes below K = 1024, on bf16 weights at every K), and 256 (one).
@pytest.mark.parametrize("M,N,K", [(300, 10950, 64), (1290, 3260, 128), (1921, 4301, 192),
                                   (1290, 3260, 960), (1290, 3260, 1024), (1000, 4096, 128)])
def test_hif4_plain_tiles_two_per_cu(M, N, K):
    """The bits of the same rows in blocks of 150, whose tiles run one per CU."""
    q, w = _hif4(M, N, K)
    wv = rfq.rfq_hif4_dequant(*w, out_dtype=torch.bfloat16)
    print("HiF4 plain tiles: M=%d N=%d K=%d" % (M, N, K), flush=True)
    for dt in (torch.float32, torch.bfloat16):
        z, intact = _guarded(M, N, dt)
        rfq.rfq_hif4_gemm(q[0], q[1], None, None, *w, out=z)
        want = torch.cat([rfq.rfq_hif4_gemm(q[0][r:r + 150], q[1][r:r + 150], None, None, *w,
                                            out_dtype=dt) for r in range(0, M // 150 * 150, 150)])
        assert torch.equal(z[:len(want)], want) and intact()
        zb, intact = _guarded(M, N, dt)
        rfq.rfq_hif4_gemm_wbf16(q[0], q[1], None, None, wv, out=zb)
        assert torch.equal(zb, z) and intact()


# Both sides of where W is decoded into the workspace: 256 tiles of 128 x 128 (not)
# and 257 or more; the plain product with K = 512 (not) and 576, below N =
# 2048 320 (not) and 384, up to 256 tiles of 128 x 256; N not a multiple of 32 (row by row, with the
# residual from K = 8192 and 2048 rows at fewer tiles too).
@pytest.mark.parametrize("M,N,K", [(1024, 4096, 192), (1025, 4064, 192), (1300, 4224, 512),
                                   (1300, 4224, 576), (1025, 4100, 512), (1025, 4100, 576),
                                   (4100, 4096, 192), (3600, 1184, 320), (3600, 1184, 384),
                                   (2100, 1250, 8128), (2047, 1250, 8192), (2100, 1250, 8192),
                                   (2100, 1248, 8192)])
@pytest.mark.parametrize("residual", [True, False])
def test_hif4_decoded_weights_from_their_smallest_sizes(M, N, K, residual):
    q, w = _hif4(M, N, K)
    q = q if residual else (q[0], q[1], None, None)
    nbytes = rfq.rfq_hif4_gemm_workspace_bytes(M, N, K)
    assert nbytes == N * K * 2
    print("HiF4 decoded weights: M=%d N=%d K=%d" % (M, N, K), flush=True)
    ws = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    z, intact = _guarded(M, N, torch.float32)
    rfq.rfq_hif4_gemm_split(*q, *w, ws[:nbytes], out=z)
    assert torch.equal(z, rfq.rfq_hif4_gemm(*q, *w)) and intact()
    assert (ws[nbytes:] == 0x5A).all()
    # The line lies where the comments say: the workspace is written or not.
    tiles, wide = -(-M // 128) * -(-N // 128), -(-M // 128) * -(-N // 256)
    used = tiles > 256 and (residual or K >= (384 if N < 2048 else 576) or wide >= 256)
    used |= tiles <= 256 and residual and N % 32 != 0 and K >= 8192 and M >= 2048
    assert bool((ws[:nbytes] != 0x5A).any()) == used


# The HiF4 quantizer: four units a lane from 2^25 elements (with the residual 2^27;
# fp32 without it one at every size), several launches past 2^31 elements.
@pytest.mark.parametrize("M,dtype,residual", [
    (8191, torch.bfloat16, False), (8193, torch.bfloat16, False), (8193, torch.float32, False),
    (32769, torch.bfloat16, True), (32769, torch.float32, True),
    ((1 << 19) + 3, torch.bfloat16, True), ((1 << 19) + 3, torch.float32, False)])
def test_hif4_quantizer_units_and_launches(M, dtype, residual):
    """The codes of blocks of 4096 rows, which a lane a unit quantizes in one
    launch."""
    K = 4096
    print("HiF4 quantizer: M=%d %s residual=%s" % (M, dtype, residual), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M)
    x = torch.empty((M, K), dtype=dtype, device="cuda")
    for r in range(0, M, 4096):
        x[r:r + 4096] = torch.randn((min(4096, M - r), K), generator=gen, device="cuda")
    q = rfq.rfq_hif4_quantize(x, residual=residual)
    for r in range(0, M, 4096):
        want = rfq.rfq_hif4_quantize(x[r:r + 4096], residual=residual)
        for a, b in zip(q, want):
            assert (a is None) == (b is None) and (a is None or torch.equal(a[r:r + 4096], b))
