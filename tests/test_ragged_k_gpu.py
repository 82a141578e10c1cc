"""Products whose K is a multiple of 32 but not of 512: the few-row, 128-wide,
256-wide, split and fallback-map kernels take their last group or stage short
and read scale rows that start at any byte.  Against the oracle within the
product's tolerance (gpu_util); the general kernel, which takes scale tensors
that are not 16-byte aligned, gives the same products."""
import numpy as np
import pytest
import torch

import paper_2608_26581_amd as rfq
from gpu_util import assert_gemm_close, dev, host, host_bf16_as_f32

pytestmark = pytest.mark.gpu

# K / 32 blocks: 1 to 4 in the last stage of 4, scale rows that start at every
# byte of a dword, 1 to 4 stages in the last group of 4.
SHAPES = [
    (1, 40, 32),             # few rows: a single block
    (5, 300, 544),           # 17 blocks: one past a whole group
    (16, 70, 1504),          # 47 blocks
    (40, 130, 2016),         # 63 blocks, three slices
    (100, 260, 992),         # two workgroup rows
    (7, 12300, 672),         # 64 weight rows per workgroup
    (20, 8200, 736),         # 32 weight rows per workgroup
    (129, 257, 96),          # 128-wide tiles: one short stage
    (130, 140, 256),         # two and three stages (the loads' whole lead)
    (130, 140, 384),
    (200, 328, 672),         # 21 blocks: 6 stages
    (300, 130, 896),         # 28 blocks: 7 whole stages
    (385, 260, 1120),        # 35 blocks: 9 stages
    (2900, 2900, 608),       # 256-wide tiles: 19 blocks, 5 stages
    (520, 7200, 544),        # 256 x 128 tiles: 17 blocks, 5 stages, ragged rows
    (700, 5600, 96),         # the same, one short stage
    (300, 12300, 256),       # the same, two stages, ragged columns
    (2830, 3000, 1440),      # 45 blocks, 12 stages
    (150, 200, 2848),        # split (see below): 89 blocks
]


def _operands(M, N, K, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, :: max(7, K // 5)] *= 50
    w = rng.normal(0, 0.02, (N, K)).astype(np.float32)
    return rfq.rfq_quantize_act(dev(x)), rfq.rfq_quantize_weight(dev(w))


def _check(orc, z, q, w, what, phi=None):
    """Every row of small products, 24 rows of large ones."""
    M = q[0].shape[0]
    rows = np.arange(M) if M <= 400 else np.unique(np.concatenate(
        [[0, 255, 256, M - 1], np.random.default_rng(1).integers(0, M, 20)]))
    hq = [None if t is None else host(t)[rows] for t in q]
    zr, bound = orc.gemm(*hq, host(w[0]), host(w[1]))
    bf16 = z.dtype == torch.bfloat16
    zh = host_bf16_as_f32(z) if bf16 else host(z)
    assert_gemm_close(zh[rows], zr, bound, bf16, what)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_product(orc, M, N, K):
    q, w = _operands(M, N, K, M + K)
    print("ragged K: M=%d N=%d K=%d" % (M, N, K), flush=True)
    for dt in (torch.float32, torch.bfloat16):
        _check(orc, rfq.rfq_gemm(*q, *w, out_dtype=dt), q, w, "RFQ %s" % dt)
    plain = (q[0], q[1], None, None)
    _check(orc, rfq.rfq_gemm(*plain, *w), plain, w, "plain")
    if M > 128:
        ones = torch.ones(((M + 63) // 64, (K + 255) // 256), dtype=torch.uint8, device="cuda")
        _check(orc, rfq.rfq_gemm_phi(*q, *w, ones), q, w, "map of ones")
        _check(orc, rfq.rfq_gemm_phi(*q, *w, 0 * ones), plain, w, "map of zeros")


@pytest.mark.parametrize("M,N,K", [(150, 200, 2848), (40, 96, 1056), (33, 64, 5024),
                                   (9, 5000, 12320)])
def test_split_product(orc, M, N, K):
    assert rfq.rfq_gemm_workspace_bytes(M, N, K) > 0
    q, w = _operands(M, N, K, M + K)
    print("ragged K, split: M=%d N=%d K=%d" % (M, N, K), flush=True)
    _check(orc, rfq.rfq_gemm(*q, *w, split=True), q, w, "split")
    if K < 5000:
        _check(orc, rfq.rfq_gemm_split_noalloc(*q, *w), q, w, "split, static array")


@pytest.mark.parametrize("M,N,K", [(5, 64, 544), (150, 64, 1184), (2900, 2900, 608)])
def test_bytes_past_a_row_do_not_reach_it(M, N, K):
    """The bytes after a row's last block are the next row's: with NaN scale
    bytes (0xFF) in every odd row, the even rows of Z in even columns keep
    their bits."""
    q, w = _operands(M, N, K, 3)
    z = rfq.rfq_gemm(*q, *w)
    print("ragged K, NaN rows: M=%d N=%d K=%d" % (M, N, K), flush=True)
    q2, w2 = [t.clone() for t in q], [t.clone() for t in w]
    for t in (q2[1], q2[3], w2[1]):
        t[1::2] = 0xFF
    z2 = rfq.rfq_gemm(*q2, *w2)
    assert torch.equal(z2[::2, ::2], z[::2, ::2])
    assert torch.isnan(z2[1::2]).all() and torch.isnan(z2[:, 1::2]).all()


@pytest.mark.parametrize("M,N,K", [(5, 300, 544), (129, 257, 512), (200, 328, 672)])
def test_unaligned_scale_tensors(orc, M, N, K):
    q, w = _operands(M, N, K, 8)

    def shifted(t):
        raw = torch.empty(t.numel() + 1, dtype=torch.uint8, device="cuda")
        v = raw[1:].view(t.shape)
        v.copy_(t)
        return v

    print("unaligned scales: M=%d N=%d K=%d" % (M, N, K), flush=True)
    _check(orc, rfq.rfq_gemm(q[0], shifted(q[1]), q[2], shifted(q[3]), w[0], shifted(w[1])), q, w,
           "unaligned scales")


@pytest.mark.parametrize("M,N,K", [(1, 70, 512), (16, 300, 1312), (20, 8200, 800), (40, 130, 2048),
                                   (100, 260, 992), (7, 12300, 1024), (100, 12300, 1056),
                                   (200, 130, 2336), (700, 2900, 1120), (520, 7200, 544), (2900, 2900, 608)])
def test_random_maps(orc, M, N, K):
    """Maps on the few-row, 128-wide and 256-wide kernels (the last two rows of
    256-wide tiles run 128-wide ones): random, one all-ones column and row."""
    q, w = _operands(M, N, K, M + N)
    rng = np.random.default_rng(N)
    phi = (rng.random(((M + 63) // 64, (K + 255) // 256)) < 0.5).astype(np.uint8) * 3
    phi[:, -1] = 1
    phi[-1] = 1
    rows = np.arange(M) if M <= 200 else np.unique(np.concatenate(
        [np.arange(64 * ((M - 1) // 64) - 2, M), rng.integers(0, M, 24)]))
    print("maps: M=%d N=%d K=%d" % (M, N, K), flush=True)
    # The oracle on the sampled rows: their map rows repeated for 64-row tiles.
    hq = [host(t) for t in q]
    for dt in (torch.float32, torch.bfloat16):
        z = rfq.rfq_gemm_phi(*q, *w, dev(phi), out_dtype=dt)
        zh = host_bf16_as_f32(z) if dt == torch.bfloat16 else host(z)
        for p in range(phi.shape[0]):
            r = rows[rows // 64 == p]
            if len(r):
                zr, bound = orc.gemm_phi(*[t[r] for t in hq], host(w[0]), host(w[1]), phi[p:p + 1])
                assert_gemm_close(zh[r], zr, bound, dt == torch.bfloat16, "map row %d" % p)
