"""HiF4 product given a workspace, from 1024 rows: W decoded into it in the
order the matrix instructions take it (N a multiple of 32; else row by row),
128 x 256 or 128 x 512 tiles.  Bit-identical to rfq_hif4_gemm, which decodes
W inside the product, at ragged rows, columns and one to six K blocks."""
import pytest
import torch

import paper_2608_26581_amd as rfq

pytestmark = pytest.mark.gpu

# 256-wide tiles; the last column tile or its second half past N; the last
# two: N not a multiple of 32 (rows as they are).
NARROW = [(1024, 4096, 64), (1030, 4128, 128), (1151, 4384, 192), (4100, 4096, 64),
          (1300, 4224, 384), (1025, 4100, 192), (1024, 12290, 64)]
# 512-wide tiles: their rounds of 256 take less than those of 256-wide ones.
WIDE = [(1024, 12288, 64), (1030, 12256, 128), (1153, 10784, 192), (1024, 10272, 320),
        (2000, 8192, 320)]


@pytest.mark.parametrize("M,N,K", NARROW + WIDE)
def test_workspace_form_keeps_the_bits(M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    x = torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16)
    x[:, ::37] *= 40
    w = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    q = rfq.rfq_hif4_quantize(x)
    wq = rfq.rfq_hif4_quantize(w, residual=False)[:2]
    assert rfq.rfq_hif4_gemm_workspace_bytes(M, N, K) == N * K * 2
    print("HiF4 workspace form: M=%d N=%d K=%d" % (M, N, K), flush=True)
    for dt, iv in ((torch.float32, torch.int32), (torch.bfloat16, torch.int16)):
        for ops in (q, (q[0], q[1], None, None)):
            want = rfq.rfq_hif4_gemm(*ops, *wq, out_dtype=dt)
            # Guard bytes after the workspace stay as they were.
            ws = torch.full((N * K * 2 + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
            got = rfq.rfq_hif4_gemm_split(*ops, *wq, ws[:N * K * 2], out_dtype=dt)
            assert torch.equal(got.view(iv), want.view(iv)), (dt, ops[2] is None)
            assert (ws[N * K * 2:] == 0x5A).all()
