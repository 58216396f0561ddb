"""biq_query on tables in device memory, read in place (few lookups) or copied to LDS: the bits of the fused table
kernel of the same plan, at the edges of tiles, chunks, rows and vectors and on both sides of the rule."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [
    # m, n, q, batch
    (1, 1, 1, 1), (7, 9, 2, 2), (9, 1023, 3, 3), (65, 1025, 4, 5), (300, 512, 1, 7), (31, 513, 2, 4), (250, 1024, 2, 8),
    (17, 129, 4, 6), (513, 2048, 3, 1), (40, 2049, 2, 1), (333, 1000, 4, 1), (100, 3000, 1, 1), (2050, 2050, 2, 9),
    (4096, 2056, 4, 8),                 # copied: 8.4 million reads
    (5000, 1024, 4, 1), (9000, 1024, 4, 1),   # 2.6 million: in place; 4.6: copied
    # rows of many splits: in the waves of a workgroup, up to 8 of them and in turns (11, 25, 40)
    (1, 8192, 1, 64), (5, 11264, 1, 9), (17, 25600, 1, 16), (1, 40960, 1, 13),
    # ... and in workgroups of their own: few rows, the last row of a workgroup alone, odd lengths, more splits than waves hold
    (64, 16384, 2, 8), (9, 40001, 2, 4), (128, 40000, 2, 4), (3, 20000, 4, 3), (11, 35841, 2, 17), (64, 131072, 1, 4), (2, 66560, 3, 5),
]


@pytest.mark.parametrize("m,n,q,b", SHAPES)
def test_query_equals_the_fused_kernel_bit_for_bit(m, n, q, b):
    import torch

    import paper_2005_09904_amd as biq

    print("query", m, n, q, b, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    stride = biq.biq_key_row_stride(n)
    bits = torch.randint(0, 2, (q, m, n), dtype=torch.int8, device="cuda", generator=g) * 2 - 1
    K = torch.empty(q * m * stride, dtype=torch.uint8, device="cuda")
    biq.biq_pack(bits, K, m, n, q, 8)
    alpha = torch.rand((q, m), device="cuda", generator=g)
    # inputs and tables on odd float addresses: nothing may rely on more than 4 bytes
    X = torch.randn(b * n + 1, device="cuda", generator=g)[1:].view(b, n)
    LUT = torch.empty(biq.biq_num_chunks(n, 8) * 256 * b + 1, device="cuda")[1:]
    biq.biq_build_lut(X, LUT, n, b, 8)
    ws = torch.empty(max(biq.biq_workspace_bytes(m, n, q, b, 8), 16), dtype=torch.uint8, device="cuda")
    guard = torch.full((b * m + 64,), 7.0, device="cuda")
    Y = guard[:b * m].view(b, m)
    biq.biq_query(K, alpha, LUT, Y, m, n, q, b, 8, workspace=ws)
    Yf = torch.full((b, m), float("nan"), device="cuda")
    biq.biq_gemm_ex(K, alpha, X, Yf, m, n, q, b, 8, biq.biq_plan_get_lut(m, n, q, b, 8), workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(Y, Yf) and bool((guard[b * m:] == 7.0).all())


@pytest.mark.parametrize("m,n,q,b,apart", [(64, 4096, 2, 8, False), (17, 25600, 1, 16, False), (64, 16384, 2, 8, True), (16, 65536, 2, 4, True)])
def test_splits_of_few_rows_have_workgroups_of_their_own(m, n, q, b, apart):
    """Then, and only then, their sums pass through the workspace."""
    import torch

    import paper_2005_09904_amd as biq

    print("query splits", m, n, q, b, flush=True)
    K = torch.zeros(biq.biq_packed_bytes(m, n, q), dtype=torch.uint8, device="cuda")
    alpha = torch.ones((q, m), device="cuda")
    LUT = torch.ones((biq.biq_num_chunks(n, 8) << 8) * b, device="cuda")
    ws = torch.full((biq.biq_workspace_bytes(m, n, q, b, 8),), 0xA5, dtype=torch.uint8, device="cuda")
    Y = torch.empty((b, m), device="cuda")
    biq.biq_query(K, alpha, LUT, Y, m, n, q, b, 8, workspace=ws)
    torch.cuda.synchronize()
    assert bool((Y == q * biq.biq_num_chunks(n, 8)).all())
    splits = biq.biq_plan_get_lut(m, n, q, b, 8).chunk_splits
    assert splits > 1 and bool((ws[:4 * splits * b * m].view(torch.float32) == q * 128).all()) == apart
