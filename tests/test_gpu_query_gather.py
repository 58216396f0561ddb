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
