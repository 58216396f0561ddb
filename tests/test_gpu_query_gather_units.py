"""biq_query, any mu, on tables in device memory: read in place (few lookups, tiles of a row side by side in a wave or
in a workgroup's waves) or copied to LDS, the bits of the fused table kernel of the same plan."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [
    # m, n, q, batch, mu
    (1, 1, 1, 1, 4), (7, 9, 2, 2, 6), (33, 128, 3, 3, 6), (65, 129, 5, 5, 8), (130, 1000, 2, 4, 7), (187, 2894, 4, 15, 7),
    (64, 640, 1, 9, 1), (31, 257, 2, 8, 2), (90, 511, 1, 1, 3), (75, 2500, 2, 3, 4), (75, 2500, 2, 14, 4), (40, 1023, 2, 13, 5),
    (17, 4096, 1, 6, 6), (300, 321, 3, 1, 7), (21, 1300, 2, 5, 9), (21, 1300, 2, 1, 10), (257, 3000, 2, 16, 10),
    (400, 1000, 6, 2, 8),                 # more planes than the mu = 8 kernels hold
    (2000, 3072, 4, 3, 6), (2200, 3072, 4, 4, 6),      # query_wide: 4.1 million reads in place, 4.5 copied
    (4096, 2000, 4, 14, 5), (4096, 1500, 4, 14, 5),    # generic: 26 million copied, 19.7 in place
    # few long rows: in place up to what a workgroup reads, copied beyond
    (4, 53398, 1, 3, 5), (31, 11428, 4, 4, 7), (4, 100000, 2, 4, 6), (10, 124685, 4, 5, 5), (176, 76222, 4, 1, 7),
    (4200, 10240, 1, 12, 10),             # the most LDS: 64 splits, a lane per row
]


@pytest.mark.parametrize("m,n,q,b,mu", SHAPES)
def test_query_equals_the_fused_kernel_bit_for_bit(m, n, q, b, mu):
    import torch

    import paper_2005_09904_amd as biq

    print("query", m, n, q, b, mu, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    bits = torch.randint(0, 2, (q, m, n), dtype=torch.int8, device="cuda", generator=g) * 2 - 1
    K = torch.empty(biq.biq_packed_bytes(m, n, q), dtype=torch.uint8, device="cuda")
    biq.biq_pack(bits, K, m, n, q, mu)
    alpha = torch.rand((q, m), device="cuda", generator=g)
    # inputs and tables on odd float addresses: nothing may rely on more than 4 bytes
    X = torch.randn(b * n + 1, device="cuda", generator=g)[1:].view(b, n)
    LUT = torch.empty((biq.biq_num_chunks(n, mu) << mu) * b + 1, device="cuda")[1:]
    biq.biq_build_lut(X, LUT, n, b, mu)
    ws = torch.empty(max(biq.biq_workspace_bytes(m, n, q, b, mu), 16), dtype=torch.uint8, device="cuda")
    guard = torch.full((b * m + 64,), 7.0, device="cuda")
    Y = guard[:b * m].view(b, m)
    biq.biq_query(K, alpha, LUT, Y, m, n, q, b, mu, workspace=ws)
    Yf = torch.full((b, m), float("nan"), device="cuda")
    biq.biq_gemm_ex(K, alpha, X, Yf, m, n, q, b, mu, biq.biq_plan_get_lut(m, n, q, b, mu), workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(Y, Yf) and bool((guard[b * m:] == 7.0).all())


@pytest.mark.parametrize("m,n,q,b,mu,copied", [(4, 53398, 1, 3, 5, False), (4, 100000, 2, 4, 6, True), (176, 76222, 4, 1, 7, True)])
def test_few_long_rows_are_copied(m, n, q, b, mu, copied):
    """Then, and only then, the sums of the splits pass through the workspace."""
    import torch

    import paper_2005_09904_amd as biq

    print("query few long rows", m, n, q, b, mu, flush=True)
    K = torch.zeros(biq.biq_packed_bytes(m, n, q), dtype=torch.uint8, device="cuda")
    alpha = torch.ones((q, m), device="cuda")
    LUT = torch.ones((biq.biq_num_chunks(n, mu) << mu) * b, device="cuda")
    ws = torch.full((biq.biq_workspace_bytes(m, n, q, b, mu),), 0xA5, dtype=torch.uint8, device="cuda")
    Y = torch.empty((b, m), device="cuda")
    biq.biq_query(K, alpha, LUT, Y, m, n, q, b, mu, workspace=ws)
    torch.cuda.synchronize()
    assert bool((Y == q * biq.biq_num_chunks(n, mu)).all())
    p = biq.biq_plan_get_lut(m, n, q, b, mu)
    assert p.chunk_splits > 1
    assert bool((ws[:4 * b * m].view(torch.float32) == q * p.tiles_per_split * p.chunks_per_tile).all()) == copied
