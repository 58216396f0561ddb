"""biq_query, mu = 8, few lookups with very many input vectors: the tables' entries that a tile's chunks past the end of a
row would have lie beyond 32-bit byte offsets there.  Every result against a plain product in 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [
    # m, n, batch: chunks past the row, up to the end of the tile (63 or 127), times 1 KiB per vector
    (64, 8, 131072),        # chunk 32 at exactly 2^32 bytes
    (16, 64, 70000),        # chunks 60 .. 63 past 2^32
    (64, 8, 65535),         # the whole tile below 2^32
    (2, 520, 33000),        # two tiles of 64 (wider than one)
    (4, 8, 300000),         # more than 65535 groups of four vectors
]


@pytest.mark.parametrize("m,n,b", SHAPES)
def test_query_many_vectors(m, n, b):
    import torch

    import paper_2005_09904_amd as biq

    print("query many vectors", m, n, b, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n + b)
    signs = torch.randint(0, 2, (1, m, n), dtype=torch.int8, device="cuda", generator=g) * 2 - 1
    K = torch.empty(biq.biq_packed_bytes(m, n, 1), dtype=torch.uint8, device="cuda")
    biq.biq_pack(signs, K, m, n, 1, 8)
    alpha = torch.rand((1, m), device="cuda", generator=g) + 0.5
    X = torch.randn((b, n), device="cuda", generator=g)
    LUT = torch.empty(biq.biq_num_chunks(n, 8) * 256 * b, device="cuda")
    biq.biq_build_lut(X, LUT, n, b, 8)
    ws = torch.empty(max(biq.biq_workspace_bytes(m, n, 1, b, 8), 16), dtype=torch.uint8, device="cuda")
    Y = torch.full((b, m), float("nan"), device="cuda")
    biq.biq_query(K, alpha, LUT, Y, m, n, 1, b, 8, workspace=ws)
    torch.cuda.synchronize()
    ref = (X.double() @ signs[0].double().t()) * alpha.double()
    # n additions and a product, each rounded by at most 2^-24 of the sum of magnitudes
    bound = (n + 2) * 2.0 ** -24 * X.double().abs().sum(dim=1, keepdim=True) * alpha.double()
    assert bool(((Y.double() - ref).abs() <= bound).all())
