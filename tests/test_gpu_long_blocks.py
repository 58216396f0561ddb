"""gemm8x2 with more than 4096 rows per workgroup (one tile each, so that one round of workgroups covers the rows): the same
bits as with blocks of 4096 rows, fused and with tables from memory, and the oracle's values."""
import numpy as np
import pytest

from gpu_util import assert_within_tolerance, device_inputs, gpu_gemm, gpu_pack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,q,b,rows", [
    (4171, 1047, 1, 104, 4224), (8147, 1073, 1, 85, 8192), (21290, 15, 2, 85, 4288), (20584, 11, 3, 89, 4160), (17105, 8, 4, 107, 4288)])
def test_blocks_of_more_than_4096_rows(oracle, m, n, q, b, rows):
    import torch

    import paper_2005_09904_amd as biq

    plan = biq.biq_plan_get_lut(m, n, q, b, 8)
    assert (biq.biq_kernel_name(plan.kernel), plan.rows_per_wg, plan.tiles_per_split, plan.row_mode) == ("gemm8x2", rows, 1, 0)
    print("long blocks", m, n, q, b, flush=True)
    rng = np.random.default_rng(54000 + m)
    X = rng.standard_normal((b, n), dtype=np.float32)
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32)
    Bd, ad, Xd = device_inputs(B, alpha, X)
    K = gpu_pack(biq, Bd)
    Y = gpu_gemm(biq, K, ad, Xd, m, n, q, 8, plan)
    short = biq.biq_plan_get_lut(m, n, q, b, 8)
    short.rows_per_wg = 4096
    assert torch.equal(Y, gpu_gemm(biq, K, ad, Xd, m, n, q, 8, short))
    LUT = torch.empty((biq.biq_num_chunks(n, 8), 256, b), device="cuda")
    biq.biq_build_lut(Xd, LUT, n, b, 8)
    ws = torch.empty(max(biq.biq_workspace_bytes(m, n, q, b, 8), 16), dtype=torch.uint8, device="cuda")
    Z = torch.full((b, m), float("nan"), device="cuda")
    biq.biq_query(K, ad, LUT, Z, m, n, q, b, 8, workspace=ws)
    pick = np.unique(np.r_[0:100, 4000:min(m, 4300), m - 100:m])
    ref = oracle.gemm_dense(B[:, pick], alpha[:, pick], X)
    for out in (Y, Z):
        assert_within_tolerance(out.cpu().numpy()[:, pick], ref, alpha[:, pick], X, "long blocks")
    # each rounds the sums of n / 8 entries and their tables, scales and planes: (n / 8 + 24) * 2^-24 of ||x||_1 at most
    limit = 2 * 2.0 ** -24 * (-(-n // 8) + 24) * float(np.abs(alpha).sum(axis=0).max() * np.abs(X).sum(axis=1).max())
    assert float((Y - Z).abs().max()) <= limit
