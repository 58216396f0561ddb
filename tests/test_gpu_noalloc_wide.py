"""biq_gemm_noalloc where the digit plan needs more than the fixed buffer: a plan that fits it takes the call."""
import pytest

from gpu_util import assert_within_tolerance, device_inputs, gpu_pack
from test_zz_no_alloc import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,q,b,mu", [(1006, 23448, 1, 207, 5), (2499, 11820, 1, 392, 2)])
def test_noalloc_takes_a_smaller_plan(oracle, m, n, q, b, mu):
    import torch

    import paper_2005_09904_amd as biq

    assert biq.biq_workspace_bytes(m, n, q, b, mu) > biq.biq_noalloc_scratch_bytes()
    print("noalloc m=%d n=%d q=%d b=%d mu=%d" % (m, n, q, b, mu), flush=True)
    B, alpha, X = _inputs(m, n, q, b, 77)
    Bd, ad, Xd = device_inputs(B, alpha, X)
    K = gpu_pack(biq, Bd)
    Y = torch.full((b, m), float("nan"), dtype=torch.float32, device="cuda")
    biq.biq_gemm_noalloc(K, ad, Xd, Y, m, n, q, b, mu)
    torch.cuda.synchronize()
    assert_within_tolerance(Y[:4].cpu().numpy(), oracle.gemm_dense(B, alpha, X[:4]), alpha, X[:4], "noalloc")


@pytest.mark.parametrize("m,n,q,b,mu", [(20, 62289, 4, 193, 8), (16, 165265, 2, 82, 8)])
def test_noalloc_few_rows(oracle, m, n, q, b, mu):
    """Few rows of many columns: where the fitting plan is the table kernels', whose partial sums are small."""
    import torch

    import paper_2005_09904_amd as biq

    print("noalloc m=%d n=%d q=%d b=%d mu=%d" % (m, n, q, b, mu), flush=True)
    B, alpha, X = _inputs(m, n, q, b, 78)
    Bd, ad, Xd = device_inputs(B, alpha, X)
    Y = torch.full((b, m), float("nan"), dtype=torch.float32, device="cuda")
    biq.biq_gemm_noalloc(gpu_pack(biq, Bd), ad, Xd, Y, m, n, q, b, mu)
    torch.cuda.synchronize()
    assert_within_tolerance(Y[:4].cpu().numpy(), oracle.gemm_dense(B, alpha, X[:4]), alpha, X[:4], "noalloc")


@pytest.mark.parametrize("m,n,q,b,mu", [
    # the plan that fits: tables (generic kernel; batched), digits, three 16-bit terms
    (61, 186587, 1, 1, 9), (20, 62289, 4, 193, 8), (292233, 1950, 1, 8, 5), (49252, 145771, 1, 4, 3)])
def test_noalloc_any_plan_that_fits(m, n, q, b, mu):
    """Neither biq_gemm's plan nor the one for small workspaces fits: each of the others, on rows at both ends."""
    import torch

    import paper_2005_09904_amd as biq

    assert biq.biq_plan_workspace_bytes(biq.biq_plan_get(m, n, q, b, mu), m, b) > biq.biq_noalloc_scratch_bytes()
    print("noalloc m=%d n=%d q=%d b=%d mu=%d" % (m, n, q, b, mu), flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(79)
    K = torch.randint(0, 256, (q, m, biq.biq_key_row_stride(n)), dtype=torch.uint8, device="cuda", generator=g)
    K[:, :, n // 8] &= (1 << n % 8) - 1
    K[:, :, n // 8 + 1:] = 0
    alpha = torch.rand((q, m), device="cuda", generator=g) + 0.05
    X = torch.randn((b, n), device="cuda", generator=g)
    Y = torch.full((b, m), float("nan"), dtype=torch.float32, device="cuda")
    biq.biq_gemm_noalloc(K, alpha, X, Y, m, n, q, b, mu)
    torch.cuda.synchronize()
    assert not bool(torch.isnan(Y).any())
    rows = sorted({*range(min(m, 40)), *range(max(0, m - 40), m)})
    bits = torch.arange(8, dtype=torch.uint8, device="cuda")
    W = sum((((K[i, rows, :, None] >> bits) & 1).reshape(len(rows), -1)[:, :n].double() * 2 - 1) * alpha[i, rows, None].double()
            for i in range(q))
    ref = (X.double() @ W.t()).cpu().numpy()
    assert_within_tolerance(Y[:, rows].cpu().numpy(), ref, alpha[:, rows].cpu().numpy(), X.cpu().numpy(), "noalloc")
