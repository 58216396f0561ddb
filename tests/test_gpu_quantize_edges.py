"""biq_quantize at the edges of its rows: exactly full registers, one element less and more, a piece of a
16-byte read past the end, rows on odd float addresses; signs and scales against the oracle, and nothing written
outside the outputs."""
import numpy as np
import pytest

from test_gpu_quantize import _check_against_oracle, _signs_from_bitmap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 255, 256, 257, 511, 512, 1024, 1026, 2048, 4095, 4096, 4097, 8192, 16383, 16384, 32766])
def test_quantize_row_edges(oracle, n):
    import torch

    import paper_2005_09904_amd as biq

    m, q = 5, 3
    print("quantize edges n=%d" % n, flush=True)
    rng = np.random.default_rng(8400 + n)
    W = rng.standard_normal((m, n)).astype(np.float32)
    buf = torch.full((m * n + 1 + 64,), float("nan"), device="cuda")     # what lies behind a row must not count
    Wd = buf[1:1 + m * n].view(m, n)
    Wd.copy_(torch.from_numpy(W))
    size = biq.biq_packed_bytes(m, n, q)
    K = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    alpha = torch.full((q * m + 16,), 7.0, device="cuda")
    biq.biq_quantize(Wd, K, alpha, m, n, q)
    torch.cuda.synchronize()
    assert bool((K[size:] == 0xA5).all()) and bool((alpha[q * m:] == 7.0).all())
    B_ref, alpha_ref, R = oracle.quantize_greedy(W, q, with_residuals=True)
    B, padding = _signs_from_bitmap(K[:size].cpu().numpy(), q, m, n)
    assert not padding.any()
    _check_against_oracle(W, q, B, alpha[:q * m].cpu().numpy().reshape(q, m).astype(np.float64), B_ref, alpha_ref, R)
