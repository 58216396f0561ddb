"""biq_quantize at the edges of its rows: exactly full registers, one element less and more, a piece of a
16-byte read past the end, rows on odd float addresses; signs and scales against the oracle, and nothing written
outside the outputs."""
import numpy as np
import pytest

from test_gpu_quantize import _check_against_oracle, _signs_from_bitmap

pytestmark = pytest.mark.gpu
SEED_PIECES = 9100


def _row_lengths(waves, pieces):
    """Lengths of rows of `waves` waves with `pieces` pieces of 256 elements each: filled, one element less, one element more
    than with a piece less, and of four waves one whose last piece exists for two of them.  (From 4 elements on: the
    residuals of one or two are exactly 0 after a plane or two, and their signs then undecided.)"""
    whole = 256 * waves * pieces
    lengths = [whole, whole - 1, max(4, whole - 256 * waves + 1)]
    return lengths + [whole - 256 * 3 + 7] if waves > 1 else lengths


@pytest.mark.parametrize("waves,pieces", [(1, p) for p in range(1, 33)] + [(4, p) for p in range(9, 33)])
def test_quantize_every_number_of_pieces(oracle, waves, pieces):
    # (the seed is one with which the oracle alone leaves fewer elements undecided than the check admits at every length:
    # it expects about 31 +- 6 of the 46 admitted at n = 28000)
    for n in _row_lengths(waves, pieces):
        _check_row_length(oracle, n, SEED_PIECES + n)


@pytest.mark.parametrize("n", [4, 255, 256, 257, 511, 512, 1024, 1026, 2048, 4095, 4096, 4097, 8192, 16383, 16384, 32766])
def test_quantize_row_edges(oracle, n):
    _check_row_length(oracle, n, 8400 + n)


def _check_row_length(oracle, n, seed):
    import torch

    import paper_2005_09904_amd as biq

    m, q = 5, 3
    print("quantize edges n=%d" % n, flush=True)
    rng = np.random.default_rng(seed)
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
