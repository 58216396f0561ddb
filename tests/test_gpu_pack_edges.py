"""biq_pack at the edges of its rows and of its input: lengths around whole dwords and 16-byte reads, rows and inputs on
any byte address, the last bytes of the input, nothing written outside the output."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,q", [(1, 1, 1), (1, 31, 1), (3, 32, 2), (5, 33, 1), (7, 63, 3), (2, 127, 2), (3, 128, 1), (9, 129, 2),
                                   (70, 300, 2), (33, 1001, 3), (2, 4293, 1)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 16])
def test_pack_row_edges(m, n, q, offset):
    import torch

    import paper_2005_09904_amd as biq

    print("pack edges", m, n, q, offset, flush=True)
    rng = np.random.default_rng(100 * n + offset)
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    buf = torch.ones(q * m * n + offset, dtype=torch.int8, device="cuda")          # (the input ends with its memory)
    Bd = buf[offset:].view(q, m, n)
    Bd.copy_(torch.from_numpy(B))
    size = biq.biq_packed_bytes(m, n, q)
    K = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    biq.biq_pack(Bd, K, m, n, q, 8)
    torch.cuda.synchronize()
    assert bool((K[size:] == 0xA5).all())
    bits = np.unpackbits(K[:size].cpu().numpy().reshape(q, m, -1), axis=2, bitorder="little")
    assert np.array_equal(bits[:, :, :n], (B > 0).astype(np.uint8)) and not bits[:, :, n:].any()
