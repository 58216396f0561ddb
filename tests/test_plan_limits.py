"""Planning at the ends of the ranges the header admits (m * q and n below 2^31, any batch): every call returns a status, and
what a plan says covers the shape (host logic only)."""
import pytest

TOP = (1 << 31) - 1


@pytest.fixture(scope="module")
def biq():
    import paper_2005_09904_amd as biq

    biq.load_library()
    return biq


@pytest.mark.parametrize("m,n,q,b,mu", [
    (TOP, 100, 1, 3, 8), (TOP, 8, 1, 1, 8), (TOP, 2000, 1, 1, 4), (TOP // 2, 300, 2, 70, 6), (TOP, 40, 1, TOP, 8),
    (64, TOP, 1, 1, 8), (64, TOP, 1, 2, 8), (64, TOP, 1, 33, 3), (1, TOP, 5, 1, 10), (300, TOP, 4, TOP, 1),
    (8, 8, 1, TOP, 8), (5000, 3000, 3, TOP, 7), (TOP, TOP, 1, TOP, 2),
])
def test_plans_at_the_limits(biq, m, n, q, b, mu):
    assert biq.biq_key_row_stride(n) == -(-n // 128) * 16
    assert biq.biq_num_chunks(n, mu) == -(-n // mu)
    for get in (biq.biq_plan_get, biq.biq_plan_get_lut):
        try:
            p = get(m, n, q, b, mu)
        except biq.BiqError as e:
            assert e.status == biq.BIQ_EUNSUPPORTED
            continue
        assert 1 <= p.rows_per_wg and p.rows_per_wg * p.row_blocks >= m and p.batch_tile * p.batch_tiles >= b
        assert 1 <= p.row_blocks * p.chunk_splits * p.batch_tiles <= 1 << 30
    biq.biq_workspace_bytes(m, n, q, b, mu)
