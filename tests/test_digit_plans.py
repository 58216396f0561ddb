"""Plans of the block-scaled matrix-core path (unpack_mfma, row_mode 1): which mappings are accepted, and what
the library chooses (host logic only)."""
import pytest


@pytest.fixture(scope="module")
def biq():
    import paper_2005_09904_amd as biq

    biq.load_library()
    return biq


def _plan(biq, q, bt, gps, ws, r, **fields):
    p = biq.BiqPlan()
    p.kernel, p.threads, p.chunks_per_tile, p.row_mode = 3, 256, 32, 1
    p.batch_tile, p.tiles_per_split, p.wave_splits, p.rows_per_wg = bt, gps, ws, (4 // ws) * 32 * r
    for k, v in fields.items():
        setattr(p, k, v)
    return p


@pytest.mark.parametrize("q", [1, 2, 3, 4])
@pytest.mark.parametrize("bt", [32, 64])
@pytest.mark.parametrize("ws", [1, 2, 4])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 8])
def test_tile_limits(biq, q, bt, ws, r):
    ok = r in (1, 2, 4) and q * r * (bt // 32) <= 8
    if ok:
        p = biq.biq_plan_check(500, 3000, q, 70, 8, _plan(biq, q, bt, 4, ws, r))
        assert p.chunk_splits == 3 and p.input_terms == 3 and p.lds_bytes <= 160 * 1024
    else:
        with pytest.raises(biq.BiqError):
            biq.biq_plan_check(500, 3000, q, 70, 8, _plan(biq, q, bt, 4, ws, r))


def test_refused_fields_and_long_rows(biq):
    for fields in (dict(input_terms=2), dict(row_mode=2), dict(xcd_skew=32), dict(table_fill=1, kernel=1)):
        with pytest.raises(biq.BiqError):
            biq.biq_plan_check(500, 3000, 2, 70, 8, _plan(biq, 2, 32, 4, 1, 1, **fields))
    n = 65 * 256                                        # 65 key groups: one more than a wave can look at together
    biq.biq_plan_check(500, n, 2, 70, 8, _plan(biq, 2, 32, 64, 1, 1))
    biq.biq_plan_check(500, n, 2, 70, 8, _plan(biq, 2, 32, 65, 2, 1))
    with pytest.raises(biq.BiqError):
        biq.biq_plan_check(500, n, 2, 70, 8, _plan(biq, 2, 32, 65, 1, 1))
    # rows beyond every such plan keep the 16-bit terms; the 16-bit plans themselves are what they were
    p = biq.biq_plan_get(4096, 3000000, 1, 200, 8)
    assert p.kernel == 3 and p.row_mode == 0 and p.input_terms == 3
    p = biq.biq_plan_get_mfma(4096, 4096, 3, 32, 8, 3)
    assert p.row_mode == 0 and p.input_terms == 3
    assert biq.biq_plan_get(16384, 4096, 2, 128, 8).row_mode == 1
