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


def test_direct_plans(biq):
    """table_fill = 2: which plans take it, where the library chooses it, and that the plan is otherwise the table
    kernel's, workspace included."""
    for (m, n, q, b, mu, want) in [(512, 512, 1, 1, 8, 0), (2048, 2048, 2, 1, 8, 0), (5000, 3001, 2, 1, 8, 2), (32000, 1024, 3, 6, 8, 2),
                                   (1 << 20, 2048, 2, 1, 8, 0), (5003, 3001, 3, 7, 6, 2), (90, 1000, 2, 3, 4, 0),
                                   (50, 600, 1, 2, 6, 0), (100, 700, 3, 6, 8, 0), (200, 1500, 2, 1, 8, 0)]:
        p, lut = biq.biq_plan_get(m, n, q, b, mu), biq.biq_plan_get_lut(m, n, q, b, mu)
        assert p.table_fill == want and lut.table_fill == 0
        want_fields = dict(lut.as_dict(), table_fill=want)
        assert p.as_dict() == want_fields
        assert biq.biq_plan_workspace_bytes(p, m, b) == biq.biq_plan_workspace_bytes(lut, m, b)
    p = biq.biq_plan_get_lut(300, 700, 5, 2, 8)              # five planes
    p.table_fill = 2
    with pytest.raises(biq.BiqError):
        biq.biq_plan_check(300, 700, 5, 2, 8, p)
    p = biq.biq_plan_get_lut(300, 42000, 1, 1, 8)            # a vector's digits do not fit the LDS
    p.table_fill = 2
    with pytest.raises(biq.BiqError):
        biq.biq_plan_check(300, 42000, 1, 1, 8, p)


@pytest.mark.parametrize("m,n,q,direct", [
    (4096, 4096, 2, True), (16384, 4096, 2, True), (256, 5952, 3, True), (4096, 11008, 2, True), (128, 2052, 2, True),
    (4096, 2048, 2, False), (127, 4096, 2, False), (1088, 9288, 4, False), (234, 32722, 4, False), (36294, 3136, 2, False),
    (47993, 6847, 3, False), (256, 42000, 1, False), (4096, 4096, 5, False)])
def test_one_vector_plans(biq, m, n, q, direct):
    """One vector on wide rows: tables or none by the estimates of both; the plan is the table kernel's in any case."""
    p, lut = biq.biq_plan_get(m, n, q, 1, 8), biq.biq_plan_get_lut(m, n, q, 1, 8)
    assert p.as_dict() == dict(lut.as_dict(), table_fill=2 if direct else 0)
    assert biq.biq_plan_workspace_bytes(p, m, 1) == biq.biq_plan_workspace_bytes(lut, m, 1)


@pytest.mark.parametrize("m,n,q,b,mu", [
    (25633, 11584, 1, 1, 8), (3639, 13054, 1, 1, 8), (10240, 11353, 4, 1, 8), (963, 11927, 4, 21, 8), (384, 519, 4, 51, 8),
    (17664, 13056, 2, 3, 8), (4736, 2781, 3, 29, 8), (6080, 13568, 1, 3, 8), (681, 5504, 1, 18, 5), (136, 7558, 2, 58, 4),
    (1010, 20480, 2, 1, 8), (4096, 4096, 2, 1, 8), (128, 256, 1, 2, 8)])
def test_table_plans_fill_one_round(biq, m, n, q, b, mu):
    """No more workgroups than the 256 CUs where fewer blocks of rows make that possible, and every row in one of them."""
    p = biq.biq_plan_get_lut(m, n, q, b, mu)
    each = p.chunk_splits * p.batch_tiles
    assert each > 256 or p.row_blocks * each <= 256
    assert (p.row_blocks - 1) * p.rows_per_wg < m <= p.row_blocks * p.rows_per_wg


def test_direct_row_limit(biq):
    """The direct kernel counts rows in 32 bits, those its last row steps have past the end included."""
    for m, ok in ((1 << 30, True), ((1 << 30) + 1, False), (3 << 29, False)):
        p = biq.biq_plan_get_lut(m, 100, 1, 3, 8)
        assert biq.biq_plan_get(m, 100, 1, 3, 8).table_fill in ((0, 2) if ok else (0,))
        p.table_fill = 2
        if ok:
            assert biq.biq_plan_check(m, 100, 1, 3, 8, p).table_fill == 2
        else:
            with pytest.raises(biq.BiqError):
                biq.biq_plan_check(m, 100, 1, 3, 8, p)


@pytest.mark.parametrize("m,n,q,b,mu", [
    (310460, 192, 1, 1, 4), (70016, 286, 1, 1, 4), (90816, 128, 1, 1, 6), (300000, 256, 1, 1, 5), (1 << 20, 128, 1, 1, 4),
    (320782, 131, 2, 1, 6), (367424, 154, 4, 1, 6), (209107, 128, 3, 1, 6), (145712, 512, 1, 1, 4), (65088, 128, 1, 1, 7),
    (982, 144, 2, 1, 4), (221, 3376, 4, 25, 4), (150, 3086, 2, 51, 4), (458, 2061, 3, 15, 4), (133, 3208, 1, 10, 4)])
def test_tables_where_they_are_faster(biq, m, n, q, b, mu):
    """Short rows with one vector and few rows of narrow keys: 1.1 to 5.7 times the tables' time without them.  (What runs is
    allowed to be the direct kernel for one vector on rows of several key units, never the 32-vector one.)"""
    p, lut = biq.biq_plan_get(m, n, q, b, mu), biq.biq_plan_get_lut(m, n, q, b, mu)
    if (m, n) in ((70016, 286), (300000, 256), (145712, 512)):
        assert p.kernel == lut.kernel
    else:
        assert p.as_dict() == lut.as_dict()


def test_two_column_tiles_for_long_rows_and_eight_tiles(biq):
    """Where estimates tie, the mapping that bf16 values prefer (they keep 16-bit weights, expanded per column tile)."""
    for (m, n, q, b) in [(16384, 4096, 2, 128), (25237, 2972, 4, 37)]:
        p = biq.biq_plan_get(m, n, q, b, 8)
        assert p.kernel == 3 and p.row_mode == 1 and p.batch_tile == 64
    assert biq.biq_plan_get(31424, 512, 2, 104, 8).batch_tile == 32


@pytest.mark.parametrize("m,n,q,b,mu,tables,direct,digits", [
    # us per call, keys from memory; digits: 0 where they are far behind
    (174, 156, 4, 3, 8, 4.9, 4.1, 0), (184, 256, 4, 2, 8, 4.9, 4.2, 0), (512, 512, 2, 2, 8, 4.3, 3.8, 0), (1024, 512, 2, 3, 8, 4.5, 3.9, 0),
    (3477, 349, 2, 162, 8, 10.6, 8.9, 0), (1088, 510, 2, 181, 8, 7.7, 6.8, 0), (17937, 160, 3, 11, 8, 7.4, 6.5, 0),
    (7897, 2672, 1, 7, 8, 9.1, 8.0, 0), (10240, 128, 2, 64, 8, 10.2, 8.4, 8.1), (11450, 256, 3, 42, 8, 11.4, 9.1, 9.4),
    (1599, 1167, 4, 30, 8, 12.2, 11.5, 10.9), (1918, 6208, 2, 17, 8, 13.5, 11.4, 13.9), (20066, 8492, 2, 7, 8, 42.0, 36.9, 52.1),
    (766, 14080, 2, 13, 8, 13.8, 11.1, 15.6), (7342, 12160, 2, 4, 8, 21.9, 21.0, 32.3), (1145, 7117, 4, 7, 8, 12.2, 12.7, 0),
    (16834, 4928, 1, 2, 8, 9.6, 11.2, 0), (160, 14656, 2, 4, 8, 9.0, 9.7, 0), (919, 832, 3, 9, 8, 4.6, 6.5, 0), (2048, 1024, 2, 4, 8, 4.3, 5.4, 0),
    (291, 601, 2, 10, 8, 4.6, 6.4, 0), (1152, 704, 2, 10, 8, 4.1, 6.5, 0), (309, 1652, 3, 25, 8, 6.7, 8.9, 0),
    (171670, 8874, 1, 1, 6, 78.7, 58.4, 0), (576, 16355, 4, 1, 6, 13.5, 10.9, 0), (38243, 14976, 1, 1, 4, 35.0, 27.9, 0),
    (225, 3584, 2, 192, 4, 15.7, 11.4, 0), (965, 3317, 1, 106, 4, 16.3, 0, 13.6), (133, 3208, 1, 10, 4, 6.4, 9.7, 0), (80000, 128, 1, 1, 7, 4.4, 5.9, 0)])
def test_choice_by_measured_times(biq, m, n, q, b, mu, tables, direct, digits):
    """What the library chooses among tables, direct and digits takes at most 5 % longer than the best of them."""
    p = biq.biq_plan_get(m, n, q, b, mu)
    chosen = digits if p.kernel == 3 else direct if p.table_fill == 2 else tables
    assert 0 < chosen <= 1.05 * min(t for t in (tables, direct, digits) if t)
