"""GPU parity of the block-scaled matrix-core path (unpack_mfma plans with row_mode 1) at the edges of its tiles,
splits and input forms, against the CPU oracle."""
import numpy as np
import pytest

from gpu_util import assert_within_tolerance, device_inputs, gpu_gemm, gpu_pack
from test_digit_plans import _plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def biq():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_09904_amd as biq

    biq.load_library()
    return biq


def _inputs(m, n, q, b, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((b, n), dtype=np.float32)
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    return B, rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32), X


def _bound(alpha, X):
    """Per input vector.  Split: each element is off by at most u = 2^-24 of the largest of its 32 neighbours.
    Sums: the first digits' by at most one rounding per 64 elements, the others' (2^-4 of the elements) by four,
    then at most 16 roundings over wave groups, workgroups, planes and scales: u * ||x||_1 each."""
    b, n = X.shape
    A = np.zeros((b, -(-n // 32) * 32))
    A[:, :n] = np.abs(X)
    steps = -(-n // 64)
    split = 32 * A.reshape(b, -1, 32).max(axis=2).sum(axis=1)
    return 2.0 ** -24 * np.abs(alpha).sum(axis=0).max() * (split + A.sum(axis=1) * (steps * 1.25 + 16))


SHAPES = [
    # m, n, q, batch, column tile, key groups per split, wave groups, row tiles
    (64, 128, 1, 1, 32, 1, 1, 1),        # half a key group, one vector
    (257, 2050, 2, 33, 32, 9, 1, 2),     # one row, two columns, one vector past full tiles; n % 4 = 2
    (300, 1001, 1, 70, 64, 2, 1, 4),     # odd n: unaligned rows, several splits, the last one short
    (130, 1300, 3, 64, 64, 3, 2, 1),     # wave groups of 2 + 1 key groups
    (100, 2300, 2, 20, 32, 9, 4, 4),     # 3 + 3 + 3 + 0 key groups, eight tiles
    (128, 256, 4, 100, 64, 1, 4, 1),     # one key group: three wave groups without work
    (4, 512, 4, 5, 32, 2, 2, 2),
    (1, 40, 2, 2, 32, 1, 2, 1),
]


@pytest.mark.parametrize("m,n,q,b,bt,gps,ws,r", SHAPES)
@pytest.mark.parametrize("form", ["fp32", "bf16", "mixed"])
def test_digit_parity(biq, oracle, m, n, q, b, bt, gps, ws, r, form):
    import torch

    print("digits", m, n, q, b, bt, gps, ws, r, form, flush=True)
    B, alpha, X = _inputs(m, n, q, b, 31000 + m + n)
    if form != "fp32":
        full = X
        X = torch.from_numpy(X).bfloat16().float().numpy()
        if form == "mixed":                              # both forms within a row, in the first column group only
            X[0, n // 2] = full[0, n // 2] * np.float32(1.0001)
    Bd, ad, Xd = device_inputs(B, alpha, X)
    Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Xd, m, n, q, 8, plan=_plan(biq, q, bt, gps, ws, r)).cpu().numpy()
    ref = oracle.gemm_dense(B, alpha, X)
    assert_within_tolerance(Y, ref, alpha, X, "digits")
    assert np.all(np.abs(Y - ref).max(axis=1) <= _bound(alpha, X))


def test_digits_hold_what_they_promise(biq, oracle):
    """Exact inputs bit for bit; a one-hot vector returns its element; scales from 2^-100 to 2^95 and elements over
    twelve orders of magnitude within the bound; Inf and NaN stay in their vector."""
    from paper_2005_09904_amd.workloads import Workload, make_exact_inputs

    B, alpha, X = make_exact_inputs(Workload("exact", 200, 1280, 3, 40, 8, "uniform", seed=78))
    Bd, ad, Xd = device_inputs(B, alpha, X)
    K = gpu_pack(biq, Bd)
    plan = lambda: _plan(biq, 3, 64, 3, 2, 1)
    assert np.array_equal(gpu_gemm(biq, K, ad, Xd, 200, 1280, 3, 8, plan=plan()).cpu().numpy().astype(np.float64),
                          oracle.gemm_dense(B, alpha, X))
    rng = np.random.default_rng(6)
    X = rng.standard_normal((40, 1280)).astype(np.float64)
    for a in range(40):
        if a % 3 == 1:
            X[a] *= 10.0 ** rng.uniform(-9, 3, size=1280)
        X[a] *= 2.0 ** (-100 + 5 * a)
    X[7] = 0.0
    X = X.astype(np.float32)
    alpha = rng.uniform(0.05, 1.0, size=(3, 200)).astype(np.float32)
    _, ad, Xd = device_inputs(B, alpha, X)
    Y = gpu_gemm(biq, K, ad, Xd, 200, 1280, 3, 8, plan=plan()).cpu().numpy()
    ref = oracle.gemm_dense(B, alpha, X)
    assert np.all(Y[7] == 0.0) and np.all(np.abs(Y - ref).max(axis=1) <= _bound(alpha, X))
    bad = X.copy()
    bad[3, 100], bad[20, 1279] = np.inf, np.nan
    _, _, Xd = device_inputs(B, alpha, bad)
    Z = gpu_gemm(biq, K, ad, Xd, 200, 1280, 3, 8, plan=plan()).cpu().numpy()
    assert np.isnan(Z[[3, 20]]).all()
    rest = [a for a in range(40) if a not in (3, 20)]
    assert np.array_equal(Z[rest], Y[rest])
    Bh = -np.ones((1, 64, 256), dtype=np.int8)
    Xh = np.zeros((32, 256), dtype=np.float32)
    vals = rng.standard_normal(32).astype(np.float32) * np.float32(1.2345678)
    Xh[np.arange(32), rng.integers(0, 256, size=32)] = vals
    Bd, ad, Xd = device_inputs(Bh, np.ones((1, 64), dtype=np.float32), Xh)
    Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Xd, 64, 256, 1, 8, plan=_plan(biq, 1, 32, 1, 1, 1)).cpu().numpy()
    assert np.array_equal(Y, np.repeat(-vals[:, None], 64, axis=1))


@pytest.mark.parametrize("exponent", [-105, -110, -120, -126, -135])
def test_digits_small_inputs(biq, oracle, exponent):
    """Vectors far below one keep their bits: the bound relative to the elements, and what sums that are subnormal
    themselves are rounded to (half an instruction's last place, 2^-148, for each of a row's instructions)."""
    rng = np.random.default_rng(900 - exponent)
    m, n, q, b = 100, 1300, 2, 40
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32)
    X = rng.standard_normal((b, n))
    X[::3] *= 2.0 ** exponent
    X[1::3] *= 2.0 ** exponent * 10.0 ** rng.uniform(-3, 3, size=n)
    X[2] *= 2.0 ** 100                                  # large vectors among them change nothing
    X = X.astype(np.float32)
    Bd, ad, Xd = device_inputs(B, alpha, X)
    Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Xd, m, n, q, 8, plan=_plan(biq, q, 32, 6, 2, 2)).cpu().numpy()
    least = np.abs(alpha).sum(axis=0).max() * 5 * -(-n // 64) * 2.0 ** -148 + 2.0 ** -149
    assert np.all(np.abs(Y - oracle.gemm_dense(B, alpha, X)).max(axis=1) <= _bound(alpha, X) + least)


def test_digits_largest_inputs(biq, oracle):
    """The largest fp32 alone in a vector comes back as it is, in either form; sums below it do not overflow."""
    top = np.finfo(np.float32).max
    bf16_top = np.float32(2.0 ** 127 * (2 - 2.0 ** -7))
    m, n = 64, 300
    B = np.ones((1, m, n), dtype=np.int8)
    B[0, ::2] = -1
    alpha = np.full((1, m), 0.5, dtype=np.float32)
    X = np.zeros((34, n), dtype=np.float32)
    X[0, 5], X[1, 299], X[2, 17] = top, -top, top * np.float32(0.99)
    X[3] = top / np.float32(310.0)
    X[33, 40], X[33, 290] = bf16_top, -bf16_top / 4      # a column group of its own: 16-bit form
    Bd, ad, Xd = device_inputs(B, alpha, X)
    Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Xd, m, n, 1, 8, plan=_plan(biq, 1, 32, 2, 1, 1)).cpu().numpy()
    ref = oracle.gemm_dense(B, alpha, X)
    assert np.isfinite(Y).all()
    assert np.array_equal(Y[[0, 1, 2, 33]].astype(np.float64), ref[[0, 1, 2, 33]])
    assert np.all(np.abs(Y - ref).max(axis=1) <= _bound(alpha, X))


@pytest.mark.parametrize("n,b", [(256, 33), (1001, 40), (1002, 31), (1003, 64), (130, 5)])
@pytest.mark.parametrize("form", ["fp32", "bf16"])
def test_digits_inputs_on_odd_addresses(biq, oracle, n, b, form):
    """Vectors on odd float addresses, NaN in front of the first and behind the last: reads past a vector's end and past
    the batch count as zero, and no alignment is assumed.  Nothing is written outside the results."""
    import torch

    m, q = 70, 2
    print("digits, odd addresses", n, b, form, flush=True)
    B, alpha, X = _inputs(m, n, q, b, 600 + n)
    if form == "bf16":
        X = torch.from_numpy(X).bfloat16().float().numpy()
    Bd, ad, _ = device_inputs(B, alpha, X)
    buf = torch.full((b * n + 1 + 512,), float("nan"), device="cuda")
    Xd = buf[1:1 + b * n].view(b, n)
    Xd.copy_(torch.from_numpy(X))
    guard = torch.full((b * m + 1 + 64,), 7.0, device="cuda")
    Y = guard[1:1 + b * m].view(b, m)
    plan = biq.biq_plan_check(m, n, q, b, 8, _plan(biq, q, 32, 2, 2, 2))
    ws = torch.empty(max(biq.biq_plan_workspace_bytes(plan, m, b), 16), dtype=torch.uint8, device="cuda")
    biq.biq_gemm_ex(gpu_pack(biq, Bd), ad, Xd, Y, m, n, q, b, 8, plan, workspace=ws)
    torch.cuda.synchronize()
    assert bool((guard[1 + b * m:] == 7.0).all()) and float(guard[0]) == 7.0
    ref = oracle.gemm_dense(B, alpha, X)
    assert np.all(np.abs(Y.cpu().numpy() - ref).max(axis=1) <= _bound(alpha, X))


@pytest.mark.parametrize("exponent", [-110, -120, -125, -128])
def test_digits_small_bf16_values(biq, oracle, exponent):
    """bf16 values near and below the smallest normal ones: the 16-bit form, whose even steps are summed at half their size."""
    import torch

    rng = np.random.default_rng(300 - exponent)
    m, n, q, b = 100, 1300, 2, 40
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32)
    X = (rng.standard_normal((b, n)) * 2.0 ** exponent).astype(np.float32)
    X = torch.from_numpy(X).bfloat16().float().numpy()
    Bd, ad, Xd = device_inputs(B, alpha, X)
    Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Xd, m, n, q, 8, plan=_plan(biq, q, 32, 6, 2, 2)).cpu().numpy()
    least = np.abs(alpha).sum(axis=0).max() * 16 * -(-n // 256) * 2.0 ** -148 + 2.0 ** -149
    assert np.all(np.abs(Y - oracle.gemm_dense(B, alpha, X)).max(axis=1) <= _bound(alpha, X) + least)


@pytest.mark.parametrize("m,n,q,b,bt,gps,ws,r", SHAPES)
@pytest.mark.parametrize("where", [0, -1])
def test_digits_one_key_group_in_the_other_form(biq, oracle, m, n, q, b, bt, gps, ws, r, where):
    """The first or the last key group in digits, all others in bf16, and the other way round."""
    import torch

    print("digits, one group", m, n, q, b, bt, gps, ws, r, where, flush=True)
    B, alpha, X = _inputs(m, n, q, b, 41000 + m + n)
    half = torch.from_numpy(X).bfloat16().float().numpy()
    groups = -(-n // 256)
    at = slice(0, 256) if where == 0 else slice((groups - 1) * 256, n)
    for base, other in ((half, X), (X, half)):
        Z = base.copy()
        Z[:, at] = other[:, at]
        Bd, ad, Zd = device_inputs(B, alpha, Z)
        Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Zd, m, n, q, 8, plan=_plan(biq, q, bt, gps, ws, r)).cpu().numpy()
        assert np.all(np.abs(Y - oracle.gemm_dense(B, alpha, Z)).max(axis=1) <= _bound(alpha, Z))


@pytest.mark.parametrize("b", [64, 37])
@pytest.mark.parametrize("where", ["first tile", "second tile", "NaN in the second"])
def test_digits_form_of_both_column_tiles(biq, oracle, b, where):
    """The two column tiles of a column group are prepared by different workgroups, which have to agree on its form:
    bf16 values but for one tile's last vector, or a NaN there."""
    import torch

    print("digits, column tiles", b, where, flush=True)
    m, n, q = 70, 601, 2
    B, alpha, X = _inputs(m, n, q, b, 43000 + b)
    full = X
    X = torch.from_numpy(X).bfloat16().float().numpy()
    v = 31 if where == "first tile" else b - 1
    if "NaN" not in where:
        X[v, 300:] = full[v, 300:]                       # the second and third key group
    Z = X.copy()
    if "NaN" in where:
        Z[v, n - 1] = np.nan
    Bd, ad, Zd = device_inputs(B, alpha, Z)
    Y = gpu_gemm(biq, gpu_pack(biq, Bd), ad, Zd, m, n, q, 8, plan=_plan(biq, q, 64, 3, 1, 2)).cpu().numpy()
    good = np.abs(Y - oracle.gemm_dense(B, alpha, X)).max(axis=1) <= _bound(alpha, X)
    if "NaN" in where:
        assert np.isnan(Y[v]).all() and good[np.arange(b) != v].all()
    else:
        assert good.all()
