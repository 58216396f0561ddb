"""GPU parity of the direct kernel (plans with table_fill = 2: few input vectors, digits in LDS, no tables) at the edges
of its row steps, chunks, column tiles and wave groups, against the CPU oracle."""
import numpy as np
import pytest

from gpu_util import assert_within_tolerance, device_inputs, gpu_pack
from test_direct_rule import WIDE_ROWS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def biq():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_09904_amd as biq

    biq.load_library()
    return biq


def _bound(alpha, X):
    """Per input vector.  Split: each element is off by at most u = 2^-24 of the largest of its 32 neighbours.  Sums: a
    digit's column is rounded at most once per 128 elements and its magnitude is 2^-5 per digit; then at most 24
    roundings over digits, planes, scales and wave groups: u * ||x||_1 each."""
    b, n = X.shape
    A = np.zeros((b, -(-n // 32) * 32))
    A[:, :n] = np.abs(X)
    split = 32 * A.reshape(b, -1, 32).max(axis=2).sum(axis=1)
    return 2.0 ** -24 * np.abs(alpha).sum(axis=0).max() * (split + A.sum(axis=1) * (1.04 * -(-n // 128) + 24))


def _direct(biq, B, alpha, X, mu=8):
    import torch

    q, m, n = B.shape
    b = X.shape[0]
    Bd, ad, _ = device_inputs(B, alpha, X)
    buf = torch.full((b * n + 1 + 64,), float("nan"), device="cuda")      # odd float addresses, nothing behind the end
    Xd = buf[1:1 + b * n].view(b, n)
    Xd.copy_(torch.from_numpy(X))
    guard = torch.full((b * m + 1 + 64,), 7.0, device="cuda")
    Y = guard[1:1 + b * m].view(b, m)
    plan = biq.biq_plan_get_lut(m, n, q, b, mu)
    plan.table_fill = 2
    plan = biq.biq_plan_check(m, n, q, b, mu, plan)
    ws = torch.empty(max(biq.biq_plan_workspace_bytes(plan, m, b), 16), dtype=torch.uint8, device="cuda")
    biq.biq_gemm_ex(gpu_pack(biq, Bd, mu), ad, Xd, Y, m, n, q, b, mu, plan, workspace=ws)
    torch.cuda.synchronize()
    assert bool((guard[1 + b * m:] == 7.0).all()) and float(guard[0]) == 7.0
    return Y.cpu().numpy()


SHAPES = [
    # m, n, q, batch, mu
    (1, 1, 1, 1, 8), (15, 31, 4, 2, 8), (16, 512, 1, 3, 8), (17, 513, 2, 4, 8), (129, 1025, 3, 7, 6), (500, 130, 2, 15, 8),
    (333, 2049, 4, 10, 8), (100, 4096, 1, 16, 4), (260, 1500, 3, 31, 7), (64, 9000, 2, 9, 8),     # several batch tiles
    (40, 20000, 2, 2, 8), (9, 38900, 1, 1, 8),                                                     # widest rows
    (33000, 100, 1, 1, 8), (33001, 600, 1, 5, 8), (16500, 300, 2, 7, 1), (33000, 520, 1, 11, 8),   # many rows
    (33001, 1100, 2, 1, 8), (20000, 200, 4, 13, 8), (17000, 700, 3, 2, 8), (40000, 257, 2, 3, 8),  # ... two steps each
]


@pytest.mark.parametrize("m,n,q,b,mu", SHAPES)
def test_direct_parity(biq, oracle, m, n, q, b, mu):
    print("direct", m, n, q, b, mu, flush=True)
    rng = np.random.default_rng(52000 + m + n + b)
    X = rng.standard_normal((b, n), dtype=np.float32)
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32)
    Y = _direct(biq, B, alpha, X, mu)
    rows = np.arange(m) if m <= 2000 else np.unique(np.r_[0:200, m // 2 - 100:m // 2 + 100, m - 200:m])
    ref = oracle.gemm_dense(B[:, rows], alpha[:, rows], X)
    assert np.isfinite(Y).all()
    assert_within_tolerance(Y[:, rows], ref, alpha[:, rows], X, "direct")
    assert np.all(np.abs(Y[:, rows] - ref).max(axis=1) <= _bound(alpha[:, rows], X))


@pytest.mark.parametrize("m,n,q", [w[:3] for w in WIDE_ROWS])
def test_one_vector_on_wide_rows(biq, oracle, m, n, q):
    """The mappings of one vector beyond the table workgroups' rows: against the oracle, and against the table kernels."""
    import torch

    print("wide rows", m, n, q, flush=True)
    rng = np.random.default_rng(53000 + m + n)
    X = rng.standard_normal((1, n), dtype=np.float32)
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32)
    Y = _direct(biq, B, alpha, X)
    rows = np.unique(np.r_[0:min(m, 200), max(0, m // 2 - 100):min(m, m // 2 + 100), max(0, m - 200):m])
    ref = oracle.gemm_dense(B[:, rows], alpha[:, rows], X)
    assert_within_tolerance(Y[:, rows], ref, alpha[:, rows], X, "wide rows")
    assert np.all(np.abs(Y[:, rows] - ref).max(axis=1) <= _bound(alpha[:, rows], X))
    # every row against the table kernels: both are within the bound, theirs rounds each of n / 8 partial sums
    Bd, ad, Xd = device_inputs(B, alpha, X)
    plan = biq.biq_plan_get_lut(m, n, q, 1, 8)
    ws = torch.empty(max(biq.biq_plan_workspace_bytes(plan, m, 1), 16), dtype=torch.uint8, device="cuda")
    T = torch.empty((1, m), device="cuda")
    biq.biq_gemm_ex(gpu_pack(biq, Bd, 8), ad, Xd, T, m, n, q, 1, 8, plan, workspace=ws)
    limit = _bound(alpha, X) + 2.0 ** -24 * np.abs(alpha).sum(axis=0).max() * np.abs(X).sum() * (-(-n // 8) + 24)
    assert np.abs(Y - T.cpu().numpy()).max() <= limit[0]


def test_direct_special_values(biq, oracle):
    """Exact inputs bit for bit; wide dynamic range within the bound; zeros; Inf and NaN stay in their vector."""
    from paper_2005_09904_amd.workloads import Workload, make_exact_inputs

    for (m, n, q, b) in [(300, 2100, 2, 1), (129, 1000, 3, 4), (40000, 64, 1, 2)]:
        B, alpha, X = make_exact_inputs(Workload("exact", m, n, q, b, 8, "uniform", seed=90 + b))
        assert np.array_equal(_direct(biq, B, alpha, X).astype(np.float64), oracle.gemm_dense(B, alpha, X))
    rng = np.random.default_rng(7)
    B = (rng.integers(0, 2, size=(2, 200, 1200), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(2, 200)).astype(np.float32)
    X = rng.standard_normal((7, 1200))
    X[1] *= 10.0 ** rng.uniform(-9, 3, size=1200)
    X[2] *= 2.0 ** -100
    X[3] *= 2.0 ** 110
    X[4] = 0.0
    X = X.astype(np.float32)
    Y = _direct(biq, B, alpha, X)
    assert np.all(np.abs(Y - oracle.gemm_dense(B, alpha, X)).max(axis=1) <= _bound(alpha, X)) and np.all(Y[4] == 0.0)
    X[0, 7], X[5, 1199] = np.nan, -np.inf
    Z = _direct(biq, B, alpha, X)
    assert np.isnan(Z[[0, 5]]).all() and np.array_equal(Z[[1, 2, 3, 4, 6]], Y[[1, 2, 3, 4, 6]])


def test_direct_most_rows(biq):
    """2^30 rows, the most the kernel takes: 4 GiB of scales.  Rows at both ends and where byte offsets of scales and keys
    pass 2^31 and 2^32, against a product in 64 bits."""
    import torch

    m, n, b = 1 << 30, 20, 2
    need = 16 * m + 4 * m + 4 * m * b
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("needs %d GiB of device memory" % (need >> 30))
    print("direct", m, n, b, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(30)
    K = torch.zeros((m, 16), dtype=torch.uint8, device="cuda")
    K[:, :3] = torch.randint(0, 256, (m, 3), dtype=torch.uint8, device="cuda", generator=g)
    K[:, 2] &= 15
    alpha = torch.rand((1, m), device="cuda", generator=g) + 0.5
    X = torch.randn((b, n), device="cuda", generator=g)
    Y = torch.full((b, m), float("nan"), device="cuda")
    plan = biq.biq_plan_get_lut(m, n, 1, b, 8)
    plan.table_fill = 2
    plan = biq.biq_plan_check(m, n, 1, b, 8, plan)
    ws = torch.empty(max(biq.biq_plan_workspace_bytes(plan, m, b), 16), dtype=torch.uint8, device="cuda")
    biq.biq_gemm_ex(K, alpha, X, Y, m, n, 1, b, 8, plan, workspace=ws)
    torch.cuda.synchronize()
    assert not bool(torch.isnan(Y).any())
    bits = torch.arange(8, dtype=torch.uint8, device="cuda")
    for first in (0, (1 << 27) - 500, (1 << 28) - 500, (1 << 29) - 500, m - 1000):
        rows = slice(first, first + 1000)
        s = ((K[rows, :3, None] >> bits) & 1).reshape(1000, 24)[:, :n].double() * 2 - 1
        ref = (X.double() @ s.t()) * alpha[:, rows].double()
        bound = _bound(np.ones((1, 1)), X.cpu().numpy())                       # per vector, for a scale of 1
        assert bool(((Y[:, rows].double() - ref).abs() <= torch.tensor(bound, device="cuda")[:, None] * alpha[:, rows]).all())


@pytest.mark.parametrize("exponent", [-105, -110, -118, -126, -135])
def test_direct_small_inputs(biq, oracle, exponent):
    """Vectors far below one keep their bits: the bound relative to the elements, and what the kernel's sums are rounded to
    where they are subnormal (they are formed at 2^-6 of their size: 2^-143 for each instruction of a row)."""
    rng = np.random.default_rng(700 - exponent)
    m, n, q, b = 200, 1200, 2, 7
    B = (rng.integers(0, 2, size=(q, m, n), dtype=np.int8) * 2 - 1).astype(np.int8)
    alpha = rng.uniform(0.05, 1.0, size=(q, m)).astype(np.float32)
    X = rng.standard_normal((b, n))
    X[::3] *= 2.0 ** exponent
    X[1::3] *= 2.0 ** exponent * 10.0 ** rng.uniform(-3, 3, size=n)
    X[2] *= 2.0 ** 100                                  # a large vector among them changes nothing
    X = X.astype(np.float32)
    Y = _direct(biq, B, alpha, X)
    least = np.abs(alpha).sum(axis=0).max() * (-(-n // 128) + 2) * 1.04 * 2.0 ** -143
    assert np.all(np.abs(Y - oracle.gemm_dense(B, alpha, X)).max(axis=1) <= _bound(alpha, X) + least)


def test_direct_largest_inputs(biq, oracle):
    """The largest fp32 alone in a vector comes back as it is; sums below it do not overflow, nor do the sums of
    later digits, whatever their signs."""
    top = np.finfo(np.float32).max
    m, n = 40, 1500
    B = np.ones((1, m, n), dtype=np.int8)
    B[0, ::2] = -1
    alpha = np.full((1, m), 0.5, dtype=np.float32)
    X = np.zeros((4, n), dtype=np.float32)
    X[0, 5], X[1, 1499] = top, -top
    X[2] = top / np.float32(1550.0)
    X[3, ::32] = top / np.float32(100.0)
    X[3, X[3] == 0] = top / np.float32(100.0 * 32.1)     # a digit below the largest of the block
    Y = _direct(biq, B, alpha, X)
    ref = oracle.gemm_dense(B, alpha, X)
    assert np.isfinite(Y).all()
    assert np.array_equal(Y[:2].astype(np.float64), ref[:2])
    assert np.all(np.abs(Y - ref).max(axis=1) <= _bound(alpha, X))
