"""GPU checks of the block kernel for s >= 1 (the automatic choice of Basis.apply
there) against the oracle and the generic digit kernel: short blocks (one lane
per row) and long ones (a wave per group of blocks), 64-bit indices, couplings
with every kind of bond and with none, and inputs that are not finite.

Tolerances are those of the suite's other H x checks: FP64 1e-13 and FP32 2e-6
of the largest row sum of |H| times the largest |x|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _couplings(N, kind):
    from paper_0706_3293_amd import inputs
    if kind == "ring":
        return inputs.ring_couplings(N, -1.1, -0.37)
    if kind == "chain":
        return inputs.chain_couplings(np.random.default_rng(N).normal(-1.0, 0.3, N - 1))
    if kind == "far":                     # one bond between the end sites
        J = np.zeros((N, N))
        J[0, N - 1] = J[N - 1, 0] = 0.7
        return J
    if kind == "none":
        return np.zeros((N, N))
    return inputs.all_to_all_couplings(N, 1)[0]


def _scale(J, two_s):
    return np.abs(np.triu(J)).sum() * two_s * (two_s + 2) / 4 + 1.0


# one lane per row: fewer than 2^20 rows, or sectors with short blocks
@pytest.mark.parametrize("N,two_s,A", [(2, 2, 2), (2, 15, 15), (3, 15, 20), (5, 4, 10), (8, 2, 3),
                                       (9, 3, 13), (4, 7, 14), (7, 2, 0), (7, 2, 14), (12, 2, 12),
                                       (6, 5, 14)])
@pytest.mark.parametrize("kind", ["ring", "chain", "far", "none", "all"])
def test_rows_match_oracle(N, two_s, A, kind):
    import oracle
    from paper_0706_3293_amd import Basis
    if kind != "none" and N == 2 and kind != "far":
        pytest.skip("two sites have one bond")
    print("digit", N, two_s, A, kind, flush=True)
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = _couplings(N, kind)
    x = np.random.default_rng(A).uniform(-1, 1, b.dim)
    ref = oracle.Subspace(N, two_s, A).apply(J, x)
    s = _scale(J, two_s)
    for dt, tol in ((torch.float64, 1e-13), (torch.float32, 2e-6)):
        xd = torch.tensor(x, device="cuda").to(dt)
        y = b.apply(J, xd)
        if dt == torch.float32:                   # the generic kernel's roundings
            assert torch.equal(y, b.apply(J, xd, kernel=1))
        y = y.double().cpu().numpy()
        assert np.abs(y - ref).max() <= tol * s


# a wave per group of blocks (1.3 to 1.8 M rows), sampled rows
@pytest.mark.parametrize("N,two_s,A", [(15, 2, 14), (15, 2, 15), (12, 3, 18), (12, 3, 15)])
@pytest.mark.parametrize("kind", ["ring", "all"])
def test_long_blocks_match_oracle_and_generic_kernel(N, two_s, A, kind):
    import oracle
    from paper_0706_3293_amd import Basis
    print("digit blocks", N, two_s, A, kind, flush=True)
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = _couplings(N, kind)
    x = np.random.default_rng(A).uniform(-1, 1, b.dim)
    rows = np.sort(np.random.default_rng(7).integers(0, b.dim, 20000))
    rows[:2] = 0, b.dim - 1
    ref = oracle.Subspace(N, two_s, A).apply_rows(J, x, rows)
    s = _scale(J, two_s)
    for dt, tol in ((torch.float64, 1e-13), (torch.float32, 2e-6)):
        xd = torch.tensor(x, device="cuda").to(dt)
        y = b.apply(J, xd)
        assert np.abs(y.double().cpu().numpy()[rows] - ref).max() <= tol * s
        assert float((y - b.apply(J, xd, kernel=1)).abs().max()) <= tol * s
        if dt == torch.float32:                   # the generic kernel's roundings
            assert torch.equal(y, b.apply(J, xd, kernel=1))


def test_64_bit_indices_match_generic_kernel():
    """N = 21, s = 1 (1,105,350,729 rows): byte offsets beyond 4 GiB."""
    from paper_0706_3293_amd import Basis
    b = Basis(21, two_s=2, two_M=0)
    assert b.dim > 1 << 30
    J = _couplings(21, "ring")
    x = torch.rand(b.dim, dtype=torch.float32, device="cuda",
                   generator=torch.Generator(device="cuda").manual_seed(1)).sub_(0.5)
    y = b.apply(J, x)
    y -= b.apply(J, x, kernel=1)
    assert float(y.abs().max()) <= 2e-6 * _scale(J, 2)


@pytest.mark.parametrize("N,two_s,A", [(9, 2, 9), (15, 2, 15)])
def test_values_that_are_not_finite_reach_the_same_rows(N, two_s, A):
    """A move that is not allowed reads nothing: rows without a path to the
    infinite or NaN entries stay finite, as with the generic kernel."""
    from paper_0706_3293_amd import Basis
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = _couplings(N, "ring")
    for dt in (torch.float64, torch.float32):
        x = torch.rand(b.dim, dtype=dt, device="cuda")
        for i, v in ((0, np.inf), (b.dim // 3, -np.inf), (b.dim // 2, np.nan), (b.dim - 1, np.inf)):
            x[i] = v
        y, y1 = b.apply(J, x), b.apply(J, x, kernel=1)
        assert torch.equal(torch.isnan(y), torch.isnan(y1))
        assert torch.equal(y[torch.isinf(y)], y1[torch.isinf(y1)])


def test_product_captured_before_its_tables_exist():
    """A graph capture cannot allocate: the generic kernel is captured then."""
    from paper_0706_3293_amd import Basis
    b = Basis(9, two_s=2, two_M=0)
    J = _couplings(9, "ring")
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda")
    ref = b.apply(J, x, kernel=1)                 # couplings uploaded, no tables
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.apply(J, x, out=y)
    for k in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
    again = b.apply(J, x)
    assert float((again - ref).abs().max()) <= 1e-13 * _scale(J, 2)
