"""GPU checks of the spin-1/2 kernel with one workgroup per block (the automatic
choice in FP64 for small subspaces) against the oracle, the edges of its range
included: few sites, blocks of one row, odd N, every kind of bond, and the calls
whose kernel it changes.  Tolerance: the suite's 1e-13 of the largest row sum."""
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
    if kind == "far":
        J = np.zeros((N, N))
        J[0, N - 1] = J[N - 1, 0] = 0.7
        return J
    if kind == "none":
        return np.zeros((N, N))
    return inputs.all_to_all_couplings(N, 1)[0]


@pytest.mark.parametrize("N,A", [(4, 2), (5, 2), (6, 0), (6, 1), (9, 4), (12, 6), (13, 6), (16, 8),
                                 (16, 3), (17, 8), (18, 9), (19, 7), (20, 10)])
@pytest.mark.parametrize("kind", ["ring", "far", "none", "all"])
def test_rows_match_oracle(N, A, kind):
    import oracle
    from paper_0706_3293_amd import Basis
    print("half wg", N, A, kind, flush=True)
    b = Basis(N, two_s=1, two_M=N - 2 * A)
    J = _couplings(N, kind)
    x = np.random.default_rng(A).uniform(-1, 1, b.dim)
    y = b.apply(J, torch.tensor(x, device="cuda")).cpu().numpy()
    ref = oracle.Subspace(N, 1, A).apply(J, x)
    assert np.abs(y - ref).max() <= 1e-13 * (np.abs(np.triu(J)).sum() + 1.0)


@pytest.mark.parametrize("kind", ["ring", "all"])
def test_step_kernels_agree(kind):
    """Coefficients of a run on this kernel and on the block kernel asked for by
    number: the same sums in another order, 20 steps before convergence."""
    from paper_0706_3293_amd import Basis
    b = Basis(16, two_s=1, two_M=0)
    J = _couplings(16, kind)
    v = torch.tensor(np.random.default_rng(0).uniform(-1, 1, b.dim), device="cuda")
    for reorth in (False, True):
        r = b.lanczos(J, v, 20, full_reorth=reorth)
        q = b.lanczos(J, v, 20, full_reorth=reorth, kernel=2)
        assert np.abs(r.alpha - q.alpha).max() <= 1e-11
        assert np.abs(r.beta - q.beta).max() <= 1e-11


def test_calls_around_the_tables():
    """A product captured before its tables exist, a schedule asked for before
    and after the first use, and FP32 on the same handle."""
    from paper_0706_3293_amd import Basis, _lib
    J = _couplings(14, "ring")
    b = Basis(14, two_s=1, two_M=0)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda")
    ref = b.apply(J, x, kernel=1)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.apply(J, x, out=y)
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert float((y - ref).abs().max()) <= 1e-12
    assert float((b.apply(J, x) - ref).abs().max()) <= 1e-12
    assert float((b.apply(J, x.float()).double() - ref).abs().max()) <= 1e-4
    with pytest.raises(_lib.HMError):
        b.set_schedule(8, 256, 1)
    c = Basis(14, two_s=1, two_M=0)
    c.set_schedule(8, 256, 1)
    assert float((c.apply(J, x) - ref).abs().max()) <= 1e-12
