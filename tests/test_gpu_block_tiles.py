"""GPU checks of the block recurrence's matrix-core dot products where their
tiles end: rows that do not fill a step of a workgroup (64 or 128 rows), column
counts beyond one tile (32 for p = 1, else 64) and a run that stops after the
host has enqueued further steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (N, two_s, A, p, steps): dims 8, 10, 70, 924, 462, 252, 924, 141
@pytest.mark.parametrize("N,two_s,A,p,steps", [
    (8, 1, 1, 1, 3), (5, 1, 2, 2, 2), (8, 1, 4, 16, 3), (12, 1, 6, 1, 36), (11, 1, 5, 2, 34),
    (10, 1, 5, 16, 6), (12, 1, 6, 8, 10), (6, 2, 6, 4, 18)])
def test_dots_at_tile_edges_match_oracle(N, two_s, A, p, steps):
    """Coefficients against the oracle's recurrence; 1e-10 of the largest entry
    is the bound of the suite's other block runs (FP64, well-conditioned steps:
    open chains with random couplings have no degenerate levels)."""
    import oracle
    from oracle import block
    from paper_0706_3293_amd import Basis, inputs
    print("block tiles", N, two_s, A, p, steps, flush=True)
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    sub = oracle.Subspace(N, two_s, A)
    J = inputs.chain_couplings(np.random.default_rng(N).normal(-1.0, 0.3, N - 1))
    X0 = np.random.default_rng(N + p).uniform(-1, 1, (b.dim, p))
    Ag, Bg, k = b.block_lanczos(J, torch.tensor(X0, device="cuda"), steps)
    Ao, Bo, _ = block.block_lanczos(sub, J, X0, steps)
    assert k == len(Ao)
    scale = np.abs(Ao).max()
    assert np.abs(Ag - Ao).max() <= 1e-10 * scale
    assert np.abs(Bg[: k - 1] - Bo[: k - 1]).max() <= 1e-10 * scale


def test_run_that_stops_early_gives_the_full_spectrum():
    """70 states, blocks of 2, 60 steps asked for: the space is exhausted after
    35 steps, past two looks at the stop flag, and the block tridiagonal matrix
    then holds every level (70 is a multiple of 2: a run stops at the first
    rank-deficient block, there is no deflation)."""
    import oracle
    from paper_0706_3293_amd import Basis, inputs
    from paper_0706_3293_amd.api import block_tridiag_eigenvalues
    N = 8
    b = Basis(N, two_s=1, two_M=0)
    sub = oracle.Subspace(N, 1, 4)
    J = inputs.chain_couplings(np.random.default_rng(3).normal(-1.0, 0.3, N - 1))
    H = np.column_stack([sub.apply(J, e) for e in np.eye(b.dim)])
    levels = np.linalg.eigvalsh(H)
    X0 = np.random.default_rng(4).uniform(-1, 1, (b.dim, 2))
    A, B, k = b.block_lanczos(J, torch.tensor(X0, device="cuda"), 60)
    assert k == 35
    got = block_tridiag_eigenvalues(A, B)
    for e in levels:
        assert np.abs(got - e).min() <= 1e-9 * np.abs(levels).max()
