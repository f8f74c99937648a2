"""GPU checks of the one-workgroup Lanczos launches on tabulated moves (the
automatic choice for up to 3,072 rows) and of the hand-over to the multi-kernel
step in long reorthogonalized runs, against the multi-kernel step alone."""
from math import comb

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")

# (N, 2s, A): rows of a thread 1, 1 and 2, 3 with a remainder; 1 to 15 bits of
# spin; 2,304 rows and more hand over after 42 (FP64) steps or fewer; 3,432 rows
# take no such launch
CASES = [(3, 1, 1), (14, 1, 4), (46, 1, 2), (12, 1, 6), (18, 1, 4), (14, 1, 7), (8, 2, 8),
         (5, 5, 12), (4, 15, 30)]


@pytest.mark.parametrize("N,two_s,A", CASES)
@pytest.mark.parametrize("precision", ["f64", "f32_mixed"])
@pytest.mark.parametrize("reorth", [False, True])
def test_table_run_matches_multi_kernel_run(N, two_s, A, precision, reorth):
    """alpha and beta before the rounding is amplified, E0, the ground state, and
    the same coefficients again, also with a graph asked for.  Tolerances: 15
    steps of rounding (2^-53 and 2^-24, amplified by the recurrence) leave
    1e-10 and 2e-6."""
    from paper_0706_3293_amd import Basis, inputs
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = inputs.ring_couplings(N, -1.0, -0.37 if N > 4 else 0.0)
    v0 = torch.tensor(inputs.start_vector(b.dim, 1), device="cuda")
    print("table run", N, two_s, A, precision, reorth, flush=True)
    steps = min(60, b.dim)
    opt = dict(precision=precision, full_reorth=reorth)
    r0 = b.lanczos(J, v0, steps, **opt)
    r1 = b.lanczos(J, v0, steps, kernel=2 if two_s == 1 and N <= 32 else 1, **opt)
    tol = 1e-10 if precision == "f64" else 2e-6
    n = min(15, r0.steps_done, r1.steps_done)
    scale = np.abs(r1.alpha).max()
    assert np.abs(r0.alpha[:n] - r1.alpha[:n]).max() <= tol * scale
    assert np.abs(r0.beta[:n - 1] - r1.beta[:n - 1]).max(initial=0.0) <= tol * scale
    assert abs(r0.E0 - r1.E0) <= tol * abs(r1.E0)
    g = b.lanczos(J, v0, steps, use_graph=True, **opt)
    assert np.array_equal(g.alpha, r0.alpha) and np.array_equal(g.beta, r0.beta)
    # the recompute pass runs the same kernels, so it repeats the coefficients, and
    # its vector has the energy of the tridiagonal matrix
    k = r0.steps_done
    T = np.diag(r0.alpha) + np.diag(r0.beta[:k - 1], 1) + np.diag(r0.beta[:k - 1], -1)
    c = np.linalg.eigh(T)[1][:, 0]
    psi, alpha, beta = b.ritz(J, v0, k, c, **opt)
    assert np.array_equal(alpha, r0.alpha) and np.array_equal(beta, r0.beta)
    assert abs(float(psi @ psi) - 1.0) < 1e-12
    assert abs(float(psi @ b.apply(J, psi)) - r0.E0) <= 100 * tol * abs(r0.E0)


@pytest.mark.parametrize("N,two_s,A", [(12, 1, 6), (8, 2, 8)])
def test_table_run_stops_at_breakdown(N, two_s, A):
    """A start vector in a small invariant subspace: the sector's uniform vector
    is an eigenvector of a ring with equal couplings, so the run ends after one
    step."""
    from paper_0706_3293_amd import Basis, inputs
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = inputs.ring_couplings(N, -1.0)
    w = [np.prod([comb(two_s, int(d)) for d in b.unrank(i)]) for i in range(b.dim)]
    v0 = torch.tensor(np.sqrt(np.array(w, dtype=np.float64)), device="cuda")
    for reorth in (False, True):
        r = b.lanczos(J, v0, 20, full_reorth=reorth, tol=1e-10)
        assert r.steps_done == 1
