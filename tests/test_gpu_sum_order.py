"""GPU checks that the order of a run's sums does not depend on the kernels that the
automatic choice takes.  A Lanczos run without reorthogonalization amplifies the
last bit of its sums once the extreme Ritz values have converged (to 1e-8 of dE0/dJ
in 200 steps), so coefficients are compared bit for bit with the kernels asked for
by number, and gradients of such runs with stored ones."""
import json
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "gradient_past_convergence.json")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _couplings(N, kind):
    from paper_0706_3293_amd import inputs
    if kind == "all":
        return inputs.all_to_all_couplings(N, 1)[0]
    if kind == "far":
        J = inputs.ring_couplings(N, -1.03)
        J[0, N - 1] = J[N - 1, 0] = 0.7
        J[1, N - 2] = J[N - 2, 1] = 0.3
        return J
    return inputs.ring_couplings(N, -1.03, -0.37)


# spin 1/2: one block (12 sites), chains of 14, 6 and 3 items of a wave (14, 15, 16
# sites), one or two (17 on), sectors with short blocks, vectors of 64 and more
# workgroups, pass B in groups (21 sites) and over the fold's limit (24 sites, FP32)
HALF = [(12, 6, "all"), (13, 4, "ring"), (14, 7, "ring"), (14, 7, "all"), (15, 7, "far"),
        (15, 8, "ring"), (16, 8, "ring"), (16, 8, "all"), (16, 5, "all"), (17, 8, "ring"),
        (17, 8, "all"), (18, 9, "all"), (20, 10, "all"), (20, 10, "ring"), (24, 5, "all"),
        (21, 10, "ring"), (22, 11, "far")]


@pytest.mark.parametrize("N,A,kind", HALF)
@pytest.mark.parametrize("precision", ["f64", "f32_mixed"])
def test_half_spin_run_has_the_bits_of_the_block_kernel(N, A, kind, precision):
    from paper_0706_3293_amd import Basis, inputs
    print("sum order", N, A, kind, precision, flush=True)
    b = Basis(N, two_s=1, two_M=N - 2 * A)
    J = _couplings(N, kind)
    v = torch.tensor(inputs.start_vector(b.dim, 1), device="cuda")
    r = b.lanczos(J, v, 40, precision=precision)
    q = b.lanczos(J, v, 40, precision=precision, kernel=2)
    assert np.array_equal(r.alpha, q.alpha) and np.array_equal(r.beta, q.beta)
    x = v if precision == "f64" else v.float()
    assert torch.equal(b.apply(J, x), b.apply(J, x, kernel=2))


# s >= 1: 1,107 to 488,187 rows, one lane per row
GENERAL = [(8, 2, 8, "ring"), (8, 2, 8, "all"), (9, 2, 9, "ring"), (11, 2, 11, "all"),
           (8, 3, 12, "ring"), (6, 4, 12, "all"), (6, 5, 14, "far"), (14, 2, 11, "ring")]


@pytest.mark.parametrize("N,two_s,A,kind", GENERAL)
@pytest.mark.parametrize("precision", ["f64", "f32_mixed"])
def test_general_spin_run_has_the_bits_of_the_generic_kernel(N, two_s, A, kind, precision):
    from paper_0706_3293_amd import Basis, inputs
    print("sum order", N, two_s, A, kind, precision, flush=True)
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = _couplings(N, kind)
    v = torch.tensor(inputs.start_vector(b.dim, 1), device="cuda")
    r = b.lanczos(J, v, 40, precision=precision)
    q = b.lanczos(J, v, 40, precision=precision, kernel=1)
    assert np.array_equal(r.alpha, q.alpha) and np.array_equal(r.beta, q.beta)
    x = v if precision == "f64" else v.float()
    assert torch.equal(b.apply(J, x), b.apply(J, x, kernel=1))


@pytest.mark.parametrize("case", range(6))
def test_gradient_past_convergence(case):
    """The stored gradients come from the same coefficients bit for bit, so what is
    left is the rounding of the correlations' own sums: 2^-53 times a few hundred
    terms of a thread."""
    from paper_0706_3293_amd import Basis, ground_state_energy, inputs
    g = json.load(open(GOLDEN))["cases"][case]
    N, two_s = g["N"], g["two_s"]
    b = Basis(N, two_s=two_s, two_M=N * two_s % 2)
    _, bonds, vals = inputs.all_to_all_couplings(N, g["seed"])
    v0 = torch.tensor(inputs.start_vector(b.dim, g["seed"]), device="cuda")
    Jv = torch.tensor(vals, dtype=torch.float64, requires_grad=True)
    E0 = ground_state_energy(Jv, b, bonds, v0, g["steps"])
    E0.backward()
    grad, ref = Jv.grad.numpy(), np.array(g["grad"])
    off = np.linalg.norm(grad - ref) / np.linalg.norm(ref)
    print(f"{N} sites, 2s = {two_s}: {off:.1e}", flush=True)
    assert float(E0) == g["E0"]
    assert off <= 1e-13
