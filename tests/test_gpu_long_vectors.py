"""GPU check of a step's second pass on long vectors (more than 2,048 slices, a
workgroup each, whose sums a kernel of their own finishes): coefficients and the
recomputed vector of two steps against the recurrence in torch.  Slices end at any row,
so their first and last rows go one by one.

Tolerances: sums of 1e7 products in FP64 1e-12 relative; FP32 rows 2e-6 of the row
sum of |H|, here 1e-5 of the largest entry."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N,A,precision,schedule", [
    (26, 12, "f64", None), (27, 12, "f64", (10, 256, 1, 2, 4)),
    (28, 11, "f32_mixed", (10, 256, 2, 2, 4)), (27, 13, "f32_mixed", (10, 256, 1, 2, 4))])
def test_two_steps(N, A, precision, schedule):
    from paper_0706_3293_amd import Basis, inputs
    print("long", N, A, precision, flush=True)
    b = Basis(N, two_s=1, two_M=N - 2 * A)
    if schedule:
        b.set_schedule(*schedule)
    J = inputs.ring_couplings(N, -1.1, -0.37)
    g = torch.Generator(device="cuda").manual_seed(N)
    v0 = torch.rand(b.dim, dtype=torch.float64, device="cuda", generator=g) - 0.4
    r = b.lanczos(J, v0, 2, precision=precision)
    c = np.array([0.6, 0.8])
    psi, alpha, beta = b.ritz(J, v0, 2, c, precision=precision)
    assert np.array_equal(alpha, r.alpha) and np.array_equal(beta, r.beta)

    v = v0 / v0.norm()
    w = b.apply(J, v)
    a0 = float(torch.dot(w, v))
    w -= a0 * v
    b0 = float(w.norm())
    u = w / b0
    w = b.apply(J, u) - b0 * v
    a1 = float(torch.dot(w, u))
    w -= a1 * u
    tol = 1e-12 if precision == "f64" else 1e-5
    scale = float(np.abs(np.triu(J)).sum())
    assert np.abs(r.alpha - [a0, a1]).max() <= tol * scale
    assert np.abs(r.beta[:2] - [b0, float(w.norm())]).max() <= tol * scale
    ref = 0.6 * v + 0.8 * u
    ref /= ref.norm()
    assert float((psi - ref).abs().max()) <= 10 * tol * float(ref.abs().max())
    b.free()
