"""GPU checks of the block kernel for s >= 1 with couplings whose matrix elements
leave FP32, and of where infinite and NaN inputs end up: the same rows as with the
generic kernel, value for value."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _same(y, z):
    assert torch.equal(torch.isnan(y), torch.isnan(z))
    assert torch.equal(torch.isinf(y), torch.isinf(z))
    at = torch.isinf(y)
    assert torch.equal(y[at], z[at])


# one lane per row, and a wave per group of blocks
@pytest.mark.parametrize("N,two_s,A", [(8, 2, 8), (5, 3, 7), (15, 2, 15)])
@pytest.mark.parametrize("J1", [8e38, 1.3e39, 4e39])
def test_couplings_beyond_fp32(N, two_s, A, J1):
    """-J/2 infinite in FP32 (and -J/4 too in the last): a row is infinite or NaN
    where an allowed term makes it so."""
    from paper_0706_3293_amd import Basis, inputs
    print("overflow", N, two_s, A, J1, flush=True)
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = np.zeros((N, N))
    for u, v in ((0, 1), (0, N - 1), (N - 2, N - 1)):     # low, straddling, high
        J[u, v] = J[v, u] = J1
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.rand(b.dim, dtype=torch.float32, device="cuda", generator=g) * 1e-3
    y = b.apply(J, x)
    _same(y, b.apply(J, x, kernel=1))


@pytest.mark.parametrize("N,two_s,A", [(9, 2, 9), (7, 4, 14), (15, 2, 15)])
@pytest.mark.parametrize("kind", ["ring", "all"])
def test_infinite_and_nan_entries(N, two_s, A, kind):
    from paper_0706_3293_amd import Basis, inputs
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    J = inputs.ring_couplings(N, -1.1, -0.37) if kind == "ring" else \
        inputs.all_to_all_couplings(N, 1)[0]
    for dt in (torch.float64, torch.float32):
        x = torch.rand(b.dim, dtype=dt, device="cuda")
        for i, v in ((0, np.inf), (b.dim // 3, -np.inf), (b.dim // 2, np.nan),
                     (b.dim - 1, np.inf)):
            x[i] = v
        _same(b.apply(J, x), b.apply(J, x, kernel=1))
