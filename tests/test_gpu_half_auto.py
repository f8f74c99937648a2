"""GPU checks of the spin-1/2 block kernel's automatic FP64 split: staged blocks in
large, well-filled subspaces, the handle's split below and beside them and in FP32."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (N, A, staged): rows from 497,420 (too few) to 7.7 M; 57 (not taken), 106, 123
# and 165 rows per block; spin up and down sides of a sector
@pytest.mark.parametrize("N,A,staged", [(22, 9, False), (23, 11, True), (24, 8, False),
                                        (24, 14, True), (25, 10, False), (26, 11, True)])
@pytest.mark.parametrize("kind", ["ring", "all"])
def test_automatic_schedule(N, A, staged, kind):
    """The automatic split gives the rows of a chunked schedule with its low sites bit
    for bit, and those of the generic kernel within rounding (2^-53 times a few
    hundred terms of the largest row sum); FP32 products keep the handle's split."""
    from paper_0706_3293_amd import Basis, inputs
    print("half auto", N, A, kind, flush=True)
    J = inputs.ring_couplings(N, -1.1, -0.37) if kind == "ring" else \
        inputs.all_to_all_couplings(N, 1)[0]
    b = Basis(N, two_s=1, two_M=N - 2 * A)
    same = Basis(N, two_s=1, two_M=N - 2 * A)
    if staged:
        same.set_schedule(10, 256, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda", generator=g) - 0.5
    scale = float(np.abs(J).sum() / 2)
    y = b.apply(J, x)
    assert torch.equal(y, same.apply(J, x, kernel=2))
    assert float((y - b.apply(J, x, kernel=1)).abs().max()) <= 1e-13 * scale
    v = x.float()
    assert torch.equal(b.apply(J, v), b.apply(J, v, kernel=2))
    z = b.lanczos(J, x, 3).alpha - b.lanczos(J, x, 3, kernel=1).alpha
    assert np.abs(z).max() <= 1e-12 * scale
