"""GPU checks of the batched H x: rows with more allowed moves than a list holds,
every vector width, partial waves and items, and a batch long enough for two
items per chunk."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("nvec", [1, 2, 4, 8, 16])
def test_long_and_short_rows_vs_oracle(nvec):
    """All-to-all and single-bond couplings, dimensions 1 to 1,107 around the 64
    rows of a wave and the 256 of an item.  Tolerance: 1e-5 of the largest
    coefficient, 2^-24 amplified over 8 steps and up to 120 moves a row."""
    import oracle
    from paper_0706_3293_amd import Basis, inputs, lanczos_batched
    print("batched lists", nvec, flush=True)
    rng = np.random.default_rng(nvec)
    specs = [(12, 1, 6, "all"), (6, 3, 9, "all"), (7, 2, 7, "all"), (8, 2, 8, "one"),
             (5, 2, 0, "all"), (8, 1, 3, "all"), (11, 1, 2, "all"), (4, 7, 14, "all"),
             (10, 1, 5, "all")]
    bases, Js, V0s = [], [], []
    for N, two_s, A, kind in specs:
        b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
        J = inputs.all_to_all_couplings(N, 1)[0] if kind == "all" else np.zeros((N, N))
        if kind == "one":
            J[0, N - 1] = J[N - 1, 0] = -0.8
        bases.append(b)
        Js.append(J)
        V0s.append(rng.uniform(-1, 1, (nvec, b.dim)))
    res = lanczos_batched(bases, Js, V0s, 8)
    for k, (N, two_s, A, _) in enumerate(specs):
        sub = oracle.Subspace(N, two_s, A)
        for r in range(nvec):
            ref = oracle.lanczos(sub, Js[k], V0s[k][r], 8)
            n = min(int(res.steps_done[k, r]), ref["steps_done"])
            # a breakdown is found at the FP32 rounding floor or at the FP64 one
            scale = max(np.abs(ref["alpha"]).max(), np.abs(ref["beta"][:-1]).max(initial=0.0))
            m = n if n < 4 else n - 1
            assert np.abs(res.alpha[k, r, :m] - ref["alpha"][:m]).max() <= 1e-5 * scale, (k, r)


def test_two_items_per_chunk_vs_single():
    """2.6 M rows in two instances of different length, against the single path."""
    from paper_0706_3293_amd import Basis, inputs, lanczos_batched
    bases = [Basis(14, two_s=2, two_M=0), Basis(24, two_s=1, two_M=4)]
    Js = [inputs.chain_couplings(np.linspace(-1.3, -0.7, 13)), inputs.ring_couplings(24, -1.0)]
    V0s = [torch.tensor(np.stack([inputs.start_vector(b.dim, q) for q in range(2)]),
                        device="cuda") for b in bases]
    res = lanczos_batched(bases, Js, V0s, 6)
    for k, b in enumerate(bases):
        for q in range(2):
            one = b.lanczos(Js[k], V0s[k][q].contiguous(), 6, precision="f32_mixed")
            scale = np.abs(one.alpha).max()
            assert np.abs(res.alpha[k, q] - one.alpha).max() <= 1e-5 * scale
            assert abs(res.E0[k, q] - one.E0) <= 1e-5 * scale
