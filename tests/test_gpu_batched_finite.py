"""GPU checks that a batched run without an energy is an error: coefficients that
are not finite were refused by the tridiagonal solver of each pair, whichever pair
and step they come from."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _batch(scale=1.0, bad=None, nvec=3):
    """Three instances; `scale` multiplies the last one's couplings, `bad` is put
    into one entry of its middle start vector."""
    from paper_0706_3293_amd import Basis, inputs
    bases = [Basis(10, two_s=1, two_M=0), Basis(6, two_s=2, two_M=0), Basis(8, two_s=1, two_M=2)]
    Js = [inputs.chain_couplings(np.linspace(-1.3, -0.7, b.N - 1)) for b in bases]
    Js[2] = Js[2] * scale
    V0s = [np.random.default_rng(b.dim).uniform(-1, 1, (nvec, b.dim)) for b in bases]
    if bad is not None:
        V0s[2][1, 5] = bad
    return bases, Js, V0s


# 1e39: matrix elements beyond FP32 in the first step; 1e25: the second product
# (the vectors keep the scale of the first) overflows
@pytest.mark.parametrize("scale,bad", [(1e39, None), (1e25, None), (1.0, np.inf), (1.0, -np.inf)])
@pytest.mark.parametrize("steps", [1, 6])
def test_run_without_an_energy_is_refused(scale, bad, steps):
    from paper_0706_3293_amd import _lib, lanczos_batched
    if scale == 1e25 and steps == 1:
        pytest.skip("finite in the first step")
    print("batched finite", scale, bad, steps, flush=True)
    with pytest.raises(_lib.HMError) as e:
        lanczos_batched(*_batch(scale, bad), steps)
    assert e.value.code == _lib.HM_EINVAL


def test_magnetization_curve_refuses_couplings_beyond_fp32():
    from paper_0706_3293_amd import _lib, inputs, magnetization_curve
    with pytest.raises(_lib.HMError):
        magnetization_curve(6, 2, inputs.ring_couplings(6, -1e39), steps=4, method="batched")


def test_finite_runs_are_as_before():
    """Large but representable couplings, and a breakdown (one state)."""
    from paper_0706_3293_amd import Basis, lanczos_batched
    r = lanczos_batched(*_batch(1e15), 6)
    assert np.isfinite(r.E0).all() and (r.steps_done == 6).all()
    b = Basis(6, two_s=1, two_M=6)
    J = np.zeros((6, 6))
    J[0, 1] = J[1, 0] = 0.5
    r = lanczos_batched([b], [J], [np.ones((2, 1))], 4)
    assert (r.steps_done == 1).all() and np.abs(r.E0 + 0.125).max() <= 1e-7
