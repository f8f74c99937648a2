"""GPU checks that the block kernel's schedule is refused after the first use of the
handle, whichever kernel that use took."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N", [8, 12, 14, 16, 24])
@pytest.mark.parametrize("use", ["reorth", "reorth_mixed", "run", "product", "product_f32"])
def test_schedule_is_refused_after_the_first_use(N, use):
    from paper_0706_3293_amd import Basis, _lib, inputs
    if N == 8 and use == "run":
        pytest.skip("a run of kernel 3, which takes nothing from the schedule")
    b = Basis(N, two_s=1, two_M=0 if N < 24 else 18)
    J = inputs.ring_couplings(N, -1.0, -0.3)
    v = torch.tensor(inputs.start_vector(b.dim, 0), device="cuda")
    if use.startswith("reorth"):
        b.lanczos(J, v, 6, full_reorth=True, precision="f32_mixed" if "mixed" in use else "f64")
    elif use == "run":
        b.lanczos(J, v, 6)
    else:
        b.apply(J, v if use == "product" else v.float())
    for call in ((6, 256, 1), (6, 64, 2, 1)):
        with pytest.raises(_lib.HMError) as e:
            b.set_schedule(*call)
        assert e.value.code == _lib.HM_EINVAL
    assert _lib.lib().hm_basis_set_staging(b.handle, 1) == _lib.HM_EINVAL
    assert _lib.lib().hm_basis_set_items_per_wave(b.handle, 4) == _lib.HM_EINVAL
