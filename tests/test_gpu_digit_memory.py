"""GPU check of the device memory that the kernel for s >= 1 takes beside the vectors."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# blocks of 2.8 to 9 rows: tables of 1.1 to 2.8 GB for vectors of 2.5 to 275 MB, and
# one of 0.4 GB that stays
@pytest.mark.parametrize("N,A,kind,most", [(31, 5, "all", 1 << 30), (28, 6, "all", 1 << 30),
                                           (26, 9, "ring", 34370050 * 32), (24, 8, "ring", 1 << 30)])
def test_tables_are_bounded_by_the_vector(N, A, kind, most):
    from paper_0706_3293_amd import Basis, inputs
    print("digit memory", N, A, kind, flush=True)
    b = Basis(N, two_s=2, two_M=2 * N - 2 * A)
    J = inputs.all_to_all_couplings(N, 1)[0] if kind == "all" else inputs.ring_couplings(N, -1.0)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda")
    y, ref = torch.empty_like(x), torch.empty_like(x)
    b.apply(J, x, out=ref, kernel=1)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    b.apply(J, x, out=y)
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    print(f"{taken / 1e6:.0f} MB", flush=True)
    assert taken <= most + (64 << 20)             # the allocator's granularity
    assert float((y - ref).abs().max()) <= 1e-13 * abs(J).sum() * 4
    b.free()
