"""GPU checks of the kernel for s >= 1 on a coupling list's second product.  The first
goes to the generic kernel where it costs less than the block kernel's tables, so
every check of the block kernel's products is repeated here on products whose tables
exist, and the two have to be the same bits."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_digit import (test_64_bit_indices_match_generic_kernel,  # noqa: F401, E402
                            test_long_blocks_match_oracle_and_generic_kernel,
                            test_rows_match_oracle,
                            test_values_that_are_not_finite_reach_the_same_rows)
from test_gpu_digit_lds import test_products_at_the_lds_budget  # noqa: F401, E402
from test_gpu_digit_memory import test_tables_are_bounded_by_the_vector  # noqa: F401, E402
from test_gpu_digit_overflow import (test_couplings_beyond_fp32,  # noqa: F401, E402
                                     test_infinite_and_nan_entries)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(autouse=True)
def _second(request, monkeypatch):
    from paper_0706_3293_amd import Basis
    if request.function.__module__ == __name__:
        return
    once = Basis.apply

    def twice(self, J, x, out=None, kernel=0):
        y = once(self, J, x, out=out, kernel=kernel)
        if kernel != 0:
            return y
        first = y.clone()
        y = once(self, J, x, out=out, kernel=kernel)
        assert bool(((first == y) | (first.isnan() & y.isnan())).all())
        return y

    monkeypatch.setattr(Basis, "apply", twice)


# rows, blocks and bonds on both sides of the rule that puts the tables off
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("N,A,kind", [(9, 9, "ring"), (14, 14, "ring"), (14, 14, "all"), (15, 15, "ring"),
                                      (20, 7, "ring"), (20, 7, "all"), (24, 8, "ring")])
def test_products_of_one_list_are_the_same(N, A, kind, dtype):
    from paper_0706_3293_amd import Basis, inputs
    print("digit first", N, A, kind, dtype, flush=True)
    b = Basis(N, two_s=2, two_M=2 * N - 2 * A)
    J = inputs.all_to_all_couplings(N, 1)[0] if kind == "all" else inputs.ring_couplings(N, -1.1, -0.37)
    x = torch.rand(b.dim, dtype=dtype, device="cuda") - 0.5
    ref = b.apply(J, x, kernel=1)
    y = [b.apply(J, x) for _ in range(3)]
    assert torch.equal(y[0], y[1]) and torch.equal(y[1], y[2])
    # the generic kernel's bits, in FP64 up to 2^20 rows
    if dtype == torch.float32 or b.dim <= 1 << 20:
        assert torch.equal(y[2], ref)
    else:
        assert float((y[2] - ref).abs().max()) <= 1e-13 * abs(J).sum() * 4
    b.free()


def test_a_list_used_once_builds_no_tables():
    """484,500 rows in 47,672 blocks of 10: 40 bonds' tables are 30 MB, and more time
    than a product of the generic kernel."""
    from paper_0706_3293_amd import Basis, inputs
    b = Basis(20, two_s=2, two_M=26)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    b.apply(inputs.ring_couplings(20, -1.0), x, out=y, kernel=1)
    free = []
    for s in (1.0, 1.0, 2.0):
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
        b.apply(inputs.ring_couplings(20, -s, -0.5), x, out=y)
        torch.cuda.synchronize()
    free.append(torch.cuda.mem_get_info()[0])
    took = [a - c for a, c in zip(free, free[1:])]
    print(took, flush=True)
    assert took[0] <= 4 << 20 and took[2] <= 4 << 20
    assert took[1] >= 16 << 20
    b.free()
