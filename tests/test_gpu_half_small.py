"""GPU checks of FP64 products in the smallest spin-1/2 sectors, where a wave of the
block kernel has one item and one workgroup per block is slower: they take the block
kernel, give its bits and build the tables that both types share."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# one item for a wave up to 28 items, two and more from 32 on
SMALL = [(4, 2), (8, 4), (12, 6), (13, 6), (14, 4), (16, 3)]
MORE = [(14, 5), (14, 7), (16, 4), (17, 8)]


def _case(N, A, kind):
    from paper_0706_3293_amd import Basis, inputs
    b = Basis(N, two_s=1, two_M=N - 2 * A)
    J = inputs.all_to_all_couplings(N, 1)[0] if kind == "all" else inputs.ring_couplings(N, -1.1, -0.37)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda") - 0.5
    return b, J, x


@pytest.mark.parametrize("N,A", SMALL + MORE)
@pytest.mark.parametrize("kind", ["ring", "all"])
def test_products_have_the_bits_of_the_block_kernel(N, A, kind):
    print("half small", N, A, kind, flush=True)
    b, J, x = _case(N, A, kind)
    y = [b.apply(J, x) for _ in range(2)]
    ref = b.apply(J, x, kernel=2)
    assert torch.equal(y[0], ref) and torch.equal(y[1], ref)
    b.free()


def _captured(b, J, x):
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.apply(J, x, out=y)
    out = []
    for _ in range(3):
        y.zero_()
        x.clone()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        out.append(y.clone())
    return out


@pytest.mark.parametrize("N,A", SMALL)
def test_fp32_is_captured_after_an_fp64_product(N, A):
    print("half small capture", N, A, flush=True)
    b, J, x = _case(N, A, "ring")
    b.apply(J, x)
    xf = x.float()
    got = _captured(b, J, xf)
    ref = b.apply(J, xf, kernel=2)
    assert all(torch.equal(y, ref) for y in got)
    b.free()


@pytest.mark.parametrize("N,A", [(12, 6), (16, 3), (14, 7), (21, 10)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_first_product_is_captured(N, A, dtype):
    """Nothing built but the couplings: the generic kernel."""
    print("half small first", N, A, flush=True)
    b, J, x = _case(N, A, "ring")
    x = x.to(dtype)
    ref = b.apply(J, x, kernel=1)
    assert all(torch.equal(y, ref) for y in _captured(b, J, x))
    b.free()
