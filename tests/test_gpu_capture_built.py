"""GPU checks of FP64 products captured in a graph on a handle that has only been
used in FP32, or through the block kernel by number: the automatic FP64 kernels have
tables of their own, which a capture cannot build, so the split that is built is
captured.  Each graph is replayed with eager work in between."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# staged blocks from 2^20 rows on, one workgroup per block up to 2^18, and between
# them the block kernel's own split
@pytest.mark.parametrize("N,A", [(23, 11), (24, 12), (16, 8), (20, 10), (21, 10)])
@pytest.mark.parametrize("first", ["f32", "kernel2", "f64"])
def test_fp64_product_captured_on_a_used_handle(N, A, first):
    from paper_0706_3293_amd import Basis, inputs
    print("capture", N, A, first, flush=True)
    J = inputs.ring_couplings(N, -1.1, -0.37)
    b, other = (Basis(N, two_s=1, two_M=N - 2 * A) for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda", generator=g) - 0.5
    if first == "f32":
        b.apply(J, x.float())
    elif first == "kernel2":
        b.apply(J, x, kernel=2)
    else:
        b.apply(J, x)
    ref = other.apply(J, x, kernel=0 if first == "f64" else 2)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.apply(J, x, out=y)
    for _ in range(3):
        y.zero_()
        other.apply(J, x.float())
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
    # the handle builds the tables afterwards, and the graph still gives its rows
    after = b.apply(J, x)
    assert float((after - ref).abs().max()) <= 1e-13 * 60
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(y, ref)


def test_first_product_captured_in_a_large_sector():
    """Nothing built but the couplings: the generic kernel, as in smaller sectors."""
    from paper_0706_3293_amd import Basis, inputs
    b = Basis(23, two_s=1, two_M=1)
    J = inputs.ring_couplings(23, -1.1, -0.37)
    x = torch.rand(b.dim, dtype=torch.float64, device="cuda")
    ref = b.apply(J, x, kernel=1)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.apply(J, x, out=y)
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
