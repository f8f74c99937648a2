"""GPU checks of the spin-1/2 codec (low words from a table, set bits only) against
the host codec: sectors around the table's 12 sites, 32- and 64-bit words, full and
empty sectors, indices and states outside the subspace."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N,A", [(2, 1), (11, 5), (12, 6), (13, 0), (13, 13), (13, 6), (20, 10),
                                 (32, 16), (32, 32), (33, 4), (36, 18), (44, 22), (45, 3),
                                 (60, 5), (64, 2), (64, 62)])
def test_codec_matches_host(N, A):
    from paper_0706_3293_amd import Basis
    print("codec half", N, A, flush=True)
    b = Basis(N, two_s=1, two_M=N - 2 * A)
    rng = np.random.default_rng(N * 100 + A)
    idx = np.unique(np.concatenate([[0, b.dim - 1], rng.integers(0, b.dim, 400)]))
    want = np.array([sum(int(d) << u for u, d in enumerate(b.unrank(int(i)))) for i in idx],
                    dtype=np.uint64).view(np.int64)
    got = b.unrank_dev(torch.tensor(np.concatenate([idx, [-1, b.dim]]), device="cuda"))
    assert np.array_equal(got.cpu().numpy()[:-2], want)
    assert (got.cpu().numpy()[-2:] == -1).all()
    st = want.view(np.uint64)
    bad = st[:50] ^ np.uint64(1)                      # one bit too many or too few
    if N < 64:
        bad = np.concatenate([bad, st[:5] | np.uint64(1 << N)])
    back = b.rank_dev(torch.tensor(np.concatenate([st, bad]).view(np.int64), device="cuda"))
    assert np.array_equal(back.cpu().numpy()[:len(st)], idx)
    assert (back.cpu().numpy()[len(st):] == -1).all()
