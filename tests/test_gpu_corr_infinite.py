"""GPU checks of the bond correlations of a vector with an infinite entry: a move that
a row does not allow reads nothing, so a correlation is infinite or NaN exactly where
the plain sum over the allowed terms is."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _plain(b, bonds, psi):
    """<psi|s(u).s(v)|psi> from each row's allowed terms, in FP64 (infinities kept)."""
    rows = np.array([b.unrank(i) for i in range(b.dim)])
    index = {tuple(r): i for i, r in enumerate(rows)}
    two_s, out = b.two_s, []
    F = np.sqrt(np.arange(two_s + 2) * (two_s + 1.0 - np.arange(two_s + 2)))
    with np.errstate(invalid="ignore"):
        for u, v in bonds:
            total = 0.0
            for i, r in enumerate(rows):
                a, c = r[u], r[v]
                s = 0.25 * ((two_s - 2 * a) * (two_s - 2 * c)) * psi[i]
                for x, y in ((u, v), (v, u)):
                    if r[x] >= 1 and r[y] < two_s:
                        t = r.copy()
                        t[x] -= 1
                        t[y] += 1
                        s = s + 0.5 * F[r[x]] * F[r[y] + 1] * psi[index[tuple(t)]]
                total = total + psi[i] * s
            out.append(total)
    return np.array(out)


@pytest.mark.parametrize("N,two_s,A", [(10, 1, 5), (10, 1, 3), (6, 2, 6), (5, 3, 7)])
def test_infinite_entry(N, two_s, A):
    from paper_0706_3293_amd import Basis
    b = Basis(N, two_s=two_s, two_M=N * two_s - 2 * A)
    bonds = [(u, v) for u in range(N) for v in range(u + 1, N)]
    base = np.random.default_rng(N).uniform(-1, 1, b.dim)
    for at in (0, b.dim // 3, b.dim - 1):
        psi = base.copy()
        psi[at] = np.inf
        got = b.bond_corr(bonds, torch.tensor(psi, device="cuda"))
        ref = _plain(b, bonds, psi)
        print(N, two_s, A, at, np.isnan(ref).sum(), np.isinf(ref).sum(), flush=True)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(got[~np.isnan(ref)], ref[~np.isnan(ref)])
    got = b.bond_corr(bonds, torch.tensor(base, device="cuda"))
    assert np.abs(got - _plain(b, bonds, base)).max() <= 1e-13 * (base @ base) * two_s * (two_s + 2)
