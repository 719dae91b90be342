"""The 64 x 64 diagonal-block factor and its inverse beside the edges of its
16-wide panels, at the ends of the range of magnitudes, and where it fails."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return gevp.Handle(0)


def _hpd(n, seed, scale=1.0):
    rng = np.random.default_rng(seed)
    G = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return (G @ G.conj().T / n + np.eye(n)) * scale


@pytest.mark.parametrize("scale", [1.0, 1e-300, 1e300])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 48, 49, 63, 64, 65, 81, 127])
def test_factor_and_inverse(h, n, scale):
    """L L^H = M to a few roundings of the diagonal's size per summed term, and
    L^{-1} R through the blocks' inverses."""
    M = _hpd(n, n, scale)
    L, piv = h.potrf(torch.from_numpy(np.asfortranarray(M)).cuda())
    assert piv == 0
    Ln = L.cpu().numpy()
    assert np.array_equal(np.triu(Ln, 1), np.zeros_like(Ln))
    assert np.array_equal(np.diagonal(Ln).imag, np.zeros(n))
    s = Ln / np.sqrt(scale)
    d = np.sqrt(np.diagonal(M).real / scale)
    err = np.abs(s @ s.conj().T - M / scale) / np.outer(d, d)
    assert err.max() <= 4 * (n + 8) * 2.0**-53
    R = np.random.default_rng(7).standard_normal((n, 5)) + 0j
    X = h.trsm("L", "N", torch.from_numpy(np.asfortranarray(s)).cuda(),
               torch.from_numpy(np.asfortranarray(R)).cuda()).cpu().numpy()
    # the condition number of M is below 100 by its construction
    assert np.abs(s @ X - R).max() <= 100 * n * 2.0**-53 * max(1.0, np.abs(X).max())


@pytest.mark.parametrize("n,bad", [(64, 0), (64, 15), (64, 16), (50, 49), (130, 100)])
@pytest.mark.parametrize("val", [0.0, -1.0, float("nan"), float("inf")])
def test_failing_pivot(h, n, bad, val):
    M = np.eye(n, dtype=complex)
    M[bad, bad] = val
    _, piv = h.potrf(torch.from_numpy(np.asfortranarray(M)).cuda())
    assert piv == bad + 1


@pytest.mark.parametrize("n", [5, 16, 17, 64, 100])
def test_complex_diagonal(h, n):
    """Triangular solves invert blocks whose diagonal need not be real."""
    rng = np.random.default_rng(n)
    L = np.tril(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) * 0.05
    L[range(n), range(n)] = (1 + rng.random(n)) * np.exp(2j * np.pi * rng.random(n))
    R = rng.standard_normal((n, 9)) + 1j * rng.standard_normal((n, 9))
    for trans in ("N", "C"):
        X = h.trsm("L", trans, torch.from_numpy(np.asfortranarray(L)).cuda(),
                   torch.from_numpy(np.asfortranarray(R)).cuda()).cpu().numpy()
        op = L if trans == "N" else L.conj().T
        assert np.abs(op @ X - R).max() <= 100 * n * 2.0**-53 * max(1.0, np.abs(X).max())
