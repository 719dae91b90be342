"""Eigensolves of matrices of low rank: the columns left after a few reflectors are
rounding errors, of rounding errors, and so on down to where their squares
underflow, and all but a few eigenvalues are one cluster."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _matrix(kind, n):
    i = np.arange(n)
    if kind == "ones":
        return np.ones((n, n), complex)
    if kind == "alternating":
        return ((-1.0) ** (i[:, None] + i)).astype(complex)
    if kind == "phases":  # entries 1, i, -1, -i
        u = 1j ** (i % 4)
        return np.outer(u, u.conj())
    if kind == "two blocks":
        H = np.zeros((n, n), complex)
        H[: n // 2, : n // 2] = 1
        H[n // 2 :, n // 2 :] = -2
        return H
    if kind == "tiny column":  # nothing but the first column beside the diagonal
        H = np.diag(np.linspace(1.0, 2.0, n)).astype(complex)
        H[1:, 0] = 1e-160 * (1 + 1j * (i[1:] % 3))
        H[0, 1:] = H[1:, 0].conj()
        return H
    u, v = np.ones(n), (i % 5).astype(float)
    return (np.outer(u, v) + np.outer(v, u) + 1j * (np.outer(u, v) - np.outer(v, u))).astype(complex)


@pytest.mark.parametrize("route", ["one launch", "launches per reflector"])
@pytest.mark.parametrize("kind", ["ones", "alternating", "phases", "two blocks", "tiny column", "rank 2"])
def test_orthogonal(kind, route):
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = gevp.Handle(0)
    if route != "one launch":
        h.set_poll_limit(0)
    for n in (3, 33, 60, 61, 67, 127, 128, 255, 300, 520):
        print(f"heev {kind} n={n} {route}", flush=True)
        H = _matrix(kind, n)
        th, Z = (t.cpu().numpy() for t in h.heev(torch.from_numpy(np.asfortranarray(H)).cuda()))
        lam = np.linalg.eigvalsh(H)
        nrm = np.max(np.abs(lam))
        assert np.max(np.abs(th - lam)) <= 1e-13 * nrm * np.sqrt(n)
        assert np.max(np.abs(H @ Z - Z * th[None, :])) <= 1e-12 * nrm * np.sqrt(n)
        assert np.max(np.abs(Z.conj().T @ Z - np.eye(n))) <= 1e-12 * np.sqrt(n)
    h.close()
