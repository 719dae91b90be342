"""The tridiagonalisation that keeps H in registers (one work-group up to order
128, one launch of many work-groups above):
orders at the edges of the two and of the row counts per thread, against
numpy's eigenvalues; residual and orthogonality bound the vectors."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(h, H):
    from paper_1007_4400_amd import gevp

    n = H.shape[0]
    Hd = gevp.empty_colmajor(n, n, device="cuda")
    Hd.copy_(torch.from_numpy(H))
    th, Z = h.heev(Hd)
    th, Z = th.cpu().numpy(), Z.cpu().resolve_conj().numpy()
    lam = np.linalg.eigvalsh(H)
    nrm = max(1e-300, np.max(np.abs(lam)))
    # backward error of n reflectors, each of a few rounding errors
    assert np.max(np.abs(th - lam)) <= 1e-13 * nrm * np.sqrt(n)
    assert np.max(np.abs(H @ Z - Z * th[None, :])) <= 1e-12 * nrm * np.sqrt(n)
    assert np.max(np.abs(Z.conj().T @ Z - np.eye(n))) <= 1e-10
    return th, Z


@pytest.fixture(scope="module")
def h():
    from paper_1007_4400_amd import gevp

    hd = gevp.Handle(0)
    yield hd
    hd.close()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 60, 61, 64, 65, 126, 127, 128, 129, 131, 192, 255, 256, 257, 511, 513,
                               767, 769, 1021, 1024, 1025, 1537, 2048])
def test_orders(h, n):
    print(f"hetrd n={n}", flush=True)
    rng = np.random.default_rng(n)
    G = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    H = 0.5 * (G + G.conj().T)
    a = _check(h, H)
    b = _check(h, H)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("n", [50, 300])
def test_identity_reflectors(h, n):
    """Columns that are already tridiagonal (tau = 0) between dense blocks, and
    magnitudes far from 1."""
    print(f"hetrd blocks n={n}", flush=True)
    rng = np.random.default_rng(n)
    H = np.zeros((n, n), dtype=complex)
    i = 0
    while i < n:
        b = min(int(rng.integers(1, 40)), n - i)
        G = rng.standard_normal((b, b)) + 1j * rng.standard_normal((b, b))
        H[i:i + b, i:i + b] = (0.5 if b > 1 else 1.0) * (G + G.conj().T)
        i += b
    for scale in (1.0, 2.0 ** 300, 2.0 ** -300):
        _check(h, H * scale)
