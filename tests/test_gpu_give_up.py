"""The route a call takes when the work-groups of a single-launch kernel do not come
together: a poll limit of 0 makes every wait in one give up at once (the kernels
then end normally), as a device shared with other processes does after a time."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gevp():
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return gevp


def _dev(a):
    return torch.from_numpy(np.asfortranarray(a)).cuda()


def _hermitian(rng, n):
    G = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return 0.5 * (G + G.conj().T)


def _pencil(n, nev, seeded, seed=0):
    """Spectrum known; the seed is the exact eigenvectors, rotated a little."""
    rng = np.random.default_rng(seed + n)
    lam = np.concatenate([np.sort(rng.uniform(-3.0, -0.5, nev)), np.sort(rng.uniform(0.0, 20.0, n - nev))])
    Q = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))[0]
    A = (Q * lam) @ Q.conj().T
    return lam, _dev(0.5 * (A + A.conj().T)), _dev(np.eye(n, dtype=complex)), Q


@pytest.mark.parametrize("n", [61, 256, 300, 513, 948, 1537, 2048])
def test_heev_by_launches_per_reflector(gevp, n):
    """Each of three matrices of one order: the first call gives up and captures the
    sequence of launches, the later ones replay it; a fresh handle's results are the
    same bits."""
    print(f"give up heev n={n}", flush=True)
    rng = np.random.default_rng(n)
    h = gevp.Handle(0)
    h.set_poll_limit(0)
    for r in range(3 if n < 1000 else 2):
        H = _hermitian(rng, n) + r * np.eye(n)
        th, Z = (t.cpu().numpy() for t in h.heev(_dev(H)))
        lam = np.linalg.eigvalsh(H)
        nrm = max(1.0, np.max(np.abs(lam)))
        assert np.max(np.abs(th - lam)) <= 1e-13 * nrm * np.sqrt(n)
        assert np.max(np.abs(H @ Z - Z * th[None, :])) <= 1e-12 * nrm * np.sqrt(n)
        assert np.max(np.abs(Z.conj().T @ Z - np.eye(n))) <= 1e-10
    h2 = gevp.Handle(0)
    h2.set_poll_limit(0)
    th2, Z2 = (t.cpu().numpy() for t in h2.heev(_dev(H)))
    assert np.array_equal(th, th2) and np.array_equal(Z, Z2)
    # and the single launch again, once the limit is lifted
    h2.set_poll_limit(-1)
    th3, _ = h2.heev(_dev(H))
    h3 = gevp.Handle(0)
    th4, _ = h3.heev(_dev(H))
    assert torch.equal(th3, th4)
    assert np.max(np.abs(th3.cpu().numpy() - lam)) <= 1e-13 * nrm * np.sqrt(n)
    for x in (h, h2, h3):
        x.close()


# orders at the edges of the single-launch Lanczos steps, and one beyond them
@pytest.mark.parametrize("n", [64, 257, 700, 1100, 2049])
@pytest.mark.parametrize("seeded", [False, True])
def test_solve(gevp, n, seeded):
    print(f"give up solve n={n} seeded={seeded}", flush=True)
    nev = max(4, n // 12)
    lam, A, B, Q = _pencil(n, nev, seeded)
    h = gevp.Handle(0)
    kx = h.block_size(n, nev)
    X0 = None
    if seeded:
        rng = np.random.default_rng(1)
        D = rng.standard_normal((n, kx)) + 1j * rng.standard_normal((n, kx))
        X0 = _dev(np.linalg.qr(Q[:, :kx] + 1e-4 * D / np.sqrt(n))[0])
        kept = X0.clone()
    want, _, _, info0 = h.solve(A, B, nev, X0=X0, kx=kx)
    h.set_poll_limit(0)
    Ak, Bk = A.clone(), B.clone()
    for _ in range(2):  # the call that gives up, and one after it
        th, X, _, info = h.solve(A, B, nev, X0=X0, kx=kx)
        assert info["max_resid"] <= 1e-10
        assert np.max(np.abs(th.cpu().numpy()[:nev] - lam[:nev])) <= 1e-10 * 20
        assert ((th[:nev] - want[:nev]).abs() <= 1e-10 * 20).all()
        # the norm estimates come from a few steps: alike but for rounding
        assert abs(info["normA"] - info0["normA"]) <= 1e-6 * info0["normA"]
        assert info["nconv"] == nev
    assert torch.equal(A, Ak) and torch.equal(B, Bk)
    if seeded:
        assert torch.equal(X0, kept)
    # no share of the device stayed behind: another thread's handle gets all of it
    out = []

    def other():
        h2 = gevp.Handle(0)
        out.append(h2.solve(A, B, nev, X0=X0, kx=kx)[0])
        h2.close()

    t = threading.Thread(target=other, daemon=True)
    t.start()
    t.join(60)
    assert out and torch.equal(out[0], want)
    h.close()


def test_batch(gevp):
    """Workers take the handle's limit."""
    problems, lams = [], []
    for i, n in enumerate((150, 300, 450)):
        lam, A, B, _ = _pencil(n, 12, False, seed=i)
        problems.append({"A": A, "B": B, "nev": 12})
        lams.append(lam)
    h = gevp.Handle(0)
    h.set_poll_limit(0)
    for _ in range(2):
        for (th, _, _, info), lam in zip(h.solve_batched(problems), lams):
            assert info["max_resid"] <= 1e-10
            assert np.max(np.abs(th.cpu().numpy()[:12] - lam[:12])) <= 1e-10 * 20
    h.close()
