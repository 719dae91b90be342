"""Cold solves at the edges of the single-launch Lanczos steps (orders 64 to
2048, eight rows a work-group, one to four rows a thread): the eigenvalues are
known by construction, and with B = I every run on B ends after one step (its
second vector is zero), so its norm estimate is exactly that of I."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 64, 65, 255, 256, 257, 512, 513, 1024, 1025, 1537, 2047, 2048, 2049])
def test_cold_solve(n):
    from paper_1007_4400_amd import gevp

    print(f"lanczos n={n}", flush=True)
    rng = np.random.default_rng(n)
    nev = 8
    lam = np.concatenate([np.sort(rng.uniform(-5.0, -4.0, nev)), np.sort(rng.uniform(0.0, 10.0, n - nev))])
    u = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    u /= np.linalg.norm(u)
    # A = H diag(lam) H with H = I - 2 u u^H
    lu = lam * u
    A = np.diag(lam).astype(complex) - 2 * np.outer(u, lu.conj()) - 2 * np.outer(lu, u.conj())
    A += 4 * np.vdot(u, lu) * np.outer(u, u.conj())
    A = 0.5 * (A + A.conj().T)
    dev = lambda a: torch.from_numpy(np.asfortranarray(a)).to("cuda")  # noqa: E731
    h = gevp.Handle(0)
    th, _, _, info = h.solve(dev(A), dev(np.eye(n, dtype=complex)), nev, opts=gevp.make_opts())
    h.close()
    th = th.cpu().numpy()[:nev]
    assert np.max(np.abs(th - lam[:nev])) <= 1e-10 * 10.0
    # an estimate from inside the spectrum plus the last coefficient
    assert 0.8 * lam[-1] <= info["normA"] <= 2.0 * lam[-1]
    assert abs(info["normB"] - 1.0) <= 1e-12
