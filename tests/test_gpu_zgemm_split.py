"""Products of few output tiles: K ranges at the edges of two-slice parts (a
slice is 16 long) and of the skinny kernels' chunks, ragged edges included,
against numpy's product within a few rounding errors of the sum of sizes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opA,opB", [("N", "N"), ("C", "N"), ("N", "C"), ("C", "C")])
@pytest.mark.parametrize("m,n", [(70, 130), (64, 100), (100, 64), (16, 65), (65, 17)])
def test_short_k(opA, opB, m, n):
    from paper_1007_4400_amd import gevp

    h = gevp.Handle(0)
    rng = np.random.default_rng(m + 3 * n)
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    for k in (1, 15, 16, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 161, 256, 500):
        print(f"short K {opA}{opB} {m} x {n} x {k}", flush=True)
        A = cn(*((m, k) if opA == "N" else (k, m)))
        B = cn(*((k, n) if opB == "N" else (n, k)))
        C, E, g = cn(m, n), cn(m, n), rng.standard_normal(n)
        opa = A if opA == "N" else A.conj().T
        opb = B if opB == "N" else B.conj().T
        ref = 1.5 * opa @ opb - 0.25 * C + 0.75 * E * g
        out = h.zgemm(opA, opB, dev(A), dev(B), alpha=1.5, beta=-0.25, C=dev(C), gamma=0.75, E=dev(E),
                      gcol=dev(g)).cpu().numpy()
        scale = 1.5 * np.abs(opa) @ np.abs(opb) + 0.25 * np.abs(C) + 0.75 * np.abs(E * g)
        assert np.all(np.abs(out - ref) <= 1e-14 * np.sqrt(k) * 10 * scale)
    h.close()
