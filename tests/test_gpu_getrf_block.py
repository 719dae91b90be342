"""The 64 x 64 diagonal-block LU at the orders where its 16-wide panels and
blocks fill up, against the oracle's Doolittle factors (1e-11 of the largest
entry) and by reconstruction (1e-13 n)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 79, 113, 128])
def test_orders(oracle_mod, n):
    from paper_1007_4400_amd import gevp

    print(f"getrf block n={n}", flush=True)
    rng = np.random.default_rng(n)
    Q = np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))[0]
    C = (Q * rng.uniform(-3.0, 20.0, n)) @ Q.conj().T
    C = 0.5 * (C + C.conj().T)
    z = 0.4 + 0.7j
    M = z * np.eye(n) - C
    h = gevp.Handle(0)
    LU, piv = h.lu_shifted(torch.from_numpy(np.asfortranarray(C)).cuda(), z)
    h.close()
    assert piv == 0
    LU = LU.cpu().numpy()
    ref = oracle_mod.lu_nopivot(M)
    assert np.max(np.abs(LU - ref)) <= 1e-11 * max(1.0, np.max(np.abs(ref)))
    L, U = np.tril(LU, -1) + np.eye(n), np.triu(LU)
    assert np.max(np.abs(L @ U - M)) <= 1e-13 * n * max(1.0, np.max(np.abs(M)))
