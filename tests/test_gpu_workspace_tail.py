"""Solves in a caller's buffer with room for some or all of what the residue
products use beyond the solve's own needs: the scratch of the main stream, the
converted reduced matrix, the scratch of the second stream.  Guard bytes on both
sides of the buffer stay as they were."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MIB = 2**20
GUARD = 4 * MIB


@pytest.fixture(scope="module")
def problem():
    from paper_1007_4400_amd import gevp, synth

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, nev = 2048, 205
    h = gevp.Handle(0)
    kx = h.block_size(n, nev)
    base = synth.LARGE
    wl = synth.Workload("case", n, nev, 12, "cluster", 1.1 / math.sqrt(n), base.eps0, base.decay, 0.0)
    A, B, _, _, g, (_, X0) = synth.make_pencil_torch(wl, 1, exact_nev=kx)
    A = A + synth.eps(wl, 5) * synth.unit_hermitian_torch(n, g)
    A, B, X0 = gevp.colmajor(A), gevp.colmajor(B), gevp.colmajor(X0)
    want = [h.solve(A, B, nev, X0=x, kx=kx) for x in (None, X0)]
    h.close()
    return gevp, A, B, X0, nev, kx, want


# n = 2048, 236 columns: about 262 MiB for the main stream, 133 for the matrix, 165
# for the second stream
@pytest.mark.parametrize("extra", [0, 100, 290, 410, 600, 1500])
def test_parts_of_the_scratch(problem, extra):
    gevp, A, B, X0, nev, kx, want = problem
    h = gevp.Handle(0)
    size = h.workspace_size(A.shape[0], nev) + extra * MIB
    whole = torch.full((size + 2 * GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    start = GUARD + (-(whole.data_ptr() + GUARD)) % 256
    h.set_workspace(whole[start:start + size])
    outs = []
    for x in (None, X0, X0, None):
        lam, X, _, info = h.solve(A, B, nev, X0=x, kx=kx)
        assert info["max_resid"] <= 1e-10
        outs.append((x is not None, lam, X))
    torch.cuda.synchronize()
    for seeded, lam, X in outs:
        ref = want[int(seeded)]
        if extra >= 600:  # the same kernels as with the library's own memory
            assert torch.equal(lam, ref[0]) and torch.equal(X, ref[1])
        assert ((lam[:nev] - ref[0][:nev]).abs() <= 1e-10 * 50).all()
    # products and gradients of the same handle take the tail too
    D = h.zgemm("N", "N", A, X0)
    dA, dB = h.backward(outs[0][2][:, :nev].mT.contiguous().mT, outs[0][1][:nev],
                        torch.ones(nev, dtype=torch.float64, device="cuda"))
    assert ((D - A @ X0).abs() <= 1e-13 * (A.abs() @ X0.abs())).all()
    V = outs[0][2][:, :nev]
    assert ((dA - V @ V.mH.contiguous()).abs() <= 1e-13 * (V.abs() @ V.abs().mT)).all()
    torch.cuda.synchronize()
    assert (whole[:start] == 0xA5).all() and (whole[start + size:] == 0xA5).all()
    h.close()
