"""Large products whose operands one scale a row, a column and a k slice cannot
serve: entries of the product to which only the small entries of a row contribute
have to be as accurate as the FP64 kernels make them.

Tolerance: with terms of random sign the partial sums stay below about twice the
square root of their number, so a sum of k terms is off by 0.8 x 2^-53 of the sum
of sizes (root mean square), the three-product complex form by up to 2.5; six
times that bounds the sample.  Where one term outweighs the others, every addition
after it rounds at its size: sqrt(k) x 0.29 x 2^-53 of it, 0.71 in the
three-product form, five times that for the sample.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 16 * 2.0**-53


@pytest.fixture(scope="module")
def h():
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return gevp.Handle(0)


def _gauss(seed, m, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(n, m, generator=g, device="cuda", dtype=torch.complex128).mT


def _rel(got, opa, opb, rows, cols, tol=False):
    """Errors of sampled entries over their sums of sizes (0 where that is 0), or
    over their tolerances."""
    a, b = opa[rows].cpu().numpy(), opb[:, cols].cpu().numpy()
    ar, ai, br, bi = (np.asarray(v, dtype=np.longdouble) for v in (a.real, a.imag, b.real, b.imag))
    d = got[rows][:, cols].cpu().numpy()
    err = np.hypot((d.real - (ar @ br - ai @ bi)).astype(float), (d.imag - (ar @ bi + ai @ br)).astype(float))
    size = np.abs(a) @ np.abs(b)
    assert (err[size == 0] == 0).all()
    if tol:
        largest = np.array([[(np.abs(x) * np.abs(b[:, j])).max() for j in range(b.shape[1])] for x in a])
        size = TOL * size + 4 * np.sqrt(a.shape[1]) * 2.0**-53 * largest
    return err / np.where(size == 0, 1, size)


ROWS, COLS = [0, 3, 64, 100, 127, 128, 500, 1000, 1535], [0, 3, 17, 255, 256, 900, 1023]


def _operands(kind, s):
    m, n, k = 1536, 1024, 2048
    A, B = _gauss(1, m, k), _gauss(2, k, n)
    if kind == "zero slice":  # large entries that meet zeros only
        A[3, 17] = s
        A[100:200, 40] = s
        B[17] = 0
        B[40] = 0
    elif kind == "zero but one":  # ... zeros and one column
        A[:, 17] *= s
        B[17] = 0
        B[17, 3] = 1
    elif kind == "every chunk":  # one such entry in every run of 64 k
        A[:, 5::64] *= s
        B[5::64] = 0
        B[5::64, 3] = 1
    elif kind == "blocks":
        A[:, : k // 2] *= s
        B[: k // 2, : n // 2] = 0
        B[k // 2 :, n // 2 :] = 0
    else:  # "columns": the same on the other side
        A[: m // 2, k // 2 :] = 0
        A[m // 2 :, : k // 2] = 0
        B[: k // 2] *= s
    return A, B


@pytest.mark.parametrize("s", [1e4, 1e8, 1e12, 1e20, 1e120])
@pytest.mark.parametrize("kind", ["zero slice", "zero but one", "every chunk", "blocks", "columns"])
def test_small_entries_keep_their_accuracy(h, kind, s):
    print(f"residue check {kind} {s:g}", flush=True)
    A, B = _operands(kind, s)
    assert _rel(h.zgemm("N", "N", A, B), A, B, ROWS, COLS, tol=True).max() <= 1
    # the same product from the other side's point of view, and with the operands' sizes
    # swapped between storage orders
    out = h.zgemm("C", "C", B, A)
    assert _rel(out, B.mH, A.mH, COLS, ROWS, tol=True).max() <= 1


@pytest.mark.parametrize("bad", ["nan", "inf"])
def test_zero_slice_does_not_hide(h, bad):
    """NaN and infinity times zero are NaN, whatever the slice they stand in."""
    A, B = _operands("zero slice", 1.0)
    A[3, 17] = float(bad)
    out = h.zgemm("N", "N", A, B)
    assert torch.isnan(out[3].real).all() and torch.isnan(out[3].imag).all()
    rows = [r for r in ROWS if r != 3]
    assert _rel(out, A, B, rows, COLS, tol=True).max() <= 1


@pytest.mark.parametrize("case", ["gauss", "real", "diagonal", "triangle", "unit lower"])
def test_ordinary_operands_stay_in_residues(h, case):
    """Exact sums leave only the operands' rounding, an eighth of the FP64 kernels'
    error or less: that this is what comes out shows the route."""
    n = 3072 if case in ("triangle", "unit lower") else 1536
    A, B = _gauss(3, n, n), _gauss(4, n, n)
    if case == "real":
        A, B = A.real.to(A.dtype), B.real.to(B.dtype)
        A, B = A.mT.contiguous().mT, B.mT.contiguous().mT
    elif case == "diagonal":  # a spectrum on [0, 50] in a random basis: diagonal 22, the rest 15 a row
        A = A * (15.0 / n**0.5 / 2**0.5) + 22.0 * torch.eye(n, device="cuda", dtype=A.dtype)
    elif case in ("triangle", "unit lower"):
        if case == "unit lower":
            A = A * (1.1 / n**0.5) + torch.eye(n, device="cuda", dtype=A.dtype)
        D = torch.empty_like(B)
        h.zgemm_tri("N", "N", A, B, D, upperA=True)
        rel = _rel(D, torch.triu(A), B, [0, 1, 63, 1000, 2000, 2303], COLS)
        assert np.sqrt((rel**2).mean()) <= 2.0**-56
        assert _rel(D, torch.triu(A), B, [2303, 2304, 2600, 3000, 3071], COLS, tol=True).max() <= 1
        return
    rel = _rel(h.zgemm("N", "N", A, B), A, B, ROWS, COLS)
    assert np.sqrt((rel**2).mean()) <= 2.0**-56


def test_solve_of_a_nearly_diagonal_pencil():
    """Localised eigenvectors: no product with the reduced matrix can take the
    residues, the copy converted for them included."""
    from paper_1007_4400_amd import gevp

    n, nev = 2048, 200
    rng = np.random.default_rng(0)
    lam = np.concatenate([np.sort(rng.uniform(-3.0, -0.1, nev)), np.sort(rng.uniform(0.5, 50.0, n - nev))])
    u = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    u /= np.linalg.norm(u)
    lu = lam * u
    A = np.diag(lam).astype(complex) - 2 * np.outer(u, lu.conj()) - 2 * np.outer(lu, u.conj())
    A += 4 * np.vdot(u, lu) * np.outer(u, u.conj())
    A = 0.5 * (A + A.conj().T)
    dev = lambda a: torch.from_numpy(np.asfortranarray(a)).cuda()  # noqa: E731
    h = gevp.Handle(0)
    th, X, _, info = h.solve(dev(A), dev(np.eye(n, dtype=complex)), nev, opts=gevp.make_opts())
    h.close()
    assert info["max_resid"] <= 1e-10
    assert np.max(np.abs(th.cpu().numpy()[:nev] - lam[:nev])) <= 1e-11 * 50
