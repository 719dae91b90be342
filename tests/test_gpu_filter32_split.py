"""FP32 filter products cut along K (few output tiles) against the complex128
definition, beside the tile edges and where the cut begins."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(1001, 116), (127, 3), (128, 64), (129, 65), (640, 1), (2048, 33), (700, 700)])
def test_filter32(n, m):
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = gevp.Handle(0)
    print(f"filter32 n={n} m={m}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + m)
    C = torch.randn(n, n, generator=g, device="cuda", dtype=torch.complex128)
    C = 0.5 * (C + C.mH)
    G, P, R = (torch.randn(m, n, generator=g, device="cuda", dtype=torch.complex64).mT for _ in range(3))
    co = [torch.rand(m, generator=g, device="cuda", dtype=torch.float64) + 0.5 for _ in range(4)]
    co[1][0] = 0.0  # coefficients that leave a term out
    co[3][-1] = 0.0
    D = h.filter_gemm("fp32", gevp.colmajor(C.resolve_conj()), G, P, R, *co)
    c, gg, pp, rr = (t.cpu().numpy().astype(complex) for t in (C, G, P, R))
    al, be, ga, de = (t.cpu().numpy() for t in co)
    ref = al * (c @ gg) + be * gg + ga * pp + de * rr
    # FP32 sums of n terms (random signs: sqrt(n) roundings), three real products
    mag = (np.abs(c.real) + np.abs(c.imag)) @ (np.abs(gg.real) + np.abs(gg.imag)) * al
    size = be * np.abs(gg) + ga * np.abs(pp) + de * np.abs(rr)
    err = np.abs(D.cpu().numpy() - ref)
    assert (err <= 2.0**-24 * ((2 * np.sqrt(n) + 16) * mag / np.sqrt(n) + 8 * (mag / np.sqrt(n) + size))).all()
    h.close()
