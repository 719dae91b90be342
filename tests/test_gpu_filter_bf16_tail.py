"""Split-BF16 filter product at the widths where the last column of tiles turns
from 64 to 128 wide, against the complex128 definition; the bound is the split's
(2^-16 a product, relative to the size of the terms) as for every width."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(200, 1), (200, 64), (200, 65), (333, 128), (333, 192), (1100, 193), (2100, 129)])
def test_tail_width(n, m):
    from paper_1007_4400_amd import gevp

    print(f"filter tail n={n} m={m}", flush=True)
    rng = np.random.default_rng(n + m)
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    C = cn(n, n)
    C = 0.5 * (C + C.conj().T) / np.sqrt(n)
    G, P, R = (cn(n, m).astype(np.complex64) for _ in range(3))
    co = [rng.standard_normal(m) for _ in range(4)]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    h = gevp.Handle(0)
    out = h.filter_gemm("bf16x3", dev(C), dev(G), dev(P), dev(R), *(dev(c) for c in co)).cpu().numpy()
    h.close()
    al, be, ga, de = co
    ref = (C @ G.astype(complex)) * al + G * be + P * ga + R * de
    scale = np.abs(C) @ np.abs(G) * np.abs(al) + np.abs(G * be) + np.abs(P * ga) + np.abs(R * de)
    assert np.max(np.abs(out - ref) / scale) <= 1e-4
