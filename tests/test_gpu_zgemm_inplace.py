"""Products written over one of their operands, or over a part of one, give what the
same product gives with a result of its own, bit for bit: in residues, by the FP64
kernels behind them (an operand that cannot be scaled) and by those alone."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = gevp.Handle(0)
    yield h
    h.close()


def _cn(seed, m, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(n, m, generator=g, device="cuda", dtype=torch.complex128).mT


def _copy(t):
    return t.mT.clone().mT


# one tile wide, just over it, several tiles, residues
@pytest.mark.parametrize("tiny", [False, True])
@pytest.mark.parametrize("m,q", [(300, 64), (300, 65), (40, 64), (130, 130), (700, 300), (3000, 1200)])
def test_over_the_left_operand(h, m, q, tiny):
    A, B = _cn(1, m, q), _cn(2, q, q)
    if tiny:
        A[7] *= 1e-200
    ref = h.zgemm("N", "N", _copy(A), B)
    assert torch.equal(h.zgemm("N", "N", A, B, out=A), ref)


@pytest.mark.parametrize("tiny", [False, True])
@pytest.mark.parametrize("q,n", [(64, 300), (65, 300), (64, 40), (130, 130), (300, 700), (1200, 3000)])
def test_over_the_right_operand(h, q, n, tiny):
    A, B = _cn(3, q, q), _cn(4, q, n)
    if tiny:
        B[:, 7] *= 1e-200
    ref = h.zgemm("N", "N", A, _copy(B))
    assert torch.equal(h.zgemm("N", "N", A, B, out=B), ref)


@pytest.mark.parametrize("n", [50, 64, 200, 1400])
def test_transposed_and_both(h, n):
    A, B = _cn(5, n, n), _cn(6, n, n)
    ref = h.zgemm("C", "N", _copy(A), B)
    out = _copy(A)
    assert torch.equal(h.zgemm("C", "N", out, B, out=out), ref)
    ref = h.zgemm("N", "C", A, _copy(B))
    out = _copy(B)
    assert torch.equal(h.zgemm("N", "C", A, out, out=out), ref)
    ref = h.zgemm("N", "N", _copy(A), _copy(A))
    out = _copy(A)
    assert torch.equal(h.zgemm("N", "N", out, out, out=out), ref)


def test_parts_of_one_array(h):
    """Blocks that meet, and blocks side by side that do not."""
    for rows, cols in ((0, 40), (40, 0), (-40, 30), (200, 0), (0, 200), (200, 200)):
        P = _cn(7, 700, 700)
        A, B = P[150:350, 150:350], _cn(8, 200, 200)
        D = P[150 + rows:350 + rows, 150 + cols:350 + cols]
        rest = _copy(P)
        ref = h.zgemm("N", "N", _copy(A), B)
        h.zgemm("N", "N", A, B, out=D)
        assert torch.equal(D, ref)
        rest[150 + rows:350 + rows, 150 + cols:350 + cols] = ref
        assert torch.equal(P, rest)


@pytest.mark.parametrize("n", [200, 3000])
def test_structured(h, n):
    A, B = _cn(9, n, n), _cn(10, n, 90)
    ref = torch.empty_like(B)
    h.zgemm_tri("N", "N", A, _copy(B), ref, upperA=True)
    h.zgemm_tri("N", "N", A, B, B, upperA=True)
    assert torch.equal(B, ref)
