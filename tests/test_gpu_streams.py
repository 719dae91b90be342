"""Calls queued on one torch stream and then, without a wait, on another through
the same handle use its memory in turn: split products, skinny products cut along
K, FP32 and split-BF16 filter steps, triangular solves and gradients, each compared
bit by bit with the same call made alone."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cn(g, m, n, dtype=torch.complex128):
    return torch.randn(n, m, generator=g, device="cuda", dtype=dtype).mT


def _calls(gevp, kind, g):
    """Two calls of one kind on inputs of their own, each a function of the handle."""
    if kind.startswith("zgemm"):
        m, n, k = {"zgemm short": (256, 48, 256), "zgemm split": (300, 200, 2000),
                   "zgemm skinny cut": (600, 64, 960)}[kind]
        ops = [(_cn(g, m, k), _cn(g, k, n)) for _ in range(2)]
        return [lambda h, a=a, b=b: [h.zgemm("N", "N", a, b)] for a, b in ops]
    if kind.startswith("filter"):
        n, m = 501, 48
        precision = kind.split()[1]
        out = []
        for _ in range(2):
            C = _cn(g, n, n)
            C = gevp.colmajor(0.5 * (C + C.mH))
            v = [_cn(g, n, m, torch.complex64) for _ in range(3)]
            co = [torch.rand(m, generator=g, device="cuda", dtype=torch.float64) for _ in range(4)]
            out.append(lambda h, C=C, v=v, co=co: [h.filter_gemm(precision, C, *v, *co)])
        return out
    if kind == "trsm":
        ops = []
        for _ in range(2):
            L = torch.tril(_cn(g, 400, 400)) + 40 * torch.eye(400, device="cuda")
            ops.append((gevp.colmajor(L), _cn(g, 400, 90)))
        return [lambda h, a=a, b=b: [h.trsm("L", "N", a, b)] for a, b in ops]
    ops = [(_cn(g, 700, 60), torch.rand(60, generator=g, device="cuda", dtype=torch.float64),
            torch.rand(60, generator=g, device="cuda", dtype=torch.float64)) for _ in range(2)]
    return [lambda h, x=x, l=l, w=w: list(h.backward(x, l, w)) for x, l, w in ops]


@pytest.mark.parametrize("kind", ["zgemm short", "zgemm split", "zgemm skinny cut", "filter fp32",
                                  "filter bf16x3", "trsm", "backward"])
def test_two_streams_in_turn(kind):
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    calls = _calls(gevp, kind, g)
    alone = gevp.Handle(0)
    want = [c(alone) for c in calls]
    torch.cuda.synchronize()
    h = gevp.Handle(0)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = []
    for _ in range(20):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                got.append((i, calls[i](h)))
    torch.cuda.synchronize()
    for i, out in got:
        assert all(torch.equal(a, b) for a, b in zip(out, want[i]))
    h.close()
    alone.close()
