"""Products and FP32 filter steps captured by a handle that has no split-K buffer
yet: nothing may be allocated then, so the k range stays whole.  Each replay, with
the handle's eager work between them, gives what the capture computed, and that is
the product within a few roundings of its sum of sizes."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cn(g, m, n, dtype=torch.complex128):
    return torch.randn(n, m, generator=g, device="cuda", dtype=dtype).mT


def _replays(graph, out, eager):
    seen = []
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        seen.append(out.clone())
        eager()
        torch.cuda.synchronize()
    assert all(torch.equal(s, seen[0]) for s in seen)
    return seen[0]


# k ranges cut in parts, long ones of skinny products, large products (residues)
@pytest.mark.parametrize("m,n,k", [(256, 48, 256), (600, 64, 960), (300, 200, 2000), (1536, 1024, 1536)])
def test_product_on_a_fresh_handle(m, n, k):
    from paper_1007_4400_amd import gevp

    print(f"capture {m} x {n} x {k}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    A, B = _cn(g, m, k), _cn(g, k, n)
    D = gevp.empty_colmajor(m, n, device="cuda")
    h = gevp.Handle(0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        h.zgemm("N", "N", A, B, out=D)
    got = _replays(graph, D, lambda: h.zgemm("N", "N", A, B))
    ref = (A.cpu() @ B.cpu()).cuda()
    assert ((got - ref).abs() <= 32 * 2.0**-53 * k**0.5 * (A.abs() @ B.abs())).all()
    del graph
    h.close()


def test_filter_step_without_a_split_buffer():
    from paper_1007_4400_amd import gevp

    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    n, m = 501, 48
    C = _cn(g, n, n)
    C = gevp.colmajor(0.5 * (C + C.mH))
    v = [_cn(g, n, m, torch.complex64) for _ in range(3)]
    co = [torch.rand(m, generator=g, device="cuda", dtype=torch.float64) for _ in range(4)]
    h = gevp.Handle(0)
    h.filter_gemm("bf16x3", C, *v, *co)  # a workspace, no split-K buffer
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = h.filter_gemm("fp32", C, *v, *co)
    got = _replays(graph, out, lambda: h.filter_gemm("fp32", C, *v, *co))
    G, P, R = (x.to(torch.complex128) for x in v)
    ref = (C.cpu() @ G.cpu()).cuda() * co[0] + G * co[1] + P * co[2] + R * co[3]
    size = (C.abs() @ G.abs()) * co[0] + G.abs() * co[1] + P.abs() * co[2] + R.abs() * co[3]
    # operands and accumulators in FP32
    assert ((got - ref).abs() <= 8 * 2.0**-24 * n**0.5 * size).all()
    del graph
    h.close()
