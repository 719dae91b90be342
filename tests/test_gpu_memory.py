"""Device memory running short: the scratch of the residue products, which the
library can do without, gives way to what a call must have, and a shortage that is
over leaves no trace in later calls."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GIB = 2**30


def _cn(g, m, n):
    return torch.randn(n, m, generator=g, device="cuda", dtype=torch.complex128).mT


def _leave(nbytes):
    """A block of device memory that leaves about nbytes free."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    return torch.empty(max(1, free - nbytes), dtype=torch.uint8, device="cuda")


@pytest.fixture()
def setup():
    from paper_1007_4400_amd import gevp

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    n = 4096
    A, B = _cn(g, n, n), _cn(g, n, n)
    out = gevp.empty_colmajor(n, n, device="cuda")
    h = gevp.Handle(0)
    yield gevp, h, A, B, out
    h.close()
    torch.cuda.empty_cache()


def test_scratch_gives_way_to_a_solve(setup):
    gevp, h, A, B, out = setup
    n, nev = 4096, 64
    need = h.workspace_size(n, nev) - 6 * 128 * 2**20  # the split-K slots of a caller's buffer
    H = gevp.colmajor(0.5 * (A + A.mH) + 200 * torch.eye(n, device="cuda"))
    X = gevp.empty_colmajor(n, h.block_size(n, nev), device="cuda")
    del X
    eye = gevp.colmajor(torch.eye(n, dtype=torch.complex128, device="cuda"))
    h.zgemm("N", "N", A, B, out=out)  # the handle now holds the scratch of this product
    block = _leave(need - GIB // 2)
    print(f"solve needs {need / GIB:.2f} GiB, free {torch.cuda.mem_get_info()[0] / GIB:.2f} GiB", flush=True)
    # (also the split-K buffers: none is left for them, k stays whole)
    lam, _, _, info = h.solve(H, eye, nev, opts=gevp.make_opts(skip_final_residual=True))
    del block
    torch.cuda.empty_cache()
    h2 = gevp.Handle(0)
    ref, _, _, _ = h2.solve(H, eye, nev, opts=gevp.make_opts(skip_final_residual=True))
    h2.close()
    assert ((lam[:nev] - ref[:nev]).abs() <= 1e-9 * 300).all()


def test_a_shortage_ends_with_the_call(setup):
    gevp, h, A, B, out = setup
    first = h.zgemm("N", "N", A, B).clone()
    h.set_workspace(None)  # gives everything back
    block = _leave(GIB // 4)
    h.zgemm("N", "N", A, B, out=out)  # no scratch: the FP64 kernels
    short = (out - first).abs().max().item()
    del block
    torch.cuda.empty_cache()
    again = h.zgemm("N", "N", A, B, out=out)
    assert 0 < short <= 1e-10
    assert torch.equal(again, first)


@pytest.mark.parametrize("quarters", [4, 6, 8, 10, 12])
def test_scratch_leaves_room_for_the_runtime(setup, quarters):
    """What a call can do without never takes the device's last bytes: a kernel's code
    is loaded at its first launch, which fails where nothing is left."""
    gevp, h, A, B, out = setup
    block = _leave(quarters * GIB // 4)
    before = torch.cuda.mem_get_info()[0]
    h.zgemm("N", "N", A, B, out=out)
    h.zgemm("C", "N", A[:, :64], B[:, :64])  # a cut k
    torch.cuda.synchronize()
    left = torch.cuda.mem_get_info()[0]
    del block
    print(f"free {before / GIB:.2f} GiB, left {left / GIB:.2f} GiB", flush=True)
    assert left >= min(before, GIB // 2) - GIB // 16
