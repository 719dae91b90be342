"""Threads with a handle and a stream of their own: a solve waits for another
thread's single-launch kernels, which may share the device with it only so far, but
not for the rest of its solve; and what it computes does not depend on it."""
import threading
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pencil(n, k, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    G = torch.randn(n, n, generator=g, device="cuda", dtype=torch.complex128)
    A = (0.5 / n**0.5) * (G + G.mH)
    G = torch.randn(n, n, generator=g, device="cuda", dtype=torch.complex128)
    B = (0.1 / n**0.5) * (G + G.mH) + torch.eye(n, device="cuda")
    X0 = torch.linalg.qr(torch.randn(n, k, generator=g, device="cuda", dtype=torch.complex128))[0]
    return [t.mT.contiguous().mT for t in (A, B, X0)]


class _Solver:
    """One sweep of a seeded solve, again and again."""

    def __init__(self, gevp, n, nev, seed):
        self.gevp, self.nev = gevp, nev
        self.h = gevp.Handle(0)
        self.opts = gevp.make_opts(maxit=1)
        self.kx = self.h.block_size(n, nev, self.opts)
        self.A, self.B, self.X0 = _pencil(n, self.kx, seed)
        self.stream = torch.cuda.Stream()
        torch.cuda.synchronize()

    def __call__(self):
        with torch.cuda.stream(self.stream):
            try:
                self.h.solve(self.A, self.B, self.nev, X0=self.X0, kx=self.kx, opts=self.opts)
            except self.gevp.GevpError as e:  # one sweep is not enough
                assert e.status == self.gevp.GEVP_ERR_NOCONV


def test_small_solves_do_not_wait_for_large_ones():
    """The large one's eigensolve wants 89 work-groups of the device, the small one's
    Lanczos steps 256, which are not to be had at once.  Were the share kept from a
    solve's start to its first sweep, the threads would take turns, one small solve
    a large one."""
    from paper_1007_4400_amd import gevp

    large, small = _Solver(gevp, 6144, 600, 1), _Solver(gevp, 2048, 100, 2)
    large(), small()
    rounds, done = 10, threading.Event()

    def run():
        for _ in range(rounds):
            large()
        done.set()

    t = threading.Thread(target=run)
    t0 = time.perf_counter()
    t.start()
    count = 0
    while not done.is_set():
        small()
        count += 1
    t.join()
    print(f"{rounds} large solves in {1e3 * (time.perf_counter() - t0):.0f} ms, {count} small ones beside them",
          flush=True)
    assert count >= 1.5 * rounds
    large.h.close()
    small.h.close()


@pytest.mark.parametrize("n", [257, 1100, 2048])
def test_threads_compute_what_one_does(n):
    from paper_1007_4400_amd import gevp

    nev = n // 12
    solvers = [_Solver(gevp, n, nev, s) for s in range(4)]
    full = gevp.make_opts(precision="bf16x3")

    def solve(s, out, i):
        with torch.cuda.stream(s.stream):
            for seed in (None, s.X0):
                lam, X, _, _ = s.h.solve(s.A, s.B, nev, X0=seed, tol=1e-8, kx=s.kx, opts=full)
                out[i].append((lam, X))

    alone, together = [[] for _ in solvers], [[] for _ in solvers]
    for i, s in enumerate(solvers):
        solve(s, alone, i)
    for r in range(3):
        together = [[] for _ in solvers]
        ts = [threading.Thread(target=solve, args=(s, together, i)) for i, s in enumerate(solvers)]
        [t.start() for t in ts]
        [t.join() for t in ts]
        torch.cuda.synchronize()
        for a, b in zip(alone, together):
            assert len(b) == 2
            for (la, xa), (lb, xb) in zip(a, b):
                assert torch.equal(la, lb) and torch.equal(xa, xb)
    for s in solvers:
        s.h.close()
