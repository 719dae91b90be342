"""Performance cases: the work a user of the library has it do.

Each case is one pass through the public binding (``paper_1007_4400_amd.gevp``):
whole solves, cold and seeded, in the three precisions and with both filters, a
batch of k-points, and the blocks that a program calls by themselves (reduction
to standard form, Rayleigh-Ritz step, filter step, eigenvalue gradient,
thresholded matrix update).  Sizes are those of the named workloads in
``synth`` and of the tests and the benchmark, plus odd ones in between;
``draw`` spreads the same kinds over their ranges.

Inputs are built on the GPU from the seed alone: pencils with the synthetic
sequences' spectra and conditioning, seeds that are the exact eigenvectors of
the previous step (so they do not depend on the library), and a perturbation of
the size a step in the middle of an SCF run has.
"""
import math

import torch

from paper_1007_4400_amd import gevp, synth

TOL = 1e-10  # residual tolerance of every solve (the benchmark's and the tests')
EXACT_N = 1200  # largest order whose eigenproblem is solved densely for exact()

_handle = []


def handle():
    """The handle a program keeps for all its solves."""
    if not _handle:
        _handle.append(gevp.Handle(0))
    return _handle[0]


# ------------------------------------------------------------------- the cases


def listed():
    return [
        # one small pencil from scratch: latency, launches and host work decide
        {"name": "solve_n256_cold", "kind": "solve", "n": 256, "nev": 16, "precision": "fp64",
         "seeded": False, "filter": "chebyshev", "spectrum": "split"},
        # an odd mid-size pencil from scratch, FP32 filter
        {"name": "solve_n1001_cold_fp32", "kind": "solve", "n": 1001, "nev": 100, "precision": "fp32",
         "seeded": False, "filter": "chebyshev", "spectrum": "cluster"},
        # one step of the medium SCF sequence in plain FP64
        {"name": "solve_n2048_seeded", "kind": "solve", "n": 2048, "nev": 205, "precision": "fp64",
         "seeded": True, "filter": "chebyshev", "spectrum": "cluster"},
        # the first, direct iteration of a large run in plain FP64
        {"name": "solve_n4096_cold", "kind": "solve", "n": 4096, "nev": 410, "precision": "fp64",
         "seeded": False, "filter": "chebyshev", "spectrum": "cluster"},
        # one step of the headline SCF sequence, split-BF16 filter
        {"name": "solve_n8192_seeded_bf16x3", "kind": "solve", "n": 8192, "nev": 820,
         "precision": "bf16x3", "seeded": True, "filter": "chebyshev", "spectrum": "cluster"},
        # a seeded step with the contour-integral filter, FP32 form
        {"name": "solve_n1100_contour", "kind": "solve", "n": 1100, "nev": 110, "precision": "fp32",
         "seeded": True, "filter": "contour", "spectrum": "cluster"},
        # one SCF step of a set of uneven k-points solved together
        {"name": "batched_8_kpoints", "kind": "batched", "count": 8, "nmin": 1500, "nmax": 3000,
         "precision": "bf16x3", "seeded": True},
        # reduction of one pencil to standard form by the blocks: Cholesky, two solves
        {"name": "reduce_n3001", "kind": "reduce", "n": 3001},
        # Rayleigh-Ritz step of the headline block: two products, the small
        # eigensolve, and the weighted projector of its eigenvectors
        {"name": "rayleigh_ritz_n8192_m948", "kind": "ritz", "n": 8192, "m": 948},
        # one split-BF16 filter step at the headline's average active width
        {"name": "filter_n8192_m645_bf16x3", "kind": "filter", "n": 8192, "m": 645,
         "precision": "bf16x3"},
        # eigenvalue gradient at the differentiation workload's size
        {"name": "backward_n4096_nev410", "kind": "backward", "n": 4096, "nev": 410},
        # thresholded partial update of the headline Hamiltonian
        {"name": "update_n8192", "kind": "update", "n": 8192, "p_t": 0.1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batched", "reduce", "ritz", "filter", "backward",
                       "update"])
    if kind == "solve":
        n = _log(rng, 64, 4096)
        contour = n <= 2048 and rng.random() < 0.2
        return {"kind": "solve", "n": n, "nev": max(1, int(n * rng.uniform(0.04, 0.11))),
                "precision": rng.choice(["fp64", "fp32", "bf16x3"]),
                "seeded": contour or rng.random() < 0.6,
                "filter": "contour" if contour else "chebyshev",
                "spectrum": "split" if n < 512 else "cluster"}
    if kind == "batched":
        nmin = _log(rng, 200, 1500)
        return {"kind": "batched", "count": rng.randint(3, 8), "nmin": nmin,
                "nmax": int(nmin * rng.uniform(1.2, 2.0)),
                "precision": rng.choice(["fp64", "fp32", "bf16x3"]), "seeded": rng.random() < 0.7}
    if kind == "reduce":
        return {"kind": "reduce", "n": _log(rng, 100, 6000)}
    if kind == "ritz":
        n = _log(rng, 300, 8192)
        return {"kind": "ritz", "n": n, "m": max(1, int(n * rng.uniform(0.05, 0.115)))}
    if kind == "filter":
        n = _log(rng, 256, 8192)
        return {"kind": "filter", "n": n, "m": max(1, int(n * rng.uniform(0.03, 0.115))),
                "precision": rng.choice(["fp32", "bf16x3"])}
    if kind == "backward":
        n = _log(rng, 128, 8192)
        return {"kind": "backward", "n": n, "nev": max(1, int(n * rng.uniform(0.03, 0.1)))}
    return {"kind": "update", "n": _log(rng, 200, 8192), "p_t": round(rng.uniform(0.02, 0.5), 3)}


# ----------------------------------------------------------------- preparation


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _workload(n, nev, spectrum, shift=0.0):
    base = synth.SMALL if spectrum == "split" else synth.LARGE
    scale = synth.SMALL.lscale if spectrum == "split" else 1.1 / math.sqrt(n)
    return synth.Workload("case", n, nev, 12, spectrum, scale, base.eps0, base.decay, shift)


def _pencil(n, nev, spectrum, seeded, block, seed, shift=0.0):
    """A pencil and, for a seeded solve, the exact lowest eigenvectors of the
    pencil one step earlier (the fifth step of a run, a middle one)."""
    wl = _workload(n, nev, spectrum, shift)
    if not seeded:
        A, B, _, _, _ = synth.make_pencil_torch(wl, seed)
        return gevp.colmajor(A), gevp.colmajor(B), None
    A, B, _, _, g, (_, X0) = synth.make_pencil_torch(wl, seed, exact_nev=block)
    A = A + synth.eps(wl, 5) * synth.unit_hermitian_torch(n, g)
    return gevp.colmajor(A), gevp.colmajor(B), gevp.colmajor(X0)


def _sizes(case):
    """Orders of a batch: spread evenly over [nmin, nmax], uneven on purpose."""
    c = case["count"]
    return [case["nmin"] + (case["nmax"] - case["nmin"]) * ((5 * i + 2) % c) // max(1, c - 1) + (i % 3)
            for i in range(c)]


def _hermitian(n, g):
    G = torch.randn(n, n, generator=g, device="cuda", dtype=torch.complex128)
    return 0.5 * (G + G.conj().T)


def _orthonormal(n, m, g):
    return torch.linalg.qr(torch.randn(n, m, generator=g, device="cuda", dtype=torch.complex128))[0]


def prepare(case, seed):
    h = handle()
    kind = case["kind"]
    if kind == "solve":
        n, nev = case["n"], case["nev"]
        opts = gevp.make_opts(precision=case["precision"], filter=case["filter"])
        kx = h.block_size(n, nev, opts)  # guard vectors too: they seed the next step
        A, B, X0 = _pencil(n, nev, case["spectrum"], case["seeded"], kx, seed)
        return {"kind": kind, "A": A, "B": B, "X0": X0, "nev": nev, "opts": opts,
                "kx": kx if case["seeded"] else nev}
    if kind == "batched":
        opts = gevp.make_opts(precision=case["precision"])
        probs = []
        for i, n in enumerate(_sizes(case)):
            nev = max(1, round(0.1 * n))
            kx = h.block_size(n, nev, opts)
            A, B, X0 = _pencil(n, nev, "split" if n < 512 else "cluster", case["seeded"], kx,
                               1000 * int(seed) + i, shift=0.1 * (i % 5) - 0.2)
            p = {"A": A, "B": B, "nev": nev, "kx": kx if case["seeded"] else nev}
            if X0 is not None:
                p["X0"] = X0
            probs.append(p)
        return {"kind": kind, "problems": probs, "opts": opts}
    g = _gen(seed)
    if kind == "reduce":
        n = case["n"]
        A, B, _, _, _ = synth.make_pencil_torch(_workload(n, max(1, n // 10), "cluster"), seed)
        return {"kind": kind, "A": gevp.colmajor(A), "B": gevp.colmajor(B)}
    if kind == "ritz":
        n, m = case["n"], case["m"]
        C = _hermitian(n, g)
        w = torch.sort(torch.rand(m, generator=g, device="cuda", dtype=torch.float64)).values
        return {"kind": kind, "C": gevp.colmajor(C), "Y": gevp.colmajor(_orthonormal(n, m, g)), "w": w}
    if kind == "filter":
        n, m = case["n"], case["m"]
        C = _hermitian(n, g) / math.sqrt(n)
        v = [torch.randn(m, n, generator=g, device="cuda", dtype=torch.complex64).mT for _ in range(3)]
        co = [torch.rand(m, generator=g, device="cuda", dtype=torch.float64) + 0.5 for _ in range(4)]
        co[2] = -co[2]
        return {"kind": kind, "C": gevp.colmajor(C), "G": v[0], "P": v[1], "R": v[2], "co": co,
                "precision": case["precision"]}
    if kind == "backward":
        n, nev = case["n"], case["nev"]
        X = _orthonormal(n, nev, g)
        lam = torch.sort(torch.rand(nev, generator=g, device="cuda", dtype=torch.float64) * 3 - 3).values
        kT = 0.01  # Fermi-Dirac weights, the level below the last computed state
        w = 1.0 / (1.0 + torch.exp(torch.clamp((lam - lam[int(0.92 * nev)]) / kT, -300, 300)))
        return {"kind": kind, "X": gevp.colmajor(X), "lam": lam, "w": w}
    # update: the matrix in use and two newly generated ones, taken in turn
    n = case["n"]
    wl = synth.update_scaled(synth.UPDATE_LARGE, n, steps=2)
    A0, A1, A2 = synth.update_sequence_torch(wl, seed)
    return {"kind": kind, "A": gevp.colmajor(A0.contiguous()), "new": [gevp.colmajor(A1), gevp.colmajor(A2)],
            "turn": 0, "mask": gevp.empty_mask(n, device="cuda").zero_(), "p_t": case["p_t"]}


# ------------------------------------------------------------------- one pass


def run(s):
    h = handle()
    kind = s["kind"]
    if kind == "solve":
        lam, X, _, _ = h.solve(s["A"], s["B"], s["nev"], X0=s["X0"], tol=TOL, kx=s["kx"], opts=s["opts"],
                               want_resid=False)
        k = s["nev"]  # the guard pairs are a seed, converged to nothing in particular
        return {"lam": lam[:k], "X": X[:, :k]}
    if kind == "batched":
        out = h.solve_batched(s["problems"], tol=TOL, opts=s["opts"])
        return [{"lam": o[0][:p["nev"]], "X": o[1][:, :p["nev"]]} for o, p in zip(out, s["problems"])]
    if kind == "reduce":
        L, _ = h.potrf(s["B"])
        W = h.trsm("L", "N", L, s["A"])
        return {"L": L, "C": h.trsm("R", "C", L, W)}
    if kind == "ritz":
        W = h.zgemm("N", "N", s["C"], s["Y"])
        H = h.zgemm("C", "N", s["Y"], W)
        theta, Z = h.heev(H)
        P, _ = h.backward(Z, theta, s["w"], want_dB=False)  # Z diag(w) Z^H
        return {"W": W, "H": H, "theta": theta, "P": P}
    if kind == "filter":
        return h.filter_gemm(s["precision"], s["C"], s["G"], s["P"], s["R"], *s["co"])
    if kind == "backward":
        dA, dB = h.backward(s["X"], s["lam"], s["w"])
        return {"dA": dA, "dB": dB}
    new = s["new"][s["turn"]]
    s["turn"] ^= 1
    info = h.update_thresholded(s["A"], new, s["p_t"], mask=s["mask"])
    return {"A": s["A"], "mask": s["mask"], "delta": info["delta"], "updated": info["updated"]}


# ------------------------------------------------------------- work and values


def _solve_work(n, m, seeded):
    # Cholesky, two-sided reduction, one projection W = C Y and its Gram
    # product, back-transformation, the two residual products; A, B (lower
    # triangles), the seed in and the vectors out
    flops = (4 / 3 + 4) * n**3 + 8 * n * n * m + 4 * n * m * m + 4 * n * n * m + 16 * n * n * m
    return 16 * (n * n + n * m * (2 if seeded else 1)), flops


def work(case):
    kind = case["kind"]
    if kind == "solve":
        b, f = _solve_work(case["n"], case["nev"], case["seeded"])
    elif kind == "batched":
        w = [_solve_work(n, max(1, round(0.1 * n)), case["seeded"]) for n in _sizes(case)]
        b, f = sum(x[0] for x in w), sum(x[1] for x in w)
    elif kind == "reduce":
        n = case["n"]
        b, f = 16 * 3.5 * n * n, (4 / 3 + 4 + 4) * n**3  # A, half of B in; L and C out
    elif kind == "ritz":
        n, m = case["n"], case["m"]
        b = 16 * (n * n + 2 * n * m + 2 * m * m)
        f = 8 * n * n * m + 8 * n * m * m + (16 / 3 + 8) * m**3 + 8 * m**3
    elif kind == "filter":
        n, m = case["n"], case["m"]
        b, f = 16 * n * n + 8 * 4 * n * m, 8 * n * n * m
    elif kind == "backward":
        n, k = case["n"], case["nev"]
        b, f = 16 * (n * k + 2 * n * n), 2 * 8 * n * n * k
    else:
        n = case["n"]
        b, f = 16 * 2 * (n * n / 2) + 16 * 0.5 * (n * n / 2) + n * n / 8, 6 * n * n / 2
    return {"bytes": float(b), "flops": float(f)}


def _eig_exact(A, B, nev):
    """Lowest nev pairs, B-orthonormal, the largest entry of a vector real and
    positive, by dense factorisations on the host."""
    A, B = A.cpu(), B.cpu()
    A = torch.tril(A) + torch.tril(A, -1).mH
    B = torch.tril(B) + torch.tril(B, -1).mH
    L = torch.linalg.cholesky(B)
    W = torch.linalg.solve_triangular(L, A, upper=False)
    C = torch.linalg.solve_triangular(L, W.mH.contiguous(), upper=False)
    lam, Z = torch.linalg.eigh(0.5 * (C + C.mH))
    X = torch.linalg.solve_triangular(L.mH.contiguous(), Z[:, :nev].contiguous(), upper=True)
    top = X.gather(0, X.abs().argmax(0, keepdim=True))
    return {"lam": lam[:nev], "X": X * (top.abs() / top)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve" and case["n"] > EXACT_N or kind == "batched" and case["nmax"] > EXACT_N // 2:
        return None
    s = prepare(case, seed)
    if kind == "solve":
        return _eig_exact(s["A"], s["B"], s["nev"])
    if kind == "batched":
        return [_eig_exact(p["A"], p["B"], p["nev"]) for p in s["problems"]]
    if kind == "reduce":
        A, B = s["A"].cpu(), s["B"].cpu()
        L = torch.linalg.cholesky(B)
        W = torch.linalg.solve_triangular(L, A.contiguous(), upper=False)
        C = torch.linalg.solve_triangular(L, W.mH.contiguous(), upper=False).mH
        return {"L": L, "C": C.resolve_conj()}
    if kind == "ritz":
        W = s["C"] @ s["Y"]
        H = s["Y"].mH.contiguous() @ W
        theta, Z = torch.linalg.eigh((0.5 * (H + H.mH)).cpu())
        Z = Z.cuda()
        return {"W": W, "H": H, "theta": theta, "P": (Z * s["w"]) @ Z.mH.contiguous()}
    if kind == "filter":
        al, be, ga, de = s["co"]
        G, P, R = (s[k].to(torch.complex128) for k in "GPR")
        return al * (s["C"] @ G) + be * G + ga * P + de * R
    if kind == "backward":
        X, XH = s["X"], s["X"].mH.contiguous()
        return {"dA": (X * s["w"]) @ XH, "dB": -((X * (s["w"] * s["lam"])) @ XH)}
    A, D = s["A"], s["new"][0] - s["A"]
    d2 = torch.tril(D.real * D.real + D.imag * D.imag)
    take = torch.tril(d2 > (s["p_t"] * s["p_t"]) * d2.max())
    return {"A": torch.where(take, s["new"][0], A), "mask": None, "delta": float(d2.max().sqrt()),
            "updated": None}
