"""The work this framework is used for, as cases that can be timed.

Each case goes through a public entry point of ``paper_1404_1768_amd`` as a
program that owns the pencil would call it.  ``listed()`` names the cases,
``draw(rng)`` gives more of the same ranges, ``prepare`` makes what the program
holds before the call, ``run`` is one pass, ``work`` what the pass cannot do
without and ``exact`` its result in plain 64-bit torch.

Pencils follow the generator of the tests and the benchmark: ``A = P D Q``,
``B = P Q`` with ``P, Q = I + c G``, so that the eigenvalues inside the circle
are entries of ``D``, their right eigenvectors columns of ``Q^-1`` and their
left ones columns of ``P^-*``.  They are built on the GPU.
"""
import math

import numpy as np
import torch

import paper_1404_1768_amd as fm

C128 = torch.complex128


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: a few small products, as a program makes between
        # larger steps (latency and the call itself count)
        dict(name="gemm_small", kind="gemm", trans=0, M=64, N=33, K=64, batch=3),
        # inner products of an n x m block (Gram and projection products U^* V
        # of a subspace method): a small output, a long sum, odd sizes
        dict(name="gemm_gram", kind="gemm", trans=2, M=157, N=157, K=4001, batch=1),
        # the factorisation of the shifted matrices on its own, odd order
        dict(name="getrf", kind="getrf", n=1003, batch=16),
        # solves with given factors, many right-hand sides
        dict(name="getrs", kind="getrs", n=1000, nrhs=160, batch=8, trans=0),
        # one more filter on cached factors (an iteration of the caller's own),
        # order and block of the Table 1 problem BFW782
        dict(name="filter_fp64", kind="filter", n=782, m=40, nodes=16, prec="fp64", fresh=False),
        # a new pencil in mixed precision: factor, solve, refine to full accuracy
        dict(name="filter_mixed", kind="filter", n=2003, m=64, nodes=16, prec="mixed", fresh=True),
        # orthonormalisation and oblique projection of a filtered block
        # (the benchmark's order and subspace size)
        dict(name="project", kind="project", n=4000, m=160),
        # whole solves: the smallest workload (FP64) ...
        dict(name="solve_small", kind="solve", n=200, m=30, s=20, nodes=16, prec="fp64"),
        # ... and the benchmark's (mixed)
        dict(name="solve_large", kind="solve", n=4000, m=160, s=100, nodes=32, prec="mixed"),
        # a sparse pencil with the order and bandwidth of the MHD4800 stand-in
        dict(name="solve_csr", kind="csr", n=4800, m=40, s=15, nodes=16, wp=11, wq=11),
        # many pencils of uneven order factored and filtered in lockstep
        dict(name="batch", kind="batch", count=24, lo=256, hi=1536, nodes=16, prec="fp64", sweeps=0),
        # eigenvalues and their gradient (forward and backward of the autograd
        # function) on the adjoint workload's recipe
        dict(name="adjoint", kind="adjoint", n=2048, m=64, s=40, nodes=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "getrf", "getrs", "filter", "filter", "project", "solve",
                       "solve", "csr", "batch", "adjoint"])
    nodes = rng.choice([8, 16, 16, 32])
    prec = rng.choice(["fp64", "mixed"])
    if kind == "gemm":
        if rng.random() < 0.5:  # an inner product of tall blocks, or an n x m product
            return dict(kind=kind, trans=2, M=_log(rng, 16, 256), N=_log(rng, 16, 256),
                        K=_log(rng, 200, 8000), batch=rng.choice([1, 1, 2]))
        return dict(kind=kind, trans=rng.choice([0, 2]), M=_log(rng, 17, 2000),
                    N=_log(rng, 16, 256), K=_log(rng, 16, 2000), batch=rng.randint(1, 16))
    if kind == "getrf":
        return dict(kind=kind, n=_log(rng, 64, 2100), batch=rng.randint(1, 32))
    if kind == "getrs":
        return dict(kind=kind, n=_log(rng, 64, 1600), nrhs=_log(rng, 3, 256),
                    batch=rng.randint(1, 16), trans=rng.choice([0, 2]))
    if kind == "filter":
        n = _log(rng, 128, 2500)
        return dict(kind=kind, n=n, m=_log(rng, 12, max(16, min(160, n // 4))), nodes=nodes,
                    prec=prec, fresh=rng.random() < 0.5)
    if kind == "project":
        n = _log(rng, 200, 6000)
        return dict(kind=kind, n=n, m=_log(rng, 12, max(16, min(256, n // 6))))
    if kind == "solve":
        n = _log(rng, 150, 4000)
        s = max(6, n // rng.choice([10, 20, 40]))
        s = min(s, 100)
        return dict(kind=kind, n=n, m=max(s + 10, s * 8 // 5), s=s, nodes=rng.choice([16, 32]),
                    prec=prec)
    if kind == "csr":
        return dict(kind=kind, n=_log(rng, 398, 4800), m=rng.randint(24, 40), s=rng.randint(6, 15),
                    nodes=16, wp=rng.randint(1, 14), wq=rng.randint(1, 14))
    if kind == "batch":
        lo = rng.choice([64, 128, 256])
        return dict(kind=kind, count=rng.randint(3, 24), lo=lo, hi=_log(rng, 300, 1536), nodes=16,
                    prec=prec, sweeps=0 if prec == "fp64" else 2)
    n = _log(rng, 200, 2048)
    s = max(6, min(40, n // 25))
    return dict(kind=kind, n=n, m=max(s + 10, s * 8 // 5), s=s, nodes=rng.choice([16, 32]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 11)


def _gauss(g, *shape):
    """Complex Gaussian, unit variance."""
    return torch.randn(*shape, dtype=C128, device="cuda", generator=g)


def _annulus(g, count, r1, r2, center):
    """Points area-uniform in r1 <= |z - center| < r2."""
    u = torch.rand(2, count, dtype=torch.float64, device="cuda", generator=g)
    return center + torch.polar(torch.sqrt(r1 * r1 + u[0] * (r2 * r2 - r1 * r1)),
                                2.0 * math.pi * u[1])


def _band(n, w):
    i = torch.arange(n, device="cuda")
    return (i[:, None] - i[None, :]).abs() <= w


def _outer(n, m, s, nodes):
    """Outer radius of the annulus of the other eigenvalues: 10, or less where
    the block's m - s spare columns would otherwise fall on eigenvalues that the
    filter damps below about 1e-8 (a block of that many columns is then rank
    deficient: a program would take a smaller one)."""
    r = 10.0 ** (8.0 / nodes)
    return min(10.0, math.sqrt(1.69 + (r * r - 1.69) * (n - s) / max(1, m - s)))


def _pencil(g, n, m, s, center, c=0.05, inside=0.9, outside=(1.3, 10.0), wp=None, wq=None):
    """A = P D Q, B = P Q with s eigenvalues in |z - center| < inside, the rest
    in the annulus; wp, wq: half bandwidths of P and Q (dense if None)."""
    d = torch.cat([_annulus(g, s, 0.0, inside, center),
                   _annulus(g, n - s, outside[0], outside[1], center)])
    d = d[torch.randperm(n, device="cuda", generator=g)]
    eye = torch.eye(n, dtype=C128, device="cuda")
    P, Q = _gauss(g, n, n), _gauss(g, n, n)
    for M, w in ((P, wp), (Q, wq)):
        if w is None:
            M.mul_(c / math.sqrt(n))
        else:
            M.mul_(c / math.sqrt(2 * w + 1)).mul_(_band(n, w))
        M.add_(eye)
    return dict(P=P, Q=Q, d=d, A=(P * d[None, :]) @ Q, B=P @ Q, V=_gauss(g, n, m))


def _found(g, case, **bands):
    """The pencil of a solve: the eigenvalues inside are the ones looked for."""
    n, m, s = case["n"], case["m"], case["s"]
    return _pencil(g, n, m, s, _center(case), outside=(1.3, _outer(n, m, s, case["nodes"])),
                   **bands)


def _center(case):
    return 1.0 + 1.0j if case["n"] >= 3000 else 0.25 - 0.5j


def _prec(case):
    return fm.MIXED if case["prec"] == "mixed" else fm.FP64


def _csr(M, w):
    """(rowptr, col, val) of the band |i - j| <= w of M."""
    keep = _band(M.shape[0], w)
    rp = torch.zeros(M.shape[0] + 1, dtype=torch.int32, device="cuda")
    rp[1:] = keep.sum(1).cumsum(0)
    col = keep.nonzero()[:, 1].to(torch.int32).contiguous()
    return rp, col, M[keep].contiguous()


def _batch_pencils(case, g, seed):
    r = np.random.default_rng(int(seed) + 17)
    # the orders are the program's own and stay; the pencils change with the seed
    ro = np.random.default_rng(case["count"] * 100003 + case["lo"] * 101 + case["hi"])
    ns = [int(x) for x in ro.integers(case["lo"], max(case["lo"] + 2, case["hi"]) + 1,
                                      case["count"])]
    cs = [complex(a, b) for a, b in r.uniform(-2.0, 2.0, (case["count"], 2))]
    out = []
    for n, c in zip(ns, cs):
        s = max(2, n // 20)
        p = _pencil(g, n, 2 * s, s, c)
        p["center"] = c
        out.append(p)
    return ns, cs, out


def _blocks(case, seed):
    """Inputs of the products: op(A), B of the stated sizes."""
    g, b = _gen(seed), case["batch"]
    sh = (case["M"], case["K"]) if case["trans"] == 0 else (case["K"], case["M"])
    return _gauss(g, b, *sh), _gauss(g, b, case["K"], case["N"])


def _filtered(case, seed):
    """A pencil and a block as a filter leaves it: columns over a subspace whose
    strengths fall from 1 to 1e-3."""
    g = _gen(seed)
    n, m = case["n"], case["m"]
    p = _pencil(g, n, m, max(1, m // 2), _center(case))
    dec = torch.logspace(0, -3, m, dtype=torch.float64, device="cuda").to(C128)
    p["U"] = ((_gauss(g, n, m) / math.sqrt(n)) * dec[None, :]) @ _gauss(g, m, m)
    return p


def prepare(case, seed):
    k, g = case["kind"], _gen(seed)
    if k == "gemm":
        A, B = _blocks(case, seed)
        C = torch.empty(case["batch"], case["M"], case["N"], dtype=C128, device="cuda")
        return dict(kind=k, A=A, B=B, C=C, trans=case["trans"])
    if k == "getrf":
        M = _gauss(g, case["batch"], case["n"], case["n"])
        return dict(kind=k, M=M, F=torch.empty_like(M))
    if k == "getrs":
        LU = _gauss(g, case["batch"], case["n"], case["n"])
        R = _gauss(g, case["batch"], case["n"], case["nrhs"])
        piv, _ = fm.zgetrf_batched(LU)
        return dict(kind=k, LU=LU, piv=piv, R=R, X=torch.empty_like(R), trans=case["trans"])
    if k == "project":
        p = _filtered(case, seed)
        plan = fm.Plan(case["n"], case["m"], _center(case), 1.0, 1)
        return dict(kind=k, plan=plan, A=p["A"], B=p["B"], U=p["U"])
    if k == "batch":
        ns, cs, ps = _batch_pencils(case, g, seed)
        b = fm.Batch(ns, [p["V"].shape[1] for p in ps], cs, [1.0] * len(ns), case["nodes"],
                     prec=_prec(case))
        return dict(kind=k, batch=b, A=[p["A"] for p in ps], B=[p["B"] for p in ps],
                    V=[p["V"] for p in ps], sweeps=case["sweeps"])
    n, m, c = case["n"], case["m"], _center(case)
    if k == "csr":
        p = _found(g, case, wp=case["wp"], wq=case["wq"])
        w = case["wp"] + case["wq"]
        plan = fm.Plan(n, m, c, 1.0, case["nodes"])
        return dict(kind=k, plan=plan, A=_csr(p["A"], w), B=_csr(p["B"], w), V=p["V"])
    if k == "filter":
        p = _pencil(g, n, m, max(1, m // 2), c)
        plan = fm.Plan(n, m, c, 1.0, case["nodes"], prec=_prec(case))
        if not case["fresh"]:  # a plan that has its factors
            plan.filter(p["A"], p["B"], p["V"])
        return dict(kind=k, plan=plan, A=p["A"], B=p["B"], V=p["V"], fresh=case["fresh"])
    if k == "solve":
        p = _found(g, case)
        plan = fm.Plan(n, m, c, 1.0, case["nodes"], prec=_prec(case))
        return dict(kind=k, plan=plan, A=p["A"], B=p["B"], V=p["V"])
    p = _found(g, case)
    plan = fm.Plan(n, m, c, 1.0, case["nodes"])
    return dict(kind=k, plan=plan, A=p["A"].requires_grad_(), B=p["B"].requires_grad_(),
                V=p["V"])


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _pairs(r):
    """A solve's eigenvalues and eigenvectors, by ascending real part (the
    solver's own order carries no meaning).  Its residuals are left out: they
    measure the rounding, not the pencil."""
    order = np.argsort(r.lam.real)
    return dict(lam=r.lam[order], X=r.X[:, torch.from_numpy(order).to(r.X.device)], flag=r.flag)


def run(st):
    k = st["kind"]
    if k == "gemm":
        return fm.zgemm_batched(st["A"], st["B"], st["C"], 1.0, 0.0, st["trans"])
    if k == "getrf":
        st["F"].copy_(st["M"])  # factored in place: the program keeps its matrix
        piv, info = fm.zgetrf_batched(st["F"])
        return dict(LU=st["F"], piv=piv, info=info)
    if k == "getrs":
        st["X"].copy_(st["R"])
        return fm.zgetrs_batched(st["LU"], st["piv"], st["X"], trans=st["trans"])
    if k == "project":
        U, AU, BU, At, Bt = st["plan"].project(st["A"], st["B"], st["U"].clone())
        return dict(U=U, AU=AU, BU=BU, At=At, Bt=Bt)
    if k == "filter":
        if st["fresh"]:
            st["plan"].invalidate()  # a pencil that has not been factored yet
        return st["plan"].filter(st["A"], st["B"], st["V"], allow=(2,))
    if k == "batch":
        st["batch"].invalidate()
        return st["batch"].filter(st["A"], st["B"], st["V"], st["sweeps"])
    st["plan"].invalidate()
    if k == "csr":
        return _pairs(st["plan"].solve_csr(st["A"], st["B"], st["V"]))
    if k == "solve":
        return _pairs(st["plan"].solve(st["A"], st["B"], st["V"]))
    A, B = st["A"], st["B"]
    A.grad = B.grad = None
    lam = fm.feast_eig(A, B, st["V"], st["plan"])
    (lam.real.square() + lam.imag.square()).sum().backward()
    lam = lam.detach()
    return dict(lam=lam[torch.argsort(lam.real)], GA=A.grad, GB=B.grad)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _lu(n):
    return 8.0 / 3.0 * n ** 3


def work(case):
    """Bytes: inputs once, outputs once.  Flops: a complex multiply-add counts
    eight; LU 8/3 n^3 per matrix, solves 8 n^2 per column."""
    k = case["kind"]
    if k == "gemm":
        M, N, K, b = case["M"], case["N"], case["K"], case["batch"]
        return dict(bytes=16.0 * b * (M * K + K * N + M * N), flops=8.0 * b * M * N * K)
    if k == "getrf":
        n, b = case["n"], case["batch"]
        return dict(bytes=b * (32.0 * n * n + 4.0 * n), flops=b * _lu(n))
    if k == "getrs":
        n, r, b = case["n"], case["nrhs"], case["batch"]
        return dict(bytes=b * (16.0 * n * n + 32.0 * n * r), flops=8.0 * b * n * n * r)
    if k == "batch":
        ro = np.random.default_rng(case["count"] * 100003 + case["lo"] * 101 + case["hi"])
        ns = ro.integers(case["lo"], max(case["lo"] + 2, case["hi"]) + 1, case["count"])
        by = fl = 0.0
        for n in (float(x) for x in ns):
            m, N = 2 * max(2, n // 20), case["nodes"]
            by += 32.0 * n * n + 32.0 * n * m
            fl += N * (_lu(n) + (1 + 2 * case["sweeps"]) * 8.0 * n * n * m) + 8.0 * n * n * m
        return dict(bytes=by, flops=fl)
    n, m = float(case["n"]), float(case["m"])
    if k == "project":
        return dict(bytes=32.0 * n * n + 64.0 * n * m + 32.0 * m * m,
                    flops=16.0 * n * n * m + 32.0 * n * m * m)
    N = float(case["nodes"])
    if k == "csr":
        # band LU and three filters (two band solves each) at kl = ku = w
        w = float(case["wp"] + case["wq"])
        return dict(bytes=2 * 20.0 * n * (2 * w + 1) + 32.0 * n * m,
                    flops=N * 8.0 * n * (2 * w * w + 3 * 4 * w * m))
    solve = 8.0 * n * n * m
    if k == "filter":
        if case["fresh"]:
            f = N * _lu(n) + solve + N * solve * (3 if case["prec"] == "mixed" else 1)
            return dict(bytes=32.0 * n * n + 32.0 * n * m, flops=f)
        b = 16.0 if case["prec"] == "fp64" else 8.0
        return dict(bytes=32.0 * n * n + b * N * n * n + 32.0 * n * m,
                    flops=solve + N * solve * (1 if case["prec"] == "fp64" else 3))
    # two filters and projections (Algorithm 5 from its start block)
    f = N * _lu(n) + 2 * (N * solve + 2 * solve) + 5 * 8.0 * n * m * m
    if k == "adjoint":
        s = float(case["s"])
        return dict(bytes=64.0 * n * n + 16.0 * n * m,
                    flops=f + 3 * (N + 1) * 8.0 * n * n * s + 16.0 * n * n * s)
    if case["prec"] == "mixed":
        f += 2 * N * solve
    return dict(bytes=32.0 * n * n + 32.0 * n * m, flops=f)


# ---------------------------------------------------------------------------
# the results in plain 64-bit torch
# ---------------------------------------------------------------------------

def _weights(center, nodes):
    th = math.pi * (2.0 * torch.arange(nodes, dtype=torch.float64) + 1.0) / nodes
    z = center + torch.polar(torch.ones_like(th), th)
    return z, (z - center) / nodes


def _filter_of(p, center, nodes):
    """Q^-1 f(D) Q V: the filter of a pencil A = P D Q, B = P Q in closed form."""
    z, w = _weights(center, nodes)
    Q, V, d = p["Q"].cpu(), p["V"].cpu(), p["d"].cpu()
    f = (w[None, :] / (z[None, :] - d[:, None])).sum(1)
    return torch.linalg.solve(Q, f[:, None] * (Q @ V))


def _inside(p, center):
    """The eigenvalues inside the circle by ascending real part, and where."""
    d = p["d"].cpu()
    i = torch.nonzero((d - center).abs() < 1.0)[:, 0]
    i = i[torch.argsort(d[i].real)]
    return d[i], i


def _columns(M, i):
    """M^-1 e_j for j in i."""
    E = torch.zeros(M.shape[0], i.numel(), dtype=C128)
    E[i, torch.arange(i.numel())] = 1.0
    return torch.linalg.solve(M.cpu(), E)


def _q(U):
    """The orthonormal factor whose triangular factor has a positive diagonal."""
    Q, R = torch.linalg.qr(U)
    d = torch.diagonal(R)
    return Q * (d / d.abs())[None, :]


def exact(case, seed):
    k, g = case["kind"], _gen(seed)
    if k == "gemm":
        A, B = (x.cpu() for x in _blocks(case, seed))
        return (A if case["trans"] == 0 else A.mH) @ B
    if k == "getrf":
        M = _gauss(g, case["batch"], case["n"], case["n"]).cpu()
        LU, _ = torch.linalg.lu_factor(M)
        return dict(LU=LU, piv=None, info=None)
    if k == "getrs":
        M = _gauss(g, case["batch"], case["n"], case["n"]).cpu()
        R = _gauss(g, case["batch"], case["n"], case["nrhs"]).cpu()
        return torch.linalg.solve(M if case["trans"] == 0 else M.mH, R)
    if k == "project":
        p = _filtered(case, seed)
        A, B, U = p["A"].cpu(), p["B"].cpu(), _q(p["U"].cpu())
        AU, BU = A @ U, B @ U
        U2 = _q(BU)
        return dict(U=U, AU=AU, BU=BU, At=U2.mH @ AU, Bt=U2.mH @ BU)
    if k == "batch":
        _, _, ps = _batch_pencils(case, g, seed)
        return [_filter_of(p, p["center"], case["nodes"]) for p in ps]
    n, m, c = case["n"], case["m"], _center(case)
    if k == "csr":
        p = _found(g, case, wp=case["wp"], wq=case["wq"])
    elif k == "filter":
        return _filter_of(_pencil(g, n, m, max(1, m // 2), c), c, case["nodes"])
    else:
        p = _found(g, case)
    lam, i = _inside(p, c)
    X = _columns(p["Q"], i)
    if k == "adjoint":
        Y = _columns(p["P"].mH, i)
        GA = (Y * (2.0 * lam)[None, :]) @ X.mH
        GB = -(Y * (2.0 * lam * lam.conj())[None, :]) @ X.mH
        return dict(lam=lam, GA=GA, GB=GB)
    X = X / torch.linalg.vector_norm(X, dim=0, keepdim=True)
    big = X.gather(0, X.abs().argmax(0, keepdim=True))
    return dict(lam=lam, X=X * (big.conj() / big.abs()), flag=None)
