"""Performance cases: the calls a program makes through the public entry points.

A case is a dict of plain values:

  problem    poisson2d | poisson3d | aniso2d | fv3d | graph (N: points per side,
             for graph the number of vertices)
  call       what one pass is:
               solve    one PCG solve on a hierarchy the program keeps
               step     sparsify, then solve (the step of a gamma study, and what
                        a program does when it changes the tolerance)
               block    several right-hand sides at once
               serve    a queue of right-hand sides through the batch server
               setup    a new matrix that is already in device memory: build the
                        hierarchy there (PMIS), sparsify, solve, release it
               vcycle   the cycle alone, as the preconditioner of the caller's own
                        Krylov method
  gamma, lumping, precision, tol, adaptive, guess, relax, block_rows, nrhs,
  requests   the options of that call

Matrices are those of ``inputs.py`` (Dirichlet Poisson, rotated anisotropic Q1,
lognormal finite volumes, random graph Laplacians); right-hand sides, guesses and
the lognormal coefficients come from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1512_04629_amd import amg, inputs, serve

DEV = "cuda" if torch.cuda.is_available() else "cpu"
HOST_SETUP_ROWS = 150_000      # larger matrices are set up on the device (the same hierarchy)

_BASE = dict(precision=64, tol=1e-8, gamma=0.1, lumping="diagonal", adaptive=True, guess="zero", relax="jacobi",
             block_rows=64, nrhs=1, requests=0)


def _case(name, problem, N, call, **kw):
    c = dict(_BASE, problem=problem, N=int(N), call=call)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest system in use (the smoke size): every launch counts
        _case("poisson2d_64", "poisson2d", 64, "solve"),
        # an irregular matrix without a grid: row lengths vary, coarse levels fill in
        _case("graph_3000", "graph", 3000, "solve", tol=1e-10, gamma=0.01, adaptive=False),
        # an ordinary 3D system in a time-stepping program: the last solution is the guess
        _case("poisson3d_47_warm", "poisson3d", 47, "solve", tol=1e-10, gamma=0.01, adaptive=False, guess="warm"),
        # the benchmark step: sparsify, then solve adaptively
        _case("poisson3d_128_step", "poisson3d", 128, "step"),
        # FP32 cycle inside FP64 CG on an anisotropic 9-point operator
        _case("aniso2d_1000_fp32", "aniso2d", 1000, "solve", precision=32, tol=1e-10, gamma=0.01, adaptive=False),
        # variable coefficients: no two rows hold the same values
        _case("fv3d_100", "fv3d", 100, "solve", tol=1e-10, gamma=0.01, adaptive=False),
        # several loads of one structure: sixteen right-hand sides in a block
        _case("fv3d_96_block16", "fv3d", 96, "block", precision=32, tol=1e-10, gamma=0.01, adaptive=False, nrhs=16),
        # the solve server emptying a queue longer than its slots
        _case("serve_poisson3d_47", "poisson3d", 47, "serve", precision=32, tol=1e-10, gamma=0.01, adaptive=False,
              requests=24),
        # a new matrix for every solve: setup on the device counts
        _case("fv3d_120_setup", "fv3d", 120, "setup", gamma=0.1),
        # Algorithm 3 with its own lumping: strong neighbours
        _case("poisson3d_90_strong", "poisson3d", 90, "step", lumping="strong"),
        # the smoother of the paper's experiments
        _case("poisson3d_64_gs", "poisson3d", 64, "solve", adaptive=False, relax="hybrid_gs"),
        # one FP64 cycle, the preconditioner of somebody else's Krylov method
        _case("aniso2d_501_vcycle", "aniso2d", 501, "vcycle", gamma=0.01, adaptive=False),
    ]


def draw(rng):
    def log_n(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("solve", "solve", "solve", "step", "step", "fp32", "block", "serve", "setup", "gs", "vcycle"))
    grids = {"poisson2d": (40, 900), "poisson3d": (14, 120), "aniso2d": (48, 950), "fv3d": (14, 98)}
    if kind == "solve":
        p = rng.choice(("poisson2d", "poisson3d", "aniso2d", "fv3d", "graph"))
        N = rng.randint(1500, 4800) if p == "graph" else log_n(*grids[p])
        adaptive = p in ("poisson2d", "poisson3d") and rng.random() < 0.5
        return _case(None, p, N, "solve", tol=1e-8 if adaptive else 1e-10, gamma=rng.choice((0.0, 0.01, 0.1)),
                     adaptive=adaptive, guess=rng.choice(("zero", "warm")))
    if kind == "step":
        p = rng.choice(("poisson2d", "poisson3d"))
        lumping = rng.choice(("diagonal", "diagonal", "strong"))
        hi = 90 if (p, lumping) == ("poisson3d", "strong") else grids[p][1]
        return _case(None, p, log_n(grids[p][0], hi), "step", gamma=rng.choice((0.01, 0.1, 0.1)), lumping=lumping)
    if kind == "fp32":
        p = rng.choice(("poisson3d", "aniso2d", "fv3d"))
        return _case(None, p, log_n(*grids[p]), "solve", precision=32, tol=1e-10, gamma=0.01, adaptive=False)
    if kind == "block":
        p = rng.choice(("poisson3d", "fv3d"))
        return _case(None, p, log_n(14, 80), "block", precision=rng.choice((32, 32, 64)), tol=1e-10, gamma=0.01,
                     adaptive=False, nrhs=rng.choice((4, 5, 8, 11, 16)))
    if kind == "serve":
        p, hi = rng.choice((("poisson2d", 300), ("poisson3d", 47)))
        return _case(None, p, log_n(grids[p][0], hi), "serve", precision=rng.choice((32, 32, 64)), tol=1e-10,
                     gamma=0.01, adaptive=False, requests=rng.randint(8, 24))
    if kind == "setup":
        p = rng.choice(("poisson3d", "fv3d"))
        return _case(None, p, log_n(24, 110), "setup", gamma=rng.choice((0.0, 0.1)))
    if kind == "gs":
        p = rng.choice(("poisson2d", "poisson3d"))
        N = log_n(40, 400) if p == "poisson2d" else log_n(14, 60)
        return _case(None, p, N, "solve", adaptive=False, relax="hybrid_gs", block_rows=rng.choice((16, 64, 128)))
    p = rng.choice(("poisson3d", "aniso2d", "fv3d"))
    return _case(None, p, log_n(*grids[p]), "vcycle", precision=rng.choice((64, 64, 32)),
                 gamma=rng.choice((0.0, 0.01)), adaptive=False)


# ---- matrices ----------------------------------------------------------------

def _terms(case, seed):
    """(grid shape, z slowest; stencil terms): a term is a grid offset (slowest
    axis first) and its value, a number or a grid of values."""
    N, p = case["N"], case["problem"]
    if p == "poisson2d":
        return (N, N), [((0, 0), 4.0), ((-1, 0), -1.0), ((1, 0), -1.0), ((0, -1), -1.0), ((0, 1), -1.0)]
    if p == "poisson3d":
        t = [((0, 0, 0), 6.0)]
        for ax in range(3):
            for d in (-1, 1):
                t.append((tuple(d if k == ax else 0 for k in range(3)), -1.0))
        return (N, N, N), t
    if p == "aniso2d":
        return (N, N), [((dy, dx), v) for (dx, dy), v in inputs.q1_rotated_stencil(1e-3, math.pi / 8).items()]
    # lognormal coefficients, harmonic-mean faces, half a cell to the boundary
    g = np.random.default_rng([int(seed), 40])
    k = torch.from_numpy(np.exp(g.standard_normal((N, N, N)))).to(DEV)
    diag = torch.zeros_like(k)
    t = []
    for ax in range(3):
        lo, hi = k.narrow(ax, 0, N - 1), k.narrow(ax, 1, N - 1)
        w = 2.0 * lo * hi / (lo + hi)
        for d in (-1, 1):
            face = 2.0 * k
            face.narrow(ax, 1 if d < 0 else 0, N - 1).copy_(w)
            diag = diag + face
            t.append((tuple(d if a == ax else 0 for a in range(3)), -face))
    return (N, N, N), [((0, 0, 0), diag)] + t


def _inside(shape, off, dev):
    m = torch.ones(shape, dtype=torch.bool, device=dev)
    for ax, d in enumerate(off):
        if d:
            m.narrow(ax, 0 if d < 0 else shape[ax] - 1, 1).fill_(False)
    return m


def _csr(shape, terms):
    """CSR arrays (int32, int32, float64) of the stencil, columns ascending."""
    n = math.prod(shape)
    strides = [math.prod(shape[a + 1:]) for a in range(len(shape))]
    terms = sorted(((sum(o * s for o, s in zip(off, strides)), off, v) for off, v in terms), key=lambda q: q[0])
    row = torch.arange(n, device=DEV)
    mask = torch.stack([_inside(shape, off, DEV).reshape(-1) for _, off, _ in terms], dim=1)
    col = torch.stack([row + lin for lin, _, _ in terms], dim=1)[mask].to(torch.int32)
    val = torch.stack([torch.full((n,), v, dtype=torch.float64, device=DEV) if isinstance(v, float) else v.reshape(-1)
                       for _, _, v in terms], dim=1)[mask]
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(mask.sum(dim=1), 0, out=rp[1:])
    return n, rp.to(torch.int32), col, val.contiguous()


def _matrix(case, seed):
    if case["problem"] == "graph":
        A = inputs.random_graph_laplacian(case["N"])
        return A.n, torch.from_numpy(A.row_ptr), torch.from_numpy(A.col), torch.from_numpy(A.val)
    return _csr(*_terms(case, seed))


def _rows(case):
    return case["N"] if case["problem"] == "graph" else case["N"] ** (2 if case["problem"].endswith("2d") else 3)


def _rhs(case, seed):
    """Right-hand sides, one a row of the result (uniform in [-1, 1))."""
    k = case["requests"] or case["nrhs"]
    return np.random.default_rng([int(seed), 1]).uniform(-1.0, 1.0, (k, _rows(case)))


def _hierarchy(case, A):
    n, rp, ci, v = A
    if n <= HOST_SETUP_ROWS:
        h = amg.Hierarchy(inputs.CSR(n, rp.cpu().numpy(), ci.cpu().numpy(), v.cpu().numpy()))
    else:
        h = amg.Hierarchy(A, setup="device", coarsening="rs")
    if case["lumping"] != "diagonal":
        h.set_lumping(case["lumping"])
    if case["relax"] != "jacobi":
        h.set_relaxation(case["relax"], case["block_rows"])
    if case["gamma"] > 0:
        h.sparsify(case["gamma"], 2)
    return h


# ---- one pass ------------------------------------------------------------------

def prepare(case, seed):
    s = {"case": case}
    A = _matrix(case, seed)
    n = A[0]
    b = _rhs(case, seed)
    if case["call"] == "setup":
        s["A"] = A
    elif case["call"] == "serve":
        csr = inputs.CSR(n, A[1].cpu().numpy(), A[2].cpu().numpy(), A[3].cpu().numpy())
        s["server"] = serve.SolveServer({"p": csr}, 32 << 30, precision=case["precision"], tol=case["tol"],
                                        gamma=case["gamma"])
        s["b"] = [torch.from_numpy(r).to(DEV) for r in b]
        s["x"] = [torch.empty(n, dtype=torch.float64, device=DEV) for _ in b]
        return s
    else:
        s["h"] = _hierarchy(case, A)
    if case["call"] == "block":
        s["b"] = torch.from_numpy(np.ascontiguousarray(b.T)).to(DEV)
    else:
        s["b"] = torch.from_numpy(b[0]).to(DEV)
    if case["call"] == "vcycle":
        s["b"] = s["b"].to(torch.float32 if case["precision"] == 32 else torch.float64)
    s["x"] = torch.empty_like(s["b"])
    if case["guess"] == "warm":
        # the solution of a step before: smooth, and not that of this right-hand side
        g = np.random.default_rng([int(seed), 2]).uniform(0.5, 1.5)
        s["guess"] = g * torch.sin(torch.linspace(0.0, 3.0, n, dtype=torch.float64, device=DEV))
    return s


def _solve(case, h, b, x):
    return h.solve(b, x, method=amg.PCG, tol=case["tol"], maxit=200, adaptive=case["adaptive"], k=3, s=1,
                   precision=case["precision"], zero_guess=case["guess"] == "zero")


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "serve":
        reqs = [serve.Request(rid=i, key="p", b=b, arrival=0.0, x=x) for i, (b, x) in enumerate(zip(s["b"], s["x"]))]
        s["server"].run(reqs)
        return {"x": s["x"], "iters": [r.iters for r in reqs]}
    b, x = s["b"], s["x"]
    if call == "setup":
        with amg.Hierarchy(s["A"], setup="device", coarsening="pmis", seed=1) as h:
            if case["gamma"] > 0:
                h.sparsify(case["gamma"], 2)
            r = _solve(case, h, b, x)
        return {"x": x, "iters": r.iters}
    h = s["h"]
    if call == "vcycle":
        x.zero_()
        (h.vcycle32 if case["precision"] == 32 else h.vcycle)(b, x)
        return {"x": x}
    if call == "block":
        x.zero_()
        r = h.solve_block(b, x, method=amg.PCG, tol=case["tol"], maxit=200, precision=case["precision"])
        return {"x": x, "iters": r.col_iters}
    if call == "step":
        h.sparsify(case["gamma"], 2)
    if case["guess"] == "warm":
        x.copy_(s["guess"])
    r = _solve(case, h, b, x)
    return {"x": x, "iters": r.iters}


# ---- what a pass cannot do without -----------------------------------------------

# entries per row of the matrix, entries of all levels over those of the matrix
# (Ruge-Stueben), entries of P over rows of all levels, typical iterations to 1e-8
_SHAPE = {"poisson2d": (5, 2.2, 2.6, 8), "poisson3d": (7, 2.9, 4.0, 9), "aniso2d": (9, 2.0, 2.5, 34),
          "fv3d": (7, 3.0, 4.0, 20), "graph": (13, 3.0, 4.0, 9)}


def work(case):
    """One read of every operator of the hierarchy (values and 32-bit columns), of
    P and R, and the fine vectors r, z, p, q, x once each, per iteration."""
    n = _rows(case)
    k = case["requests"] or case["nrhs"]
    per_row, cx, pr, it = _SHAPE[case["problem"]]
    it = it * (1.25 if case["tol"] < 1e-8 else 1.0)
    if case["call"] == "vcycle":
        it = 1
    if case["relax"] != "jacobi":
        it = 1.5 * it
    if case["call"] == "setup":
        it = 3 * it
    v = 4 if case["precision"] == 32 else 8
    entries = n * (per_row * cx + 2 * pr)
    per_it = entries * (v + 4) + n * 8 * 8 * k
    if case["call"] == "serve":
        it = it * math.ceil(k / 16)
        per_it = entries * (v + 4) + n * 8 * 8 * min(k, 16)
    bytes_ = it * per_it
    if case["call"] == "step":
        bytes_ += 13 * n * per_row * (cx - 1)
    if case["call"] == "setup":
        bytes_ += 12 * n * per_row * (1 + cx) + 24 * n * pr
    return {"bytes": float(bytes_), "flops": float(it * k * (2 * entries * 2 + 10 * n))}


# ---- exact values -------------------------------------------------------------------

def _sine(N):
    j = np.arange(1, N + 1)
    return math.sqrt(2.0 / (N + 1)) * np.sin(math.pi * np.outer(j, j) / (N + 1)), 2.0 - 2.0 * np.cos(
        math.pi * j / (N + 1))


def _poisson_exact(case, b):
    """Sine transforms along every axis diagonalise the Dirichlet Laplacian."""
    N, d = case["N"], 2 if case["problem"] == "poisson2d" else 3
    S, lam = _sine(N)
    S, u = torch.from_numpy(S).to(DEV), torch.from_numpy(b).to(DEV).reshape((N,) * d)
    lam = torch.from_numpy(lam).to(DEV)

    def each_axis(u):
        for ax in range(d):
            u = torch.movedim(torch.matmul(S, torch.movedim(u, ax, 0).reshape(N, -1)).reshape((N,) * d), 0, ax)
        return u

    den = sum(lam.reshape([N if a == ax else 1 for a in range(d)]) for ax in range(d))
    return each_axis(each_axis(u) / den).reshape(-1)


def _cg_exact(case, seed, b):
    """Conjugate gradients on the stencil in float64, far below the tolerance of any case."""
    shape, terms = _terms(case, seed)
    inner = []
    diag = None
    for off, v in terms:
        if not any(off):
            diag = v
            continue
        dst = tuple(slice(max(0, -d), s - max(0, d)) for d, s in zip(off, shape))
        src = tuple(slice(max(0, d), s - max(0, -d)) for d, s in zip(off, shape))
        inner.append((dst, src, v if isinstance(v, float) else v[dst]))

    def apply(u):
        y = diag * u
        for dst, src, v in inner:
            y[dst] += v * u[src]
        return y

    r = torch.from_numpy(b).to(DEV).reshape(shape).clone()
    x, z = torch.zeros_like(r), r / diag
    p, rz, stop = z.clone(), (r * z).sum(), 1e-14 * float(r.norm())
    for it in range(20000):
        q = apply(p)
        a = rz / (p * q).sum()
        x += a * p
        r -= a * q
        if it % 50 == 49 and float(r.norm()) <= stop:
            break
        z = r / diag
        new = (r * z).sum()
        p = z + (new / rz) * p
        rz = new
    return x.reshape(-1)


def exact(case, seed):
    """The solutions A^-1 b; nothing for iteration counts and for the cycle alone."""
    if case["call"] == "vcycle":
        return None
    b = _rhs(case, seed)
    if case["problem"] in ("poisson2d", "poisson3d"):
        x = [_poisson_exact(case, r) for r in b]
    elif case["problem"] == "graph":
        A = inputs.random_graph_laplacian(case["N"])
        x = [torch.from_numpy(c) for c in np.linalg.solve(A.to_dense(), b.T).T]
    else:
        x = [_cg_exact(case, seed, r) for r in b]
    if case["call"] == "serve":
        return {"x": x, "iters": None}
    if case["call"] == "block":
        return {"x": torch.stack(x, dim=1), "iters": None}
    return {"x": x[0], "iters": None}
