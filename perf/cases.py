"""Performance cases: the work that programs built on this library have it do.

A program that uses the library creates an operator (or a batch of them) once
and then applies the Hamiltonian and the kinetic preconditioner to block after
block of vectors, orthogonalises blocks, or hands the whole problem to the
eigensolver.  Every case below is one such piece of work:

* ``step``  one Hamiltonian apply and one preconditioner apply of a block, the
  two operator calls of an inner (GMRES) iteration, 1D or 2D, in FP64, FP32 or
  BF16x3, optionally with the per-column eigenvalue shifts of the correction
  equation.
* ``batch`` the same for many independent 1D operators in grouped calls.
* ``orth``  the FP64 block orthogonalisation of a new block against a basis.
* ``solve`` one whole eigensolve.

Sizes and parameters follow ``workloads`` (c1 .. c5, c5r), the tests and the
paper's mapped parity grids; ``draw`` spreads them over the ranges between.
The mode operators of a discretisation do not depend on the blocks, so an
operator is created once per problem and kept, as a program keeps it.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2111_02534_amd as t3

PREC = {"fp64": (t3.FP64, torch.float64), "fp32": (t3.FP32, torch.float32),
        "bf16x3": (t3.BF16X3, torch.float32)}
SIGMA = -0.75   # preconditioner shift: a binding energy of the size the workloads have
ALPHA = 20.0    # heavy-to-light mass ratio of the workloads
SHIFTS = (-1.3, -0.9, -0.6, -0.4, -0.25, -0.1, 0.05, 0.2)


def listed():
    return [
        # the smallest grid (c1): a few vectors, launches and latency only
        dict(name="step_1d_tiny_fp64", kind="step", ndim=1, nx=32, ny=32, nvec=4, prec="fp64",
             shifted=False, grid="cgl"),
        # an ordinary grid (c2) inside the FP64 solver: shifted applies of a block of 8
        dict(name="step_1d_mid_fp64", kind="step", ndim=1, nx=256, ny=256, nvec=8, prec="fp64",
             shifted=True, grid="cgl"),
        # the paper's grid at its 256 x 128 size: mapped nodes, bosonic parity half grids
        dict(name="step_1d_paper_grid_fp64", kind="step", ndim=1, nx=256, ny=128, nvec=4,
             prec="fp64", shifted=False, grid="mapped"),
        # odd, ragged mode sizes and an odd number of vectors, low-precision inner solves
        dict(name="step_1d_ragged_fp32", kind="step", ndim=1, nx=333, ny=190, nvec=5, prec="fp32",
             shifted=True, grid="cgl"),
        # the finest 1D grid (c3), FP64 and the two low-precision forms of its inner solves
        dict(name="step_1d_large_fp64", kind="step", ndim=1, nx=1024, ny=1024, nvec=16,
             prec="fp64", shifted=False, grid="cgl"),
        dict(name="step_1d_large_fp32", kind="step", ndim=1, nx=1024, ny=1024, nvec=16,
             prec="fp32", shifted=True, grid="cgl"),
        dict(name="step_1d_large_bf16x3", kind="step", ndim=1, nx=1024, ny=1024, nvec=16,
             prec="bf16x3", shifted=True, grid="cgl"),
        # the reduced 2D problem (c5r, n = 20 per mode) with low-precision inner solves
        dict(name="step_2d_small_fp32", kind="step", ndim=2, nx=20, ny=20, nvec=8, prec="fp32",
             shifted=True, grid="cgl"),
        # the largest 2D problem of one GPU (c5, 16.8 M unknowns per vector)
        dict(name="step_2d_large_fp64", kind="step", ndim=2, nx=64, ny=64, nvec=8, prec="fp64",
             shifted=True, grid="cgl"),
        # a batch of instances of mixed sizes (c4), every step one grouped call
        dict(name="batch_fp64", kind="batch", count=64, nmin=64, nmax=256, nvec=4, prec="fp64"),
        # the solver's basis expansion on long vectors
        dict(name="orth_long", kind="orth", N=1 << 22, nq=40, nx=8, factors=False),
        # a whole eigensolve of the ordinary grid (c2), FP32 inner iterations
        dict(name="solve_1d_mid", kind="solve", nx=256, ny=256, nev=10, block=8, prec="fp32",
             gmres_steps=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    prec = rng.choice(["fp64", "fp32", "bf16x3"])
    if u < 0.45:
        # the paper's grid is used in FP64
        grid = "mapped" if rng.random() < 0.2 else "cgl"
        return dict(kind="step", ndim=1, nx=_log(rng, 16, 1024), ny=_log(rng, 16, 1024),
                    nvec=rng.randint(1, 16), prec="fp64" if grid == "mapped" else prec,
                    shifted=rng.random() < 0.5, grid=grid)
    if u < 0.7:
        return dict(kind="step", ndim=2, nx=_log(rng, 6, 64), ny=_log(rng, 6, 64),
                    nvec=rng.randint(1, 8), prec=prec, shifted=rng.random() < 0.5, grid="cgl")
    if u < 0.8:
        return dict(kind="batch", count=rng.randint(8, 64), nmin=rng.randint(20, 64),
                    nmax=rng.randint(65, 256), nvec=rng.randint(1, 4), prec=prec)
    if u < 0.9:
        return dict(kind="orth", N=_log(rng, 1 << 12, 1 << 22), nq=rng.randint(0, 64),
                    nx=rng.randint(1, 16), factors=rng.random() < 0.3)
    n = rng.randint(32, 200)
    return dict(kind="solve", nx=n, ny=rng.randint(max(32, n // 2), n), nev=rng.randint(2, 8),
                block=rng.randint(4, 8), prec=prec, gmres_steps=rng.choice([3, 5, 10]))


# ------------------------------------------------------------------ operators
_ops = {}


def _problem(case):
    """Arguments of t3.Operator for a case of kind step or solve."""
    cx, cy, mu = t3.jacobi_coefficients(ALPHA)
    if case["kind"] == "solve":
        return dict(ndim=1, n=[case["nx"], case["ny"]], L=15.0, c_x=cx, c_y=cy, v0=2.0, mu_hl=mu)
    nm = case["ndim"]
    n = [case["nx"]] * nm + [case["ny"]] * nm
    if case["grid"] == "mapped":
        cx, cy, mu = t3.paper_coefficients(ALPHA)
        return dict(ndim=1, n=n, L=[8.0, 4.0], c_x=cx, c_y=cy, pot="gauss_paper", v0=0.34459535,
                    mu_hl=mu, sigma=-0.1, grid="mapped", parity=[1, 1])
    return dict(ndim=nm, n=n, L=15.0, c_x=cx, c_y=cy, v0=3.0, mu_hl=mu, sigma=SIGMA)


def _instances(case):
    """Operator arguments of a batch: sizes spread over nmin .. nmax, parameters as c4's."""
    out = []
    for i in range(case["count"]):
        rng = np.random.Generator(np.random.PCG64(2111 + i))
        n = case["nmin"] + int(rng.integers(0, 4)) * (case["nmax"] - case["nmin"]) // 3
        alpha = float(math.exp(rng.uniform(0.0, math.log(100.0))))
        cx, cy, mu = t3.jacobi_coefficients(alpha)
        out.append(dict(ndim=1, n=[n, n], L=15.0, c_x=cx, c_y=cy, v0=float(rng.uniform(0.5, 5.0)),
                        width=float(rng.uniform(0.5, 2.0)), mu_hl=mu, sigma=SIGMA))
    return out


def _operator(args):
    key = repr(sorted(args.items()))
    if key not in _ops:
        while len(_ops) > 200:
            _ops.pop(next(iter(_ops))).close()
        _ops[key] = t3.Operator(**args)
    return _ops[key]


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64).to(dtype)


def _shifts(nvec):
    return torch.tensor([SHIFTS[v % len(SHIFTS)] for v in range(nvec)], dtype=torch.float64,
                        device="cuda")


def _packed(blocks):
    """One zeroed buffer and, in it, a block of the shape of each of `blocks`, every block
    at a multiple of 64 elements: a batch's results kept together."""
    at, end = [], 0
    for b in blocks:
        at.append(end)
        end += -(-b.numel() // 64) * 64
    flat = torch.zeros(end, dtype=blocks[0].dtype, device=blocks[0].device)
    return flat, [flat[o:o + b.numel()].reshape(b.shape) for o, b in zip(at, blocks)]


# ------------------------------------------------------------------ state, run
def _inputs(case, seed):
    """The input blocks of a case (device), from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * seed + 17)
    kind = case["kind"]
    if kind == "step":
        _, dt = PREC[case["prec"]]
        N = (case["nx"] * case["ny"]) ** case["ndim"]
        return _normal(g, (case["nvec"], N), dt), _normal(g, (case["nvec"], N), dt)
    if kind == "batch":
        _, dt = PREC[case["prec"]]
        sizes = [a["n"][0] * a["n"][1] for a in _instances(case)]
        return ([_normal(g, (case["nvec"], N), dt) for N in sizes],
                [_normal(g, (case["nvec"], N), dt) for N in sizes])
    if kind == "orth":
        N, nq, nx = case["N"], case["nq"], case["nx"]
        Q = _normal(g, (nq, N), torch.float64)
        for _ in range(2):
            if nq:  # orthonormal rows by Cholesky, twice
                Q = (torch.linalg.inv(torch.linalg.cholesky(Q @ Q.T)) @ Q).contiguous()
        X = _normal(g, (nx, N), torch.float64)
        if nq:  # an expansion block: mostly new directions, part of it in the basis
            X += _normal(g, (nx, nq), torch.float64) * math.sqrt(N / nq) @ Q
        return Q, X
    return int(seed)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "step":
        st["op"] = _operator(_problem(case))
        st["X"], st["B"] = _inputs(case, seed)
        st["Y"], st["Z"] = torch.empty_like(st["X"]), torch.empty_like(st["B"])
        st["shifts"] = _shifts(case["nvec"]) if case["shifted"] else None
    elif kind == "batch":
        st["ops"] = [_operator(a) for a in _instances(case)]
        st["X"], st["B"] = _inputs(case, seed)
        st["HX"], st["Y"] = _packed(st["X"])
        st["PB"], st["Z"] = _packed(st["B"])
    elif kind == "orth":
        st["Q"], st["X0"] = _inputs(case, seed)
        st["X"] = torch.empty_like(st["X0"])
    else:
        st["op"] = _operator(_problem(case))
        st["seed"] = int(seed)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        p = PREC[case["prec"]][0]
        state["op"].apply_H(state["X"], state["Y"], prec=p, shifts=state["shifts"])
        state["op"].apply_prec(state["B"], state["Z"], prec=p)
        return {"HX": state["Y"], "PB": state["Z"]}
    if kind == "batch":
        p = PREC[case["prec"]][0]
        t3.apply_H_batched(state["ops"], state["X"], state["Y"], prec=p)
        t3.apply_prec_batched(state["ops"], state["B"], state["Z"], prec=p)
        return {"HX": state["HX"], "PB": state["PB"]}
    if kind == "orth":
        # the new block arrives in a buffer of its own and is orthonormalised in the basis
        state["X"].copy_(state["X0"])
        Q = state["Q"] if case["nq"] else None
        C, R, rank = t3.block_orth(Q, state["X"], want_factors=case["factors"])
        return {"X": state["X"], "C": C, "R": R, "rank": rank}
    r = state["op"].jdqr(case["nev"], case["block"], inner_prec=PREC[case["prec"]][0],
                         gmres_steps=case["gmres_steps"], seed=state["seed"], want_Q=False)
    return r.evals


# ------------------------------------------------------------------ work
def _step_work(ndim, nx, ny, nvec, es):
    N = (nx * ny) ** ndim
    per = 2.0 * N * ndim * (nx + ny)          # one dense product per mode
    return dict(bytes=4.0 * nvec * N * es, flops=nvec * (3.0 * per + 4.0 * N))


def work(case):
    kind = case["kind"]
    if kind == "step":
        return _step_work(case["ndim"], case["nx"], case["ny"], case["nvec"],
                          8 if case["prec"] == "fp64" else 4)
    if kind == "batch":
        es = 8 if case["prec"] == "fp64" else 4
        ws = [_step_work(1, a["n"][0], a["n"][1], case["nvec"], es) for a in _instances(case)]
        return dict(bytes=sum(w["bytes"] for w in ws), flops=sum(w["flops"] for w in ws))
    if kind == "orth":
        N, nq, nx = case["N"], case["nq"], case["nx"]
        return dict(bytes=8.0 * N * (nq + 2 * nx), flops=N * (8.0 * nq * nx + 4.0 * nx * nx))
    # a solve: at the least one apply of H and of the preconditioner per wanted pair and
    # GMRES step (what it takes beyond that is the method's iteration)
    return _step_work(1, case["nx"], case["ny"], case["nev"] * case["gmres_steps"], 8)


# ------------------------------------------------------------------ 64-bit values
def _cgl(n, L):
    """Interior Gauss-Lobatto nodes (ascending) and the second-derivative matrix."""
    K = n + 1
    j = np.arange(K + 1)
    t = np.sin(np.pi * (K - 2 * j) / (2 * K))
    c = np.where(j % 2, -1.0, 1.0)
    c[0] *= 0.5
    c[K] *= 0.5
    dt = t[:, None] - t[None, :] + np.eye(K + 1)
    D = (c[None, :] / c[:, None]) / dt
    D -= np.diag(np.diag(D))
    D -= np.diag(D.sum(axis=1))
    D2 = (D @ D)[1:-1, 1:-1] / (L * L)
    return -L * t[1:-1], 0.5 * (D2 + D2[::-1, ::-1])


def _mapped_even(n, L):
    """Positive nodes of the 2n-point mapped grid and the operator on even functions."""
    N = 2 * n
    j = np.arange(N)[::-1]
    a = np.pi * (2 * j + 1) / (2.0 * N)
    t, w = np.cos(a), np.where(j % 2, -1.0, 1.0) * np.sin(a)
    dt = t[:, None] - t[None, :] + np.eye(N)
    D = (w[None, :] / w[:, None]) / dt
    D -= np.diag(np.diag(D))
    D -= np.diag(D.sum(axis=1))
    s = 1.0 - t * t
    tp, tpp = s * np.sqrt(s) / L, -3.0 * t * s * s / (L * L)
    D2 = (tp * tp)[:, None] * (D @ D) + tpp[:, None] * D
    x = L * t / np.sqrt(s)
    return x[n:], D2[n:, n:] + D2[n:, :n][:, ::-1]


def _modes64(args):
    """(nodes, kinetic matrix) of every mode, in 64 bits."""
    nm = 2 * args["ndim"]
    Ls = args["L"] if isinstance(args["L"], list) else [args["L"]] * nm
    out = []
    for k in range(nm):
        f = _mapped_even if args.get("grid") == "mapped" else _cgl
        x, D2 = f(args["n"][k], Ls[k])
        out.append((x, -(args["c_x"] if k < nm // 2 else args["c_y"]) * D2))
    return out


def _potential64(args, modes):
    w = 1.0 if args.get("pot") == "gauss_paper" else 2.0 * args.get("width", 1.0) ** 2
    X = [m[0] for m in modes]
    if args["ndim"] == 1:
        x, y = X[0][:, None], X[1][None, :]
        r2 = ((y - x / 2) ** 2, (y + x / 2) ** 2)
    else:
        x1, x2 = X[0][:, None, None, None], X[1][None, :, None, None]
        y1, y2 = X[2][None, None, :, None], X[3][None, None, None, :]
        r2 = ((y1 - x1 / 2) ** 2 + (y2 - x2 / 2) ** 2, (y1 + x1 / 2) ** 2 + (y2 + x2 / 2) ** 2)
    return -args["v0"] * (np.exp(-r2[0] / w) + np.exp(-r2[1] / w))


def _along(A, W, k):
    """The matrix A applied along mode k of the tensor W (leading axis: vectors)."""
    sh = W.shape
    W = W.movedim(k + 1, 0)
    rest = W.shape[1:]
    out = (A @ W.reshape(sh[k + 1], -1)).reshape((A.shape[0],) + rest)
    return out.movedim(0, k + 1).contiguous()


def _step64(args, X, B, shifts):
    modes = _modes64(args)
    nm = len(modes)
    dev = [torch.from_numpy(np.ascontiguousarray(m[1])).cuda() for m in modes]
    shape = (X.shape[0],) + tuple(args["n"])
    W = X.double().reshape(shape)
    V = torch.from_numpy(np.ascontiguousarray(_potential64(args, modes))).cuda()
    Y = W * V
    if shifts is not None:
        Y = Y - W * shifts.reshape((-1,) + (1,) * nm)
    for k in range(nm):
        Y += _along(dev[k], W, k)
    del W, V
    # the kinetic sum minus sigma, inverted in the modes' eigenbases, with one step of
    # iterative refinement
    eig = []
    for _, K in modes:
        lam, S = np.linalg.eig(K)
        S = np.ascontiguousarray(S.real)
        eig.append((torch.from_numpy(np.ascontiguousarray(lam.real)).cuda(), torch.from_numpy(S).cuda(),
                    torch.from_numpy(np.linalg.inv(S)).cuda()))

    def solve(R):
        for k in range(nm):
            R = _along(eig[k][2], R, k)
        den = -args["sigma"]
        for k in range(nm):
            sh = [1] * (nm + 1)
            sh[k + 1] = -1
            den = den + eig[k][0].reshape(sh)
        R = R / den
        for k in range(nm):
            R = _along(eig[k][1], R, k)
        return R

    B = B.double().reshape(shape)
    Z = solve(B)
    R = B + args["sigma"] * Z
    for k in range(nm):
        R -= _along(dev[k], Z, k)
    Z += solve(R)
    return Y.reshape(X.shape), Z.reshape(X.shape)


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        if case["nx"] * case["ny"] > 1600:
            return None  # a dense eigensolve of this size takes too long
        args = _problem(case)
        (x, Kx), (y, Ky) = modes = _modes64(args)
        H = np.kron(Kx, np.eye(len(y))) + np.kron(np.eye(len(x)), Ky)
        H += np.diag(_potential64(args, modes).ravel())
        return np.sort(np.linalg.eigvals(H).real)[: case["nev"]]
    if kind == "step":
        X, B = _inputs(case, seed)
        sh = _shifts(case["nvec"]) if case["shifted"] else None
        Y, Z = _step64(_problem(case), X, B, sh)
        return {"HX": Y, "PB": Z}
    if kind == "batch":
        Xs, Bs = _inputs(case, seed)
        pairs = [_step64(a, X, B, None) for a, X, B in zip(_instances(case), Xs, Bs)]
        out = {}
        for name, k in (("HX", 0), ("PB", 1)):
            out[name], views = _packed([p[k] for p in pairs])
            for v, p in zip(views, pairs):
                v.copy_(p[k])
        return out
    Q, X = _inputs(case, seed)
    X0 = X.clone()
    for _ in range(2):
        if case["nq"]:
            X = X - (X @ Q.T) @ Q
    for _ in range(2):
        X = torch.linalg.inv(torch.linalg.cholesky(X @ X.T)) @ X
    C = R = None
    if case["factors"]:
        C = (Q @ X0.T) if case["nq"] else None
        R = X @ X0.T
        R = torch.triu(R)
    return {"X": X, "C": C, "R": R, "rank": None}
