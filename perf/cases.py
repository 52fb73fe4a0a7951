"""Performance cases: what a user of the panel solver has it do, from one
section to a whole population.

A case describes a batch layout (how many sections, their panel counts and
angles of attack), the formulation, the precision and what is asked of the
solver:

* ``solve``       surface speed, Cp and lift of the batch (``PanelSolver.solve``)
* ``grad``        the same forward plus the shape gradient (``panel_cl_cp``
                  and its backward pass)
* ``generation``  one generation of the genetic algorithm
                  (``GeneticOptimizer.generation``)

The batches are NACA 4-digit sections drawn from the case's seed (camber
m ~ U[0, 0.06], its position p ~ U[0.2, 0.6], thickness t ~ U[0.08, 0.18],
cosine spacing, closed trailing edge), the population of B-spline contours
for the generations.  ``exact`` evaluates the same quantities in plain torch
FP64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1511_02166_amd as panel

DEG = math.pi / 180.0
VINF = 1.0


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _case(name, kind, B, n_lo, n_hi, n_step=1, k_lo=1, k_hi=1, precision="fp64", formulation="stream", cp=False):
    c = dict(kind=kind, B=B, n_lo=n_lo, n_hi=n_hi, n_step=n_step, k_lo=k_lo, k_hi=k_hi, precision=precision,
             formulation=formulation, cp=cp)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one section's polar, as an interactive tool or a test asks for it:
        # nothing to batch, so launches and the pivot chain are what counts
        _case("section polar", "solve", 1, 160, 160, k_lo=9, k_hi=9),
        # a handful of sections at a common resolution (naca128)
        _case("naca128", "solve", 32, 128, 128),
        # the genetic algorithm's population, one angle each (ga2048), in both
        # precisions
        _case("ga2048 fp64", "solve", 2048, 256, 256),
        _case("ga2048 refine", "solve", 2048, 256, 256, precision="refine"),
        # the same population in the source + vortex formulation
        _case("ga2048 hess-smith", "solve", 2048, 256, 256, formulation="hess_smith"),
        # one generation of the paper's population size (4000 individuals of
        # about 200 points): contours, solve, boundary layer, selection
        _case("generation 4000x200", "generation", 4000, 200, 200),
        # a parameter study over panel counts and four angles per section
        # (uneven4096)
        _case("uneven4096 refine", "solve", 4096, 96, 512, n_step=16, k_lo=4, k_hi=4, precision="refine"),
        # sections from several sources: any panel count, odd ones among them,
        # and a different number of angles each
        _case("ragged 1000 fp64", "solve", 1000, 65, 450, k_lo=1, k_hi=6),
        # gradient-based shape optimisation of a population (adjoint1024)
        _case("adjoint1024", "grad", 1024, 256, 256),
        # finely panelled sections over a polar (large256): mixed precision,
        # and FP64 with the shape gradient
        _case("large256 refine", "solve", 256, 1024, 1024, k_lo=8, k_hi=8, precision="refine"),
        _case("large256 gradient", "grad", 256, 1024, 1024, k_lo=8, k_hi=8),
        # inverse design of a small set on a target pressure distribution:
        # cotangents of Cp at two angles, source + vortex, mixed precision
        _case("pressure matching", "grad", 96, 180, 180, k_lo=2, k_hi=2, precision="refine",
              formulation="hess_smith", cp=True),
    ]


def _cost(c):
    n = 0.5 * (c["n_lo"] + c["n_hi"]) + 1
    return c["B"] * (n ** 3 / 1.5 + 600.0 * n * n * (2.5 if c["kind"] == "grad" else 1.0) * (c["k_hi"] if c["cp"] else 1))


def draw(rng):
    """One more batch: 1 to 4096 sections, 32 to 1024 panels, 1 to 12 angles."""
    while True:
        kind = rng.choice(["solve", "solve", "solve", "grad", "grad", "generation"])
        B = int(round(math.exp(rng.uniform(math.log(1), math.log(4096)))))
        n = int(round(math.exp(rng.uniform(math.log(32), math.log(1024)))))
        if kind == "generation":
            c = _case(None, kind, max(2, 2 * (B // 2)), n - n % 2, n - n % 2)
        else:
            lo = n if rng.random() < 0.5 else max(24, int(n * rng.uniform(0.2, 0.9)))
            k_hi = rng.choice([1, 1, 2, 3, 4, 8, 12])
            k_lo = k_hi if rng.random() < 0.5 else rng.randint(1, k_hi)
            cp = kind == "grad" and rng.random() < 0.4
            c = _case(None, kind, B, lo, n, 1, k_lo, k_hi, rng.choice(["fp64", "refine"]),
                      rng.choice(["stream", "stream", "hess_smith"]), cp)
        if _cost(c) <= 1.2e11:
            return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _layout(case):
    """Panel and angle counts: the case's own, the same for every seed (a
    program keeps its plan while the sections change)."""
    B = case["B"]
    rng = np.random.default_rng([B, case["n_lo"], case["n_hi"], case["k_hi"]])
    steps = (case["n_hi"] - case["n_lo"]) // case["n_step"]
    N = case["n_lo"] + case["n_step"] * rng.integers(0, steps + 1, B)
    K = rng.integers(case["k_lo"], case["k_hi"] + 1, B)
    node_off = np.concatenate([[0], np.cumsum(N + 1)]).astype(np.int32)
    alpha_off = np.concatenate([[0], np.cumsum(K)]).astype(np.int32)
    return N, K, node_off, alpha_off


def _sections(rng, N, node_off):
    """Nodes of seeded NACA 4-digit sections, [2 * nodes] interleaved."""
    B = len(N)
    m, p, t = rng.uniform(0.0, 0.06, B), rng.uniform(0.2, 0.6, B), rng.uniform(0.08, 0.18, B)
    b = np.repeat(np.arange(B), N + 1)
    k = np.arange(node_off[-1]) - node_off[b]
    n, m, p, t = N[b], m[b], p[b], t[b]
    k = np.where(k == n, 0, k)   # closed trailing edge: node N is node 0
    x = 0.5 * (1.0 + np.cos(2.0 * np.pi * k / n))
    yt = 5.0 * t * (0.2969 * np.sqrt(x) - 0.1260 * x - 0.3516 * x ** 2 + 0.2843 * x ** 3 - 0.1036 * x ** 4)
    fore = x < p
    q = np.where(fore, p, 1.0 - p) ** 2
    yc = m / q * np.where(fore, 2.0 * p * x - x ** 2, 1.0 - 2.0 * p + 2.0 * p * x - x ** 2)
    th = np.arctan(2.0 * m / q * (p - x))
    side = np.where(2 * k <= n, 1.0, -1.0)
    xy = np.stack([x - side * yt * np.sin(th), yc + side * yt * np.cos(th)], axis=1)
    return xy.reshape(-1)


def _angles(rng, K):
    """Per section an increasing polar within [-4, 12] degrees."""
    return np.concatenate([np.sort(rng.uniform(-4.0, 12.0, k)) for k in K]) * DEG


GA_SURFACE_POINTS = 6


def _ga_problem():
    """Control points (clamped cubic B-spline through the trailing edge), the
    coordinates the genes set and their bounds: six ordinates per surface."""
    m = GA_SURFACE_POINTS
    X = 0.5 * (1.0 + np.cos(np.pi * np.arange(1, m + 1) / m))
    X[-1] = 0.0
    T = np.zeros((2 * m + 2, 2))
    T[0] = T[-1] = (1.0, 0.0)
    T[1:m + 1, 0] = X
    T[m + 1:2 * m + 1, 0] = X[::-1]
    genes = 2 * np.arange(1, 2 * m + 1) + 1
    lo = np.concatenate([np.full(m, 0.01), np.full(m, -0.10)])
    hi = np.concatenate([np.full(m, 0.16), np.full(m, -0.01)])
    return T, genes, lo, hi


def _inputs(case, seed):
    """Everything drawn from the seed, on the host."""
    rng = np.random.default_rng([seed, case["B"], case["n_hi"]])
    if case["kind"] == "generation":
        T, genes, lo, hi = _ga_problem()
        genome = lo + (hi - lo) * rng.random((case["B"], len(genes)))
        return dict(T=T, genes=genes, lo=lo, hi=hi, genome=genome, rng=rng)
    N, K, node_off, alpha_off = _layout(case)
    d = dict(N=N, K=K, node_off=node_off, alpha_off=alpha_off, xy=_sections(rng, N, node_off),
             alpha=_angles(rng, K))
    if case["kind"] == "grad":
        d["dcl"] = rng.standard_normal(int(alpha_off[-1]))
        if case["cp"]:
            d["dcp"] = rng.standard_normal(int(np.sum(N * K))) / 100.0
    return d


def _gpu(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def prepare(case, seed):
    d = _inputs(case, seed)
    precision = panel.PANEL_FP64 if case["precision"] == "fp64" else panel.PANEL_FP32_REFINE
    if case["kind"] == "generation":
        opt = panel.GeneticOptimizer(case["B"], case["n_hi"], d["T"], d["genes"], d["lo"], d["hi"],
                                     precision=precision, max_gen=64)
        uniforms = _gpu(d["rng"].random(opt.u_gen.numel()))
        return dict(kind="generation", opt=opt, genome=_gpu(d["genome"]), uniforms=uniforms)
    formulation = panel.PANEL_STREAM_FUNCTION if case["formulation"] == "stream" else panel.PANEL_HESS_SMITH
    solver = panel.PanelSolver(d["node_off"], d["alpha_off"], precision, formulation=formulation)
    state = dict(kind=case["kind"], solver=solver, xy=_gpu(d["xy"]), alpha=_gpu(d["alpha"]))
    if case["kind"] == "grad":
        state["xy"].requires_grad_()
        state["dcl"] = _gpu(d["dcl"])
        state["dcp"] = _gpu(d["dcp"]) if case["cp"] else None
    return state


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    if state["kind"] == "generation":
        # the population handed in, evaluated and bred with the given draws
        opt = state["opt"]
        opt.genome.copy_(state["genome"])
        opt.generation(state["uniforms"])
        return dict(contours=opt.xy, cl=opt.solver.cl, gamma=opt.solver.gamma, cd=opt.cd, ld=opt.ld,
                    fitness=opt.fitness, genome=opt.genome, info=opt.solver.info)
    solver, xy, alpha = state["solver"], state["xy"], state["alpha"]
    if state["kind"] == "grad":
        cl, cp = panel.panel_cl_cp(xy, alpha, solver, vinf=VINF)
        if state["dcp"] is None:
            (dxy,) = torch.autograd.grad(cl, xy, state["dcl"])
        else:
            (dxy,) = torch.autograd.grad((cl, cp), xy, (state["dcl"], state["dcp"]))
        return dict(cl=cl.detach(), cp=cp.detach(), dxy=dxy, info=solver.info, adj_info=solver.adj_info)
    return solver.solve(xy, alpha, vinf=VINF)


def work(case):
    """Arithmetic: per influence entry about 60 operations (a logarithm, an
    arctangent, the closed form), LU and triangular solves, and for a
    gradient one transposed solve and about 100 operations per entry for each
    seed (every angle has its own with Cp cotangents).  Bytes: nodes and
    angles in; speeds, Cp, lift (or gradient, genomes) out."""
    B, step = case["B"], case["n_step"]
    N = np.arange(case["n_lo"], case["n_hi"] + 1, step).astype(float)
    n, K = N + 1, 0.5 * (case["k_lo"] + case["k_hi"])
    flops = 60.0 * N ** 2 + n ** 3 / 1.5 + 2.0 * n ** 2 * K
    nbytes = 16.0 * n + 8.0 * K * (2.0 * N + 3.0) + 4.0
    if case["kind"] == "grad":
        seeds = K if case["cp"] or case["formulation"] != "stream" else 1.0
        flops += seeds * (2.0 * n ** 2 + 100.0 * N ** 2)
        nbytes += 16.0 * n + (8.0 * K * N if case["cp"] else 0.0) - 8.0 * K * N
    if case["kind"] == "generation":
        nbytes = nbytes + 8.0 * 4 * 2 * GA_SURFACE_POINTS
    return {"bytes": float(B * nbytes.mean()), "flops": float(B * flops.mean())}


# ---------------------------------------------------------------------------
# The same quantities in plain torch FP64
# ---------------------------------------------------------------------------

def _system(P, formulation):
    """Influence blocks of [G, N + 1, 2] nodes: the bordered matrix without its
    right-hand sides and, for the source + vortex formulation, the tangential
    matrix too."""
    G, N = P.shape[0], P.shape[1] - 1
    eye = torch.eye(N, dtype=torch.bool, device=P.device)
    m = 0.5 * (P[:, :-1] + P[:, 1:])
    h = P[:, 1:] - P[:, :-1]
    L = h.square().sum(-1).sqrt()
    t = h / L[..., None]
    d1x, d1y = (m[:, :, None, i] - P[:, None, :-1, i] for i in (0, 1))
    d2x, d2y = (m[:, :, None, i] - P[:, None, 1:, i] for i in (0, 1))
    one = torch.ones((), dtype=P.dtype, device=P.device)
    # the diagonal is replaced below; keep its derivatives finite
    l1 = torch.where(eye, one, d1x ** 2 + d1y ** 2).log()
    l2 = torch.where(eye, one, d2x ** 2 + d2y ** 2).log()
    cr = torch.where(eye, 0 * one, d1x * d2y - d1y * d2x)
    ang = torch.atan2(cr, torch.where(eye, one, d1x * d2x + d1y * d2y))
    M = torch.zeros(G, N + 1, N + 1, dtype=P.dtype, device=P.device)
    if formulation == "stream":
        hx, hy, Lc = h[:, None, :, 0], h[:, None, :, 1], L[:, None, :]
        g = -((d1x * hx + d1y * hy) * l1 - (d2x * hx + d2y * hy) * l2 - 2 * Lc ** 2 + 2 * cr * ang) / (4 * math.pi * Lc)
        A = torch.where(eye, (Lc / (2 * math.pi) * (1 - (0.5 * Lc).log())).expand_as(g), g)
        last = torch.zeros(G, N + 1, dtype=P.dtype, device=P.device)
        last[:, 0] = last[:, N - 1] = 1
        top = torch.cat([A, -torch.ones(G, N, 1, dtype=P.dtype, device=P.device)], 2)
        return torch.cat([top, last[:, None]], 1), None, L, t, m
    beta = torch.where(eye, math.pi * one, -ang)
    lg = torch.where(eye, 0 * one, 0.5 * (l1 - l2))
    tjx, tjy, tix, tiy = t[:, :, None, 0], t[:, :, None, 1], t[:, None, :, 0], t[:, None, :, 1]
    c, s = tix * tjx + tiy * tjy, tix * tjy - tiy * tjx
    A, T = (lg * s + beta * c) / (2 * math.pi), (lg * c - beta * s) / (2 * math.pi)
    top = torch.cat([A, -T.sum(2, keepdim=True)], 2)
    T = torch.cat([T, A.sum(2, keepdim=True)], 2)
    return torch.cat([top, (T[:, 0] + T[:, N - 1])[:, None]], 1), T, L, t, m


def _flow(P, alpha, formulation):
    """Surface speed [G, K, N], Cp, Cl and Cl_p [G, K] of sections that share
    one panel count; alpha [G, K]."""
    M, T, L, t, m = _system(P, formulation)
    ca, sa = alpha.cos(), alpha.sin()
    if formulation == "stream":
        rhs = -VINF * (m[:, None, :, 1] * ca[..., None] - m[:, None, :, 0] * sa[..., None])
        rhs = torch.cat([rhs, torch.zeros_like(rhs[..., :1])], 2)
        u = torch.linalg.solve(M, rhs.transpose(1, 2)).transpose(1, 2)[..., :-1]
    else:
        along = VINF * (ca[..., None] * t[:, None, :, 0] + sa[..., None] * t[:, None, :, 1])
        normal = VINF * (ca[..., None] * t[:, None, :, 1] - sa[..., None] * t[:, None, :, 0])
        rhs = torch.cat([-normal, -(along[..., :1] + along[..., -1:])], 2)
        x = torch.linalg.solve(M, rhs.transpose(1, 2))
        u = (T @ x).transpose(1, 2) + along
    cp = 1 - (u / VINF) ** 2
    cl = -2 * (u * L[:, None]).sum(-1) / VINF
    lift = -t[:, None, :, 1] * sa[..., None] - t[:, None, :, 0] * ca[..., None]
    return u, cp, cl, -(cp * L[:, None] * lift).sum(-1)


def _groups(N, K):
    """Sections with the same panel and angle counts, at most 32 and about
    2^25 influence entries at a time."""
    by = {}
    for b, key in enumerate(zip(N.tolist(), K.tolist())):
        by.setdefault(key, []).append(b)
    for (n, k), idx in by.items():
        most = min(32, max(1, (1 << 25) // (n * n)))
        for i in range(0, len(idx), most):
            yield n, k, np.array(idx[i:i + most])


def _bspline(d, N):
    """Contours [B, N + 1, 2] of the genomes: clamped cubic B-spline on the
    control points, by de Boor's recursion."""
    deg, M = 3, len(d["T"])
    Q = np.repeat(d["T"].reshape(1, -1), len(d["genome"]), 0)
    Q[:, d["genes"]] = d["genome"]
    Q = Q.reshape(-1, M, 2)
    knots = np.concatenate([np.zeros(deg), np.linspace(0, 1, M - deg + 1), np.ones(deg)])
    k = np.arange(N // 2 + 1)
    u = (1 - np.cos(2 * np.pi * k / N)) / 4
    u = np.concatenate([u, 1 - u[:-1][::-1]])
    span = np.clip(np.searchsorted(knots, u, side="right") - 1, deg, M - 1)
    pts = [Q[:, span - deg + j] for j in range(deg + 1)]
    for r in range(1, deg + 1):
        for j in range(deg, r - 1, -1):
            lo, hi = knots[span - deg + j], knots[span + 1 + j - r]
            a = ((u - lo) / (hi - lo))[None, :, None]
            pts[j] = (1 - a) * pts[j - 1] + a * pts[j]
    out = pts[deg]
    out[:, -1] = out[:, 0]
    return out


def exact(case, seed):
    if case["kind"] == "generation" and case["B"] * case["n_hi"] ** 3 > 1e11:
        return None
    d = _inputs(case, seed)
    if case["kind"] == "generation":
        B, N = d["genome"].shape[0], case["n_hi"]
        xy = _bspline(d, N)
        d.update(N=np.full(B, N), K=np.ones(B, np.int64), node_off=np.arange(B + 1) * (N + 1),
                 alpha_off=np.arange(B + 1), xy=xy.reshape(-1), alpha=np.zeros(B))
    N, K, node_off, alpha_off = d["N"], d["K"], d["node_off"], d["alpha_off"]
    out_off = np.concatenate([[0], np.cumsum(N * K)])
    if len(set(zip(N.tolist(), K.tolist()))) > 2000:
        return None
    xy, alpha = _gpu(d["xy"]), _gpu(d["alpha"])
    grad = case["kind"] == "grad"
    cl, cl_p = torch.zeros_like(alpha), torch.zeros_like(alpha)
    u, cp = (torch.zeros(int(out_off[-1]), dtype=torch.float64, device="cuda") for _ in range(2))
    dxy = torch.zeros_like(xy)
    for n, k, idx in _groups(N, K):
        def at(off, count):
            return torch.as_tensor(off[idx][:, None] + np.arange(count), device="cuda")
        nodes, angles, field = at(2 * node_off.astype(np.int64), 2 * (n + 1)), at(alpha_off, k), at(out_off, n * k)
        P = xy[nodes].reshape(-1, n + 1, 2).requires_grad_(grad)
        with torch.set_grad_enabled(grad):
            gu, gcp, gcl, gclp = _flow(P, alpha[angles], case["formulation"])
            if grad:
                f = (gcl * _gpu(d["dcl"])[angles]).sum()
                if case["cp"]:
                    f = f + (gcp * _gpu(d["dcp"])[field].reshape(gcp.shape)).sum()
                f.backward()
                dxy[nodes] = P.grad.reshape(len(idx), -1)
        u[field], cp[field] = gu.detach().reshape(len(idx), -1), gcp.detach().reshape(len(idx), -1)
        cl[angles], cl_p[angles] = gcl.detach(), gclp.detach()
    if grad:
        return dict(cl=cl, cp=cp, dxy=dxy, info=None, adj_info=None)
    if case["kind"] == "generation":
        return dict(contours=xy, cl=cl, gamma=u, cd=None, ld=None, fitness=None, genome=None, info=None)
    return dict(gamma=u, cp=cp, cl=cl, cl_p=cl_p, info=None)
