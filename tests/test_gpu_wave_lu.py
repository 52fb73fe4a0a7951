"""The one-wavefront LU and refinement, which the default tiling keeps for large
batches: pinned here (wg_waves 4) on few systems, at the edges of one to five
rows per lane, of 16-column panels and 64-column super-panels, with 1 to 16
right-hand sides, pivoting at nearly every step, ties of equal magnitude, an
exactly zero column, and in the persistent launch."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

SIZES = (4, 15, 16, 17, 31, 62, 63, 64, 65, 100, 127, 128, 129, 191, 192, 193, 255, 256, 257, 300, 318, 319)
ANGLES = (1, 2, 5, 16)
TILINGS = [(320, 0, 4), (320, 1, 0)]


def _systems(precision, tiling, rng, kind):
    import torch

    import paper_1511_02166_amd as P
    K = [ANGLES[i % len(ANGLES)] for i in range(len(SIZES))]
    xy, noff = synth.joukowski_batch(5, len(SIZES), list(SIZES))
    aoff = np.concatenate([[0], np.cumsum(K)]).astype(np.int32)
    s = P.PanelSolver(noff, aoff, precision, tiling=tiling)
    s.assemble(torch.as_tensor(xy, device="cuda"), torch.full((int(aoff[-1]),), 0.05, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    mats = []
    for b, N in enumerate(SIZES):
        n, d = N + 1, s.plan.layout(b)
        A = rng.integers(-1, 2, (n, n)) + 0.0 if kind == "ties" else rng.standard_normal((n, n))
        if kind == "zero":
            A[:, n // 2] = 0.0
        A = A.astype(np.float32).astype(np.float64)   # the same matrix in both precisions
        R = rng.standard_normal((d["K"], n)).astype(np.float32).astype(np.float64)
        full = np.zeros((n + d["K"], d["ld"]))
        full[:n, :n], full[n:, :n] = A.T, R
        s.ws[d["a64"]:d["a64"] + 8 * full.size].copy_(torch.as_tensor(full.reshape(-1)).view(torch.uint8))
        if precision == 1:
            s.ws[d["a32"]:d["a32"] + 4 * full.size].copy_(
                torch.as_tensor(full.reshape(-1).astype(np.float32)).view(torch.uint8))
        mats.append((A, R))
    s.factor_solve(max_iter=30)
    torch.cuda.synchronize()
    return s, mats


def _solution(s, b):
    d = s.plan.layout(b)
    return s.ws[d["x"]:d["x"] + 8 * d["n1"] * d["K"]].cpu().numpy().view(np.float64).reshape(d["K"], d["n1"]).T


@pytest.mark.parametrize("kind", ["gauss", "ties"])
@pytest.mark.parametrize("tiling", TILINGS)
@pytest.mark.parametrize("precision", [0, 1])
def test_factors_and_solutions(precision, tiling, kind):
    s, mats = _systems(precision, tiling, np.random.default_rng(5), kind)
    info = s.info.cpu().numpy()
    eps = 2.0 ** -53 if precision == 0 else 2.0 ** -24
    for b, N in enumerate(SIZES):
        n, (A, R) = N + 1, mats[b]
        LU, Y = (m.astype(np.float64) for m in s.system(b, "a64" if precision == 0 else "a32"))
        if info[b] > 0:   # small +-1 matrices can be singular
            assert kind == "ties" and np.linalg.matrix_rank(A) < n, (N, info[b])
            continue
        piv, PA, PR = s.pivots(b), A.copy(), R.T.copy()
        if kind == "ties":
            col = np.abs(A[:, 0])
            assert piv[0] == int(np.argmax(col))   # the lowest of equal magnitude
        for i, p in enumerate(piv):
            assert i <= p < n
            PA[[i, p]], PR[[i, p]] = PA[[p, i]], PR[[p, i]]
        L, U = np.tril(LU, -1) + np.eye(n), np.triu(LU)
        # a backward stable elimination: n eps times the growth factor, which
        # stays below 100 for these matrices
        assert np.max(np.abs(LU[np.tril_indices(n, -1)]), initial=0.0) <= 1.0 + 4 * eps
        assert np.max(np.abs(PA - L @ U)) <= 100 * n * eps * np.max(np.abs(A)), N
        assert np.max(np.abs(L @ Y.T - PR)) <= 100 * n * eps * max(1.0, np.max(np.abs(Y))), N
        x = _solution(s, b)
        if precision == 0:
            res = np.max(np.abs(A @ x - R.T))
            assert res <= 100 * n * eps * np.max(np.abs(A)) * np.max(np.sum(np.abs(x), axis=0)), (N, res)
        elif info[b] == 0:   # refined against the FP64 system to a correction below 1e-10
            ref = np.linalg.solve(A, R.T)
            bound = max(1e-9, 64 * 2.0 ** -53 * np.linalg.cond(A, np.inf))
            assert np.max(np.abs(x - ref)) <= bound * np.max(np.abs(ref)), N


@pytest.mark.parametrize("tiling", TILINGS)
@pytest.mark.parametrize("precision", [0, 1])
def test_zero_column_is_reported(precision, tiling):
    s, _ = _systems(precision, tiling, np.random.default_rng(7), "zero")
    info = s.info.cpu().numpy()
    for b, N in enumerate(SIZES):
        assert info[b] == (N + 1) // 2 + 1, (N, info[b])
        assert np.all(np.isnan(_solution(s, b)))


@pytest.mark.parametrize("precision", [0, 1])
def test_most_angles(precision):
    # 16 right-hand sides on panel systems up to the largest order, against the
    # oracle; refined one right-hand side after the other
    import torch

    import paper_1511_02166_amd as P
    sizes = [30, 64, 250, 300, 316, 318]
    rng = np.random.default_rng(17)
    nodes = [oracle.naca4(0.02, 0.4, 0.1 + 0.01 * i, n) for i, n in enumerate(sizes)]
    xy_flat, noff = synth.pack_nodes(nodes)
    aoff = (16 * np.arange(len(sizes) + 1)).astype(np.int32)
    alpha = rng.uniform(-0.07, 0.2, 16 * len(sizes))
    s = P.PanelSolver(noff, aoff, precision, tiling=(320, 0, 4))
    out = s.solve(torch.as_tensor(xy_flat, device="cuda"), torch.as_tensor(alpha, device="cuda"))
    ref = oracle.solve_batch(xy_flat, noff, alpha, aoff)
    assert bool((out["info"] == 0).all())
    for k in ("cl", "gamma", "cp"):
        e = np.max(np.abs(out[k].cpu().numpy() - ref[k])) / max(1.0, np.max(np.abs(ref[k])))
        assert e < (1e-10 if precision == 0 else 1e-8), (k, e)
