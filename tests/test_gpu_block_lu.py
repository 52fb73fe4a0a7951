"""The workgroup LU (one airfoil per workgroup) on dense systems at the edges
of its tiles: panels of 16, bands of 64, the row slots of 256 and 512 threads,
1 to 16 right-hand sides, with pivoting at nearly every step, ties of equal
magnitude and an exactly zero column."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# orders n1 = N + 1 around the multiples of 16, 64, 256 and 512
SIZES = (4, 15, 16, 31, 62, 63, 64, 79, 127, 128, 191, 255, 256, 300, 511, 512, 700, 767)
ANGLES = (1, 2, 5, 16)


def _systems(precision, waves, sizes, rng, kind):
    import torch

    import paper_1511_02166_amd as P
    K = [ANGLES[i % len(ANGLES)] for i in range(len(sizes))]
    xy, noff = synth.joukowski_batch(5, len(sizes), list(sizes))
    aoff = np.concatenate([[0], np.cumsum(K)]).astype(np.int32)
    s = P.PanelSolver(noff, aoff, precision, tiling=(0, 0, waves))
    s.assemble(torch.as_tensor(xy, device="cuda"), torch.as_tensor(np.full(aoff[-1], 0.05), device="cuda"))
    torch.cuda.synchronize()
    mats = []
    for b, N in enumerate(sizes):
        n, d = N + 1, s.plan.layout(b)
        if kind == "ties":   # entries -1, 0, 1: many candidates of equal magnitude
            A = rng.integers(-1, 2, (n, n)).astype(np.float64) + 0.0
        else:
            A = rng.standard_normal((n, n))
        if kind == "zero":
            A[:, n // 2] = 0.0
        A = A.astype(np.float32).astype(np.float64)   # the same matrix in both precisions
        R = rng.standard_normal((d["K"], n)).astype(np.float32).astype(np.float64)
        full = np.zeros((n + d["K"], d["ld"]))
        full[:n, :n] = A.T
        full[n:, :n] = R
        s.ws[d["a64"]:d["a64"] + 8 * full.size].copy_(torch.as_tensor(full.reshape(-1)).view(torch.uint8))
        if precision == 1:
            s.ws[d["a32"]:d["a32"] + 4 * full.size].copy_(
                torch.as_tensor(full.reshape(-1).astype(np.float32)).view(torch.uint8))
        mats.append((A, R))
    s.factor_solve(max_iter=30)
    torch.cuda.synchronize()
    return s, mats


def _factors(s, b, precision):
    LU, Y = s.system(b, "a64" if precision == 0 else "a32")
    return LU.astype(np.float64), Y.astype(np.float64)


@pytest.mark.parametrize("kind", ["gauss", "ties"])
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("precision", [0, 1])
def test_factors_and_solutions(precision, waves, kind):
    sizes = SIZES + ((1024,) if waves == 8 else ())
    s, mats = _systems(precision, waves, sizes, np.random.default_rng(5), kind)
    info = s.info.cpu().numpy()
    # the factors of a backward stable elimination: n eps times the growth
    # factor, which stays below 100 for these matrices
    eps = 2.0 ** -53 if precision == 0 else 2.0 ** -24
    for b, N in enumerate(sizes):
        n, (A, R) = N + 1, mats[b]
        LU, Y = _factors(s, b, precision)
        if info[b] > 0:   # small +-1 matrices can be singular
            assert kind == "ties" and np.linalg.matrix_rank(A) < n, (N, info[b])
            continue
        piv = s.pivots(b)
        PA, PR = A.copy(), R.T.copy()
        for i in range(n):
            p = piv[i]
            assert i <= p < n
            PA[[i, p]] = PA[[p, i]]
            PR[[i, p]] = PR[[p, i]]
        L, U = np.tril(LU, -1) + np.eye(n), np.triu(LU)
        assert np.max(np.abs(LU[np.tril_indices(n, -1)]), initial=0.0) <= 1.0 + 4 * eps
        assert np.max(np.abs(PA - L @ U)) <= 100 * n * eps * np.max(np.abs(A)), N
        scale = 100 * n * eps * max(1.0, np.max(np.abs(Y)))
        assert np.max(np.abs(L @ Y.T - PR)) <= scale, N
        d = s.plan.layout(b)
        x = s.ws[d["x"]:d["x"] + 8 * n * d["K"]].cpu().numpy().view(np.float64).reshape(d["K"], n).T
        if precision == 0:
            # backward error of the two triangular solves
            res = np.max(np.abs(A @ x - R.T))
            assert res <= 100 * n * eps * np.max(np.abs(A)) * np.max(np.sum(np.abs(x), axis=0)), (N, res)


@pytest.mark.parametrize("waves", [4, 8])
def test_first_pivot_is_the_lowest_of_equal_magnitude(waves):
    s, mats = _systems(0, waves, SIZES, np.random.default_rng(9), "ties")
    for b, N in enumerate(SIZES):
        col = np.abs(mats[b][0][:, 0])
        if col.max() > 0:
            assert s.pivots(b)[0] == int(np.argmax(col)), N


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("waves", [4, 8])
def test_zero_column_is_reported(precision, waves):
    import torch
    s, mats = _systems(precision, waves, SIZES, np.random.default_rng(7), "zero")
    info = s.info.cpu().numpy()
    for b, N in enumerate(SIZES):
        n = N + 1
        assert info[b] == n // 2 + 1, (N, info[b])
        d = s.plan.layout(b)
        x = s.ws[d["x"]:d["x"] + 8 * n * d["K"]].view(torch.float64)
        assert bool(torch.isnan(x).all())


@pytest.mark.parametrize("tiling", [(0, 0, 0), (0, 0, 4), (0, 0, 8), (320, 0, 0), (320, 0, 4)])
@pytest.mark.parametrize("precision", [0, 1])
def test_uneven_right_hand_sides(precision, tiling):
    """1 to 16 angles per airfoil through the factorisation (with a tiling left
    to the library, small systems by workgroups too) and, in mixed precision,
    through the FP64 refinement of FP32 factors: groups of four and eight right-hand sides, rows left over from the tiles
    of 32, orders on both sides of the wave limit.  The refined solution solves
    the FP64 system to the refinement's stop rule (a correction below 1e-10 of
    the solution), so it agrees with a direct FP64 solve to 1e-9."""
    import torch

    import paper_1511_02166_amd as P
    N = [31, 32, 64, 95, 128, 159, 160, 200, 255, 256, 300, 319, 320, 330, 512, 540, 700, 767]
    K = [1 + (5 * i) % 16 for i in range(len(N))]
    K[1:4] = [2, 8, 9]
    xy, noff = synth.joukowski_batch(11, len(N), N)
    aoff = np.concatenate([[0], np.cumsum(K)]).astype(np.int32)
    alpha = torch.as_tensor(np.linspace(-0.05, 0.2, aoff[-1]), device="cuda")
    s = P.PanelSolver(noff, aoff, precision, tiling=tiling)
    s.assemble(torch.as_tensor(xy, device="cuda"), alpha)
    torch.cuda.synchronize()
    systems = [s.system(b) for b in range(len(N))]
    s.factor_solve()
    torch.cuda.synchronize()
    assert np.all(s.info.cpu().numpy() == 0)
    if precision == 1:
        assert np.all(s.refine_iterations() >= 1)
    for b, n in enumerate(np.asarray(N) + 1):
        d = s.plan.layout(b)
        x = s.ws[d["x"]:d["x"] + 8 * n * d["K"]].cpu().numpy().view(np.float64).reshape(d["K"], n)
        M, R = systems[b]
        ref = np.linalg.solve(M, R.T).T
        err = np.max(np.abs(x - ref)) / np.max(np.abs(ref))
        floor = 64 * 2.0 ** -53 * np.linalg.cond(M, np.inf)
        assert err <= max(1e-9, floor), (n - 1, d["K"], err, floor)
