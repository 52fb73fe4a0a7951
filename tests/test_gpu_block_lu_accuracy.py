"""How close the workgroup LU's solutions of panel systems come to the exact ones
(of the matrix and right-hand side the GPU assembled, from residuals in long
double), against plain elimination in the same precision: one rank-1 update
after the other, so that every product is subtracted from the entry it updates.
A blocked update that sums its products first and then subtracts the sum rounds
at the size of the entries before the update and is an order of magnitude
further off on these matrices."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _plain_elimination(M, rhs, ft):
    """x of M x = rhs by Gaussian elimination with partial pivoting in type ft."""
    A = np.concatenate([M, rhs[:, None]], axis=1).astype(ft)
    n = len(M)
    for k in range(n - 1):
        p = k + int(np.argmax(np.abs(A[k:, k])))
        if p != k:
            A[[k, p]] = A[[p, k]]
        l = A[k + 1:, k] / A[k, k]
        A[k + 1:, k + 1:] -= l[:, None] * A[k, k + 1:]
    x = A[:, n]
    for k in range(n - 1, -1, -1):
        x[k] /= A[k, k]
        x[:k] -= A[:k, k] * x[k]
    return x


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,waves", [(160, 4), (160, 8), (256, 4), (400, 4), (400, 8), (640, 4), (640, 8), (1024, 8)])
def test_solutions_as_accurate_as_plain_elimination(N, waves, precision):
    import torch

    import paper_1511_02166_amd as P
    B = 6
    rng = np.random.default_rng(N)
    xy_flat, noff = synth.pack_nodes([oracle.naca4(*rng.uniform([0.0, 0.2, 0.08], [0.06, 0.6, 0.18]), N) for _ in range(B)])
    s = P.PanelSolver(noff, np.arange(B + 1, dtype=np.int32), precision, tiling=(0, 0, waves))
    s.assemble(torch.as_tensor(xy_flat, device="cuda"), torch.as_tensor(rng.uniform(-0.05, 0.2, B), device="cuda"))
    torch.cuda.synchronize()
    systems = [s.system(b) for b in range(B)]
    s.factor_solve(max_iter=0)   # (FP32: the solution before its refinement)
    torch.cuda.synchronize()
    ours, plain = [], []
    for b, (M, R) in enumerate(systems):
        n, d = N + 1, s.plan.layout(b)
        x = np.linalg.solve(M, R[0]).astype(np.longdouble)
        for _ in range(2):
            x = x + np.linalg.solve(M, (R[0].astype(np.longdouble) - M.astype(np.longdouble) @ x).astype(np.float64))
        got = s.ws[d["x"]:d["x"] + 8 * n].cpu().numpy().view(np.float64)
        ref = _plain_elimination(M, R[0], np.float64 if precision == 0 else np.float32)
        ours.append(float(np.max(np.abs(got - x)) / np.max(np.abs(x))))
        plain.append(float(np.max(np.abs(ref - x)) / np.max(np.abs(x))))
    # geometric means over six sections: an error varies by about a factor of 2
    # from section to section, each mean by 2 ** (1 / sqrt(6)) = 1.33, their ratio
    # by 1.5; 4 is more than three of those
    ours, plain = (np.exp(np.mean(np.log(e))) for e in (ours, plain))
    print(f"N={N} waves={waves} precision={precision}: {ours:.2e} against {plain:.2e}")
    assert ours < 4.0 * plain, (ours, plain)
