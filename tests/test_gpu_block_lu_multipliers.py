"""The multipliers of the workgroup LU are quotients: correctly rounded up to
the last step's own rounding, also for pivots whose reciprocal is subnormal or
overflows."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
SIZES = (31, 128, 300, 520)


def _factored(precision, waves, exponent, seed):
    """Gaussian systems times 2^exponent, and their factors by the workgroup LU."""
    import torch

    import paper_1511_02166_amd as P
    rng = np.random.default_rng(seed)
    xy, noff = synth.joukowski_batch(5, len(SIZES), list(SIZES))
    aoff = np.arange(len(SIZES) + 1, dtype=np.int32)
    s = P.PanelSolver(noff, aoff, precision, tiling=(0, 0, waves))
    s.assemble(torch.as_tensor(xy, device="cuda"), torch.full((len(SIZES),), 0.05, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()
    ft = np.float64 if precision == 0 else np.float32
    mats = []
    for b, N in enumerate(SIZES):
        n, d = N + 1, s.plan.layout(b)
        A = np.ldexp(rng.standard_normal((n, n)).astype(ft), exponent).astype(ft)
        full = np.zeros((n + 1, d["ld"]), dtype=ft)
        full[:n, :n] = A.T
        off, view = (d["a64"], 8) if precision == 0 else (d["a32"], 4)
        s.ws[off:off + view * full.size].copy_(torch.as_tensor(full.reshape(-1)).view(torch.uint8))
        mats.append(A)
    s.factor_solve(max_iter=0)
    torch.cuda.synchronize()
    which = "a64" if precision == 0 else "a32"
    return [(A, s.system(b, which)[0], s.pivots(b)) for b, A in enumerate(mats)]


def _permuted(A, piv):
    PA = A.copy()
    for i, p in enumerate(piv):
        PA[[i, p]] = PA[[p, i]]
    return PA


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("precision", [0, 1])
def test_first_column_is_rounded_once(precision, waves):
    # nothing but the division has touched the first column; 0.505 ulp: half
    # an ulp, 2^-11 of one for the long double quotient, the estimate's square
    for A, LU, piv in _factored(precision, waves, 0, 3):
        wide = np.longdouble if precision == 0 else np.float64
        col = _permuted(A, piv)[:, 0]
        exact = col[1:].astype(wide) / wide(col[0])
        err = np.abs(LU[1:, 0].astype(wide) - exact) / np.spacing(np.abs(LU[1:, 0])).astype(wide)
        assert np.max(err) <= 0.505, float(np.max(err))


# pivots near 2^-1028 and 2^1014 (2^-130 and 2^118): the reciprocal of the
# first overflows, that of the second is subnormal
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("precision,exponent", [(0, -1030), (0, 1014), (1, -132), (1, 117)])
def test_pivots_at_the_ends_of_the_range(precision, exponent, waves):
    eps, tiny = (2.0 ** -53, -1074) if precision == 0 else (2.0 ** -24, -149)
    for A, LU, piv in _factored(precision, waves, exponent, 4):
        n = A.shape[0]
        LU, PA = LU.astype(np.float64), _permuted(A, piv).astype(np.float64)
        L, U = np.tril(LU, -1) + np.eye(n), np.ldexp(np.triu(LU), -exponent)
        PA = np.ldexp(PA, -exponent)
        assert np.max(np.abs(np.tril(LU, -1))) <= 1.0 + 4 * eps
        # n eps times the growth factor (below 100 here), and the spacing of
        # subnormal entries in the place of eps where it is larger
        bound = 100 * n * max(eps * np.max(np.abs(PA)), 2.0 ** (tiny - exponent))
        assert np.max(np.abs(PA - L @ U)) <= bound, n
