"""Which kernels a batch is given: on both sides of the lines of the dispatch,
the default tiling runs the same kernel as the tiling that pins it, bit for bit
(order, systems per CU, precision; the times behind the lines are in lu.hip)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

WAVE, BLOCK = (320, 0, 4), (0, 0, 4)


def _solved(sizes, ks, precision, tiling):
    import torch

    import paper_1511_02166_amd as P
    nodes = {n: oracle.naca4(0.02, 0.4, 0.12, n) for n in set(sizes)}
    xy_flat, noff = synth.pack_nodes([nodes[n] for n in sizes])
    aoff = np.concatenate([[0], np.cumsum(ks)]).astype(np.int32)
    s = P.PanelSolver(noff, aoff, precision, tiling=tiling)
    s.solve(torch.as_tensor(xy_flat, device="cuda"),
            torch.as_tensor(np.linspace(-0.05, 0.15, aoff[-1]), device="cuda"))
    torch.cuda.synchronize()
    assert bool((s.info == 0).all())
    return s


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("precision,n,per_cu,tiling", [
    (0, 96, 1.0, BLOCK), (0, 94, 1.0, WAVE), (0, 110, 1.75, WAVE), (0, 112, 2.0, BLOCK), (0, 256, 2.0, BLOCK),
    (0, 256, 2.1, WAVE), (1, 62, 1.0, WAVE), (1, 64, 2.0, BLOCK), (1, 64, 2.5, WAVE), (1, 128, 2.0, BLOCK),
    (1, 128, 3.0, WAVE), (1, 318, 2.1, WAVE)])
def test_factorisation_of_equal_systems(precision, n, per_cu, tiling):
    sizes = [n] * int(per_cu * _cus())
    a, b = (_solved(sizes, [1] * len(sizes), precision, t) for t in (None, tiling))
    which = "a64" if precision == 0 else "a32"
    for q in (0, len(sizes) // 2, len(sizes) - 1):
        assert np.array_equal(a.system(q, which)[0], b.system(q, which)[0]), q
        assert np.array_equal(a.pivots(q), b.pivots(q))


# (smallest and largest panel count, systems per CU): their number weighted by
# (order / largest order)^2 is about 0.38 of it for 24 to 318, 0.53 for 64 to 128
@pytest.mark.parametrize("precision,lo,hi,per_cu,tiling", [
    (0, 24, 318, 5.0, BLOCK), (0, 24, 318, 8.0, WAVE), (0, 64, 128, 2.2, BLOCK), (0, 64, 128, 4.0, WAVE),
    (1, 24, 318, 6.0, BLOCK), (1, 24, 318, 8.0, WAVE), (1, 64, 128, 2.5, BLOCK), (1, 64, 128, 4.0, WAVE)])
def test_factorisation_of_spread_systems(precision, lo, hi, per_cu, tiling):
    sizes = np.linspace(lo // 2, hi // 2, int(per_cu * _cus())).astype(int) * 2
    a, b = (_solved(list(sizes), [1] * len(sizes), precision, t) for t in (None, tiling))
    which = "a64" if precision == 0 else "a32"
    for q in (0, len(sizes) // 3, len(sizes) - 1):
        assert np.array_equal(a.system(q, which)[0], b.system(q, which)[0]), q
