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



# K angles: the line moves with them (orders of one size, or from lo to hi)
@pytest.mark.parametrize("precision,lo,hi,per_cu,K,tiling", [
    (1, 318, 318, 2.5, 4, BLOCK), (1, 318, 318, 2.5, 2, WAVE), (1, 318, 318, 3.1, 4, WAVE), (1, 192, 192, 2.1, 4, BLOCK),
    (1, 128, 128, 2.5, 8, BLOCK), (1, 128, 128, 2.5, 4, WAVE), (1, 64, 64, 2.1, 8, BLOCK), (1, 64, 64, 2.1, 4, WAVE),
    (1, 24, 104, 4.0, 5, BLOCK), (1, 24, 104, 4.0, 1, WAVE), (0, 24, 104, 3.2, 4, BLOCK), (0, 24, 104, 3.2, 1, WAVE)])
def test_factorisation_with_several_angles(precision, lo, hi, per_cu, K, tiling):
    sizes = np.linspace(lo // 2, hi // 2, int(per_cu * _cus())).astype(int) * 2
    a, b = (_solved(list(sizes), [K] * len(sizes), precision, t) for t in (None, tiling))
    which = "a64" if precision == 0 else "a32"
    for q in (0, len(sizes) // 3, len(sizes) - 1):
        assert np.array_equal(a.system(q, which)[0], b.system(q, which)[0]), q


# K angles; `wave`: refined by a wavefront each, so the solutions are those of
# the tiling that pins it.  The others differ from it in the last bits only.
@pytest.mark.parametrize("n,per_cu,K,wave", [
    (24, 0.25, 1, False), (48, 1.0, 1, False), (32, 2.0, 1, True), (64, 2.0, 1, False),
    (128, 2.5, 1, True), (24, 4.0, 2, False), (64, 8.0, 2, True),
    (86, 6.0, 2, True), (96, 8.0, 2, False), (24, 5.0, 3, True), (48, 5.0, 3, False), (24, 5.0, 4, False)])
def test_refinement(n, per_cu, K, wave):
    B = int(per_cu * _cus())
    # the same factors on both sides: the LU by wavefronts, which the second
    # tiling pins, or by workgroups for small batches
    a, b = (_solved([n] * B, [K] * B, 1, t) for t in (None, WAVE))
    assert a.refine_iterations().max() <= 4
    if np.array_equal(a.system(0, "a32")[0], b.system(0, "a32")[0]):
        assert bool((a.gamma == b.gamma).all()) == wave
    else:
        assert n + 1 > 64 and per_cu <= 2.5   # (the order is n + 1)
    assert float((a.gamma - b.gamma).abs().max()) < 1e-9 * float(b.gamma.abs().max())


def test_refinement_of_mixed_angles():
    # one to four angles each: both kernels take a share, every airfoil is
    # refined once
    sizes = [24, 32, 48, 64, 86, 88, 96, 128] * (5 * _cus() // 8)
    ks = [1 + q // 8 % 4 for q in range(len(sizes))]
    a, b = (_solved(sizes, ks, 1, t) for t in (None, WAVE))
    assert a.refine_iterations().min() >= 1 and a.refine_iterations().max() <= 4
    assert float((a.gamma - b.gamma).abs().max()) < 1e-9 * float(b.gamma.abs().max())


# orders of a range, two angles: one kernel refines the whole batch, so either
# every solution or none is that of the tiling which pins the wavefronts
@pytest.mark.parametrize("lo,hi,wave", [(24, 96, True), (24, 128, False)])
def test_refinement_of_spread_systems(lo, hi, wave):
    sizes = list(np.linspace(lo // 2, hi // 2, 8 * _cus()).astype(int) * 2)
    a, b = (_solved(sizes, [2] * len(sizes), 1, t) for t in (None, WAVE))
    for q in (0, len(sizes) // 2, len(sizes) - 1):
        assert np.array_equal(a.system(q, "a32")[0], b.system(q, "a32")[0]), q
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    assert a.gamma.numel() == off[-1]
    same = [bool((a.gamma[i:j] == b.gamma[i:j]).all()) for i, j in zip(off[:-1], off[1:])]
    assert all(same) if wave else not all(same[:len(same) // 2])
    assert float((a.gamma - b.gamma).abs().max()) < 1e-9 * float(b.gamma.abs().max())
