"""The one-wavefront adjoint.  It serves batches of more than six short sections
per CU, which the other adjoint tests are too small for: here there are enough,
up to the largest order it takes and on both sides of its 64-row blocks."""
import math

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
DEG = math.pi / 180.0


def _section(q, n):
    if n % 2 == 0:
        return oracle.naca4(0.01 + 0.005 * (q % 5), 0.3 + 0.04 * (q % 6), 0.09 + 0.01 * (q % 8), n)
    return synth.circle_nodes(n) * np.array([1.0, 0.2])   # an ellipse: any panel count


@pytest.mark.parametrize("with_cp", [False, True], ids=["cl", "cl+cp"])
@pytest.mark.parametrize("precision", [0, 1])
def test_large_batch_of_short_sections(precision, with_cp):
    import torch

    import paper_1511_02166_amd as P
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B = 6 * cus + 50
    edges = [4, 5, 62, 63, 64, 65, 78, 79] + ([126, 127, 128, 142, 143] if precision == 0 else [])
    most = max(edges)   # order 144 with FP64 factors, 80 with FP32
    rng = np.random.default_rng(13 + precision)
    sizes = edges + [int(2 * k) for k in rng.integers(3, most // 2 + 1, B - len(edges))]
    ks = [int(k) for k in rng.integers(1, 4, B)]
    xy_flat, noff = synth.pack_nodes([_section(q, n) for q, n in enumerate(sizes)])
    alphas = [rng.uniform(-4, 10, k) * DEG for k in ks]
    dcl = [rng.standard_normal(k) for k in ks]
    dcp = rng.standard_normal(int(np.dot(sizes, ks))) / 10.0 if with_cp else None
    aoff = np.concatenate([[0], np.cumsum(ks)]).astype(np.int32)
    chord = rng.uniform(0.5, 2.0, B)
    xy = torch.as_tensor(xy_flat, device="cuda")
    grads = []
    for wave_limit in (None, 0):   # a wavefront each, a workgroup each
        s = P.PanelSolver(noff, aoff, precision, wave_limit=wave_limit)
        s.step(xy, torch.as_tensor(np.concatenate(alphas), device="cuda"), torch.as_tensor(chord, device="cuda"), vinf=1.2)
        grads.append(s.adjoint(xy, torch.as_tensor(np.concatenate(dcl), device="cuda"),
                               None if dcp is None else torch.as_tensor(dcp, device="cuda")).cpu().numpy())
        assert np.all(s.info.cpu().numpy() == 0) and np.all(s.adj_info.cpu().numpy() == 0)
    so = np.concatenate([[0], np.cumsum(np.multiply(sizes, ks))])
    tol = 1e-9 if precision == 0 else 1e-8
    for b, n in enumerate(sizes):
        g, h = (a[2 * noff[b]:2 * noff[b + 1]].reshape(-1, 2) for a in grads)
        assert np.max(np.abs(g - h)) < tol * np.max(np.abs(h)), (b, n)
        if b >= len(edges) and b % 64:
            continue
        ref = 0.0
        for k in range(ks[b]):
            w = np.zeros(n) if dcp is None else dcp[so[b] + k * n:so[b] + (k + 1) * n]
            ref = ref + oracle.force_gradient(xy_flat[2 * noff[b]:2 * noff[b + 1]].reshape(-1, 2), alphas[b][k],
                                              dcl[b][k], w, 1.2, chord[b])
        e = np.max(np.abs(g - ref)) / np.max(np.abs(ref))
        assert e < tol, (b, n, ks[b], e)


@pytest.mark.parametrize("precision", [0, 1])
def test_bad_geometry_stays_with_its_section(precision):
    import torch

    import paper_1511_02166_amd as P
    B = 6 * torch.cuda.get_device_properties(0).multi_processor_count + 9
    xy_flat, noff = synth.pack_nodes([_section(q, 30) for q in range(B)])
    xy_flat[2 * (noff[7] + 4):2 * (noff[7] + 5)] = xy_flat[2 * (noff[7] + 3):2 * (noff[7] + 4)]   # a zero-length panel
    aoff = np.arange(B + 1, dtype=np.int32)
    s = P.PanelSolver(noff, aoff, precision)
    xy = torch.as_tensor(xy_flat, device="cuda")
    s.step(xy, torch.full((B,), 0.05, dtype=torch.float64, device="cuda"))
    g = s.adjoint(xy, torch.ones(B, dtype=torch.float64, device="cuda")).cpu().numpy()
    bad = np.zeros(len(g), bool)
    bad[2 * noff[7]:2 * noff[8]] = True
    assert np.all(np.isnan(g[bad])) and np.all(np.isfinite(g[~bad]))
    assert s.adj_info.cpu().numpy()[7] == -1 and np.sum(s.adj_info.cpu().numpy() != 0) == 1


@pytest.mark.parametrize("n", [24, 48])
def test_shortest_sections_with_fp32_factors_from_five_per_cu_on(n):
    # the same sections alone (five per CU) and in a batch that is large enough
    # for any order: the same kernel, so the same bits
    import torch

    import paper_1511_02166_amd as P
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sections = [_section(q, n) for q in range(6 * cus + 1)]
    grads = []
    for B in (5 * cus, 6 * cus + 1):
        xy_flat, noff = synth.pack_nodes(sections[:B])
        s = P.PanelSolver(noff, np.arange(B + 1, dtype=np.int32), P.PANEL_FP32_REFINE, tiling=(320, 0, 4))
        xy = torch.as_tensor(xy_flat, device="cuda")
        s.step(xy, torch.full((B,), 0.05, dtype=torch.float64, device="cuda"))
        grads.append(s.adjoint(xy, torch.ones(B, dtype=torch.float64, device="cuda")))
    assert torch.equal(grads[0], grads[1][:grads[0].numel()])
