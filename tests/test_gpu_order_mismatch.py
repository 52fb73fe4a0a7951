"""A workspace whose airfoil order does not match its plan: a system sent to a
kernel that cannot hold it is reported (info -3) and its outputs are NaN, in
every kernel mapping and both precisions, and its neighbours are solved."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("persistent,wg_waves", [(0, 0), (0, 4), (1, 4)])
@pytest.mark.parametrize("few", [True, False], ids=["few", "many"])
def test_system_beyond_its_group_is_refused(precision, persistent, wg_waves, few):
    # Wave limit 256: orders 321 (one angle) and 320 (16 angles) both belong
    # to the workgroup kernels, the second first (it costs more).  With the
    # limit at 320 only the larger one does, so on the older workspace the
    # place of the only large system holds the order 320, and 321 stands first
    # among the small systems.  `many` adds enough small systems that they are
    # refined by a wavefront each.
    import torch

    import paper_1511_02166_amd as P
    from paper_1511_02166_amd import _binding as C
    N, K = [320, 319] + [24] * (4 if few else 600), [1, 16] + [1] * (4 if few else 600)
    B = len(N)
    one, noff1 = synth.joukowski_batch(3, 3, [320, 319, 24])
    pieces = [one[2 * noff1[i]:2 * noff1[i + 1]] for i in range(3)]
    xy = torch.as_tensor(np.concatenate([pieces[min(i, 2)] for i in range(B)]), device="cuda")
    noff = np.concatenate([[0], np.cumsum(np.asarray(N) + 1)]).astype(np.int32)
    aoff = np.concatenate([[0], np.cumsum(K)]).astype(np.int32)
    alpha = torch.full((int(aoff[-1]),), 0.06, dtype=torch.float64, device="cuda")
    s = P.PanelSolver(noff, aoff, precision, tiling=(256, persistent, wg_waves))
    C.panel_plan_set_tiling(s.plan, 320, persistent, wg_waves)
    other = torch.empty(s.plan.workspace_size() + 256, dtype=torch.uint8, device="cuda")
    C.panel_workspace_init(s.plan, other[(-other.data_ptr()) % 256:])   # the plan counts as initialised again
    out = s.solve(xy, alpha)                                            # on the older workspace
    torch.cuda.synchronize()
    info = s.info.cpu().numpy()
    assert info[0] == -3 and np.all(info[1:] == 0), info
    cl, gamma = out["cl"].cpu().numpy(), out["gamma"].cpu().numpy()
    assert np.isnan(cl[0]) and np.all(np.isnan(gamma[:320]))
    assert np.all(np.isfinite(cl[1:])) and np.all(np.isfinite(gamma[320:]))
    ref = P.PanelSolver(noff, aoff, precision)
    cl_ref = ref.solve(xy, alpha)["cl"].cpu().numpy()
    assert np.max(np.abs(cl[1:] - cl_ref[1:])) < 1e-8   # cusped sections: their FP64 floor is near 1e-9
    dxy = s.adjoint(xy, torch.ones(int(aoff[-1]), dtype=torch.float64, device="cuda")).cpu().numpy()
    assert np.all(np.isnan(dxy[:2 * 321])) and np.all(np.isfinite(dxy[2 * 321:]))
    assert s.adj_info.cpu().numpy()[0] == -3
