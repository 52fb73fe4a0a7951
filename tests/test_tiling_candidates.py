"""The tiling search offers every kernel mapping of a batch, once."""
import numpy as np
import pytest

import paper_1511_02166_amd as P


def _candidates(n_panels):
    s = P.PanelSolver.__new__(P.PanelSolver)   # the search reads the plan only
    s.plan = P.Plan(np.concatenate([[0], np.cumsum(np.asarray(n_panels) + 1)]), np.arange(len(n_panels) + 1), 0)
    return s.tiling_candidates()


@pytest.mark.parametrize("n_panels", [[128] * 8, [24, 319, 200], [500, 128, 64], [1024, 96], [400] * 3])
def test_one_wavefront_kernels_are_offered(n_panels):
    c = _candidates(n_panels)
    assert len(c) == len(set(c))
    # wg_waves 0 lets the library factor small systems by workgroups: the
    # one-wavefront kernels need a candidate that pins them
    if min(n_panels) < 320:
        assert any(wl > min(n_panels) and pers == 0 and wg in (4, 8) for wl, pers, wg in c), c
    # and the library's own choice and the workgroup kernels are there too
    assert (320, 0, 0) in c and any(wl <= min(n_panels) and pers == 0 for wl, pers, wg in c), c


def test_persistent_launch_is_offered_once_without_large_systems():
    assert [c for c in _candidates([128] * 8) if c[0] == 320] == [(320, 1, 0), (320, 0, 0), (320, 0, 4)]
