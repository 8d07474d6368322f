"""Adaptive steps with their finalisations riding on every y-z strategy's first
launch: mode sums and stage-derivative sums of sixteen modes, gathered by
workgroups of one to eight wavefronts.  The step size is held at its largest,
so that the strategies differ by rounding alone."""
import numpy as np
import pytest

from paper_2603_03706_amd import mmcav
from tests.helpers import gpu_for
from tests.test_gpu_yz_short import DT, M_TOL, STEPS, _inst

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,paths", [((8, 12, 4), ("short", "fused", "split", "splitx")),
                                        ((6, 20, 8), ("short", "reg", "fused", "split", "splitx")),
                                        ((5, 40, 1), ("short", "fused", "split")),
                                        ((6, 20, 16), ("halves", "xch", "reg8", "reg", "fused", "split", "splitx"))])
def test_adaptive_finalisation_on_every_path(grid, paths):
    out = {}
    for p in paths:
        print("adaptive finalisation", grid, p, flush=True)
        c = gpu_for(_inst(grid, "dp45", modes=16))
        c.set_stepper(mmcav.DP45, DT, 1e-18, DT)
        c.set_sampling(DT / 2, 100)
        b = mmcav.Batch([c])
        b.set_fft_path(p)
        b.step(STEPS, 1e-3)
        st = c.stats()
        assert (st["accepted"], st["rejected"]) == (STEPS, 0) and abs(st["t"] - STEPS * DT) <= 1e-9 * DT
        out[p] = (c.get_m(), c.get_a(), c.get_trace(100))
    m, a, (t, ta, tm) = out[paths[0]]
    assert len(t) == 2 * STEPS + 1
    for p in paths[1:]:
        assert np.abs(out[p][0] - m).max() <= M_TOL
        # a gathers g T < 1e-3 of the difference of m^-
        assert np.abs(out[p][1] - a).max() <= 1e-3 * M_TOL
        assert np.abs(out[p][2][1] - ta).max() <= 1e-3 * M_TOL
        # m^- between step ends: the interpolant's weights of both ends and of their derivatives (|dm/dt| DT < 1e-2) sum to less than 1.1
        assert np.abs(out[p][2][2] - tm).max() <= 1.1 * M_TOL
