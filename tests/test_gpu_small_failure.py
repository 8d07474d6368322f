"""Runs of small instances that fail after accepted steps: a drive pulse of a
hundredth of a step's length in the middle of step n + 1 drives either only the
cavity or only the magnetisation out of range there.  State, amplitudes, trace,
time and counters are those of n steps."""
import numpy as np
import pytest

from paper_2603_03706_amd import mmcav
from tests.helpers import gpu_for, variant
from tests.test_gpu_small_steps import DT, _inst

pytestmark = pytest.mark.gpu


# Cavity: the pulse puts 8e307 into the derivatives of both middle stages, so
# that every stage amplitude (h times that) is finite and only the weighted sum
# of the derivatives overflows; without coupling the state does not notice.
# State: a middle stage whose field of 1e25 T leaves the next stage input at
# 1e23, whose torque overflows in single precision while the double-precision
# cavity, which sees 1e23 in m^-, stays finite.
def _failing(grid, n, what, **kw):
    inst = _inst(grid, seed=n, **kw)
    modes = len(inst.omega)
    if what == "cavity":
        amp, g = 8e307, 0.0
    else:
        g = inst.g[0]
        amp = 1e25 / (2 * g / 1.76e11) / (0.5 * DT)
    drive = np.zeros(modes, complex)
    drive[-1] = amp
    return variant(inst, g=np.full(modes, g), drive_amp=drive, drive_t0=np.full(modes, (n + 0.5) * DT),
                   drive_sigma=np.full(modes, 0.01 * DT))


# (the last: a second launch of the whole-step kernel; per-stage kernels)
@pytest.mark.parametrize("grid,n,kw", [((8, 8, 1), 2, {}), ((8, 8, 1), 3, dict(modes=2)),
                                       ((27, 19, 1), 3, dict(modes=3, profiled=True)), ((16, 16, 8), 4, dict(S=2)),
                                       ((16, 8, 9), 3, {}), ((8, 8, 1), 1030, {}), ((683, 3, 1), 3, {})])
@pytest.mark.parametrize("what", ["cavity", "state"])
def test_failure_after_accepted_steps(grid, n, kw, what):
    print("failure", grid, n, kw, what, flush=True)
    inst = _failing(grid, n, what, **kw)
    c, ref = gpu_for(inst), gpu_for(inst)
    for x in (c, ref):
        x.set_sampling(DT, 2000)
    with pytest.raises(mmcav.MMError) as e:
        c.run((n + 100) * DT)
    assert e.value.status == mmcav.MM_ERR_NONFINITE
    b = mmcav.Batch([ref])
    b.step(n)
    assert c.stats()["accepted"] == ref.stats()["accepted"] == n
    assert c.stats()["t"] == ref.stats()["t"]
    assert np.array_equal(c.get_m(), ref.get_m()) and np.array_equal(c.get_a(), ref.get_a())
    got, want = c.get_trace(2000), ref.get_trace(2000)
    assert len(got[0]) == n + 1
    for x, y in zip(got, want):
        assert np.array_equal(x, y)
    assert np.isfinite(c.get_m()).all() and np.isfinite(c.get_a()).all()
