"""Sizes that the no-allocation run takes: instances near the end of its array,
with the y-z strategy that keeps most beside them, equal to mm_run bit for bit."""
import numpy as np
import pytest

from paper_2603_03706_amd import workloads as W
from tests.helpers import gpu_for

pytestmark = pytest.mark.gpu


# padded y-z of 128 x 64 from where the halved strategy outgrows the array up
# to where the exchange strategy does; grids it takes with halves; 256 rows in
# halves; separate x passes; split y-z passes
@pytest.mark.parametrize("grid", [(129, 64, 32), (160, 64, 32), (219, 64, 32), (128, 64, 32), (200, 40, 20),
                                  (30, 100, 20), (300, 40, 9), (4, 100, 40)])
@pytest.mark.parametrize("method", ["rk4", "dp45"])
def test_noalloc_equals_run(grid, method):
    inst = W.Instance(grid=grid, cell=(5e-9, 4e-9, 3e-9), Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.0, 0.25),
                      demag=W.DEMAG_FFT, omega=np.array([3e10]), kappa=np.array([1e7]), g=np.array([3e8]),
                      m0=W.tilted(grid, 10.0, 0.3), a0=np.array([0.05 + 0.02j]), method=method, dt0=0.2e-12)
    ref, got = gpu_for(inst), gpu_for(inst)
    # adaptive: the second run begins where the first has left the k-slot table
    # and the third where the second has
    for T in (0.2e-12, 0.5e-12, 0.2e-12):
        print("noalloc", grid, method, T, flush=True)
        ref.run(T, 1e-6)
        got.run_noalloc(T, 1e-6)
        assert ref.stats()["accepted"] == got.stats()["accepted"] > 0
        assert np.array_equal(ref.get_m(), got.get_m()) and np.array_equal(ref.get_a(), got.get_a())
    ref.close()
    got.close()
