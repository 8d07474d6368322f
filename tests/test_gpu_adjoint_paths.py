"""The discrete adjoint on the launch sequences that only some shapes take,
against the oracle's gradient: x passes in kernels of their own (nx above 256:
the recorded demag fields come from the x-inverse output), the halved y-z
strategy by default at 128 x 64 and 256 x 32."""
import numpy as np
import pytest

from paper_2603_03706_amd import workloads as W
from tests.helpers import variant
from tests.test_gpu_adjoint import _check, _check_dp45

pytestmark = pytest.mark.gpu


def _film(grid, seed, a0, **kw):
    rng = np.random.default_rng(seed)
    m0 = W.tilted(grid, 0.0, 0.0).astype(np.float64)
    m0[0, 0] += 0.05 * rng.normal(size=m0.shape[2:])
    m0[0, 1] += 0.05 * rng.normal(size=m0.shape[2:])
    m0 /= np.linalg.norm(m0, axis=1, keepdims=True)
    small = W.multimode_film(8, 6, 3)
    u = np.stack([W.standing_wave(grid, n, 1) for n in (1, 2, 3, 4)]).astype(np.float32)
    return variant(small, grid=grid, u=u, m0=m0.astype(np.float32), a0=np.array(a0), alpha=0.01, dt0=0.5e-12, **kw)


@pytest.mark.parametrize("grid", [(260, 3, 2), (257, 5, 1), (6, 40, 17), (3, 66, 9)])
def test_adjoint_by_shape(grid):
    print("adjoint", grid, flush=True)
    _check(_film(grid, 21, [0.8, 0.3j, 0.0, 0.1], method="rk4"), steps=10, every=4)


@pytest.mark.parametrize("grid", [(260, 3, 2), (6, 40, 17)])
def test_adaptive_adjoint_by_shape(grid):
    _check_dp45(_film(grid, 14, [1.0, 0.2j, 0.0, 0.1]), 4e-12, 1e-6, 4, mode=1)
