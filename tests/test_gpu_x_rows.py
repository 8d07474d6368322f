"""The x passes inside the stage kernels for widths that are no power of two
(workgroups with threads that have no cell, padding inside the lines), at the
edges of the range, against the oracle and the separate x kernels."""
import math

import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for, m_err, oracle_for, run_oracle

pytestmark = pytest.mark.gpu

TWO_PI = 2 * math.pi
DT, STEPS = 0.1e-12, 10
M_TOL = STEPS * 4 * 2.0 ** -24        # four roundings of 2^-24 of |m| = 1 a step; the field's error turns m by 1e-9

GRIDS = [(3, 5, 2), (5, 1, 1), (7, 3, 3), (21, 4, 2), (33, 3, 1), (100, 6, 4), (127, 2, 1), (129, 5, 1), (171, 2, 2),
         (255, 3, 1), (256, 3, 1), (257, 2, 1), (2, 3, 3)]


def _inst(grid, method="rk4"):
    rng = np.random.default_rng(sum(grid))
    nx, ny, nz = grid
    m = rng.normal(size=(1, 3, nz, ny, nx))
    m[:, 2] += 1.0
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    return W.Instance(grid=grid, cell=(5e-9, 4e-9, 3e-9), Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.02, 0.2),
                      demag=W.DEMAG_FFT, omega=np.array([TWO_PI * 5e9, TWO_PI * 5.1e9]), kappa=np.full(2, TWO_PI * 1e6),
                      g=np.full(2, TWO_PI * 50e6), u=rng.uniform(-1, 1, (2, nz, ny, nx)).astype(np.float32),
                      m0=m.astype(np.float32), a0=np.array([0.05 + 0.02j, 0.01j]), method=method, dt0=DT, tol=1e-6)


@pytest.mark.parametrize("grid", GRIDS)
def test_x_rows_against_oracle(grid):
    inst = _inst(grid)
    print("x rows", grid, flush=True)
    st, ctx = oracle_for(inst), gpu_for(inst)
    run_oracle(st, STEPS * DT)
    ctx.run(STEPS * DT)
    assert m_err(ctx.get_m(), st) <= M_TOL
    assert np.abs(ctx.get_a() - st.a.numpy()).max() <= 1e-8
    # adaptive steps (stage-2 input and run start through the x-forward kernel) against the separate x kernels:
    # the error estimate is mostly rounding here, so the step sizes differ, each step within the tolerance of 1e-6
    inst = _inst(grid, "dp45")
    got = []
    for x in (None, "lds"):
        c = gpu_for(inst)
        b = mmcav.Batch([c])
        if x:
            b.set_fft_x(x)
        b.run(1e-12, 1e-6)
        got.append(c.get_m())
        steps = c.stats()["accepted"]
    assert np.abs(got[0] - got[1]).max() <= 2 * steps * 1e-6
