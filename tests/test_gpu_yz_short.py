"""The y-z convolution of few z planes at the edges of the shapes it takes,
against the oracle, and the finalisations that ride on every strategy's
first launch."""
import math

import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for, m_err, oracle_for, run_oracle

pytestmark = pytest.mark.gpu

TWO_PI = 2 * math.pi
DT, STEPS = 0.1e-12, 10
M_TOL = STEPS * 4 * 2.0 ** -24        # four roundings of 2^-24 of |m| = 1 a step; the field's error turns m by 1e-9

GRIDS = [(2, 3, 2), (3, 4, 3), (4, 5, 8), (5, 8, 5), (2, 9, 2), (3, 16, 4), (8, 17, 3), (4, 32, 8), (2, 33, 2),
         (3, 64, 7), (2, 65, 2), (2, 128, 4), (3, 100, 6),                       # padded z of 4, 8, 16
         (1, 3, 1), (2, 4, 1), (5, 8, 1), (3, 9, 1), (4, 17, 1), (2, 33, 1), (6, 64, 1), (3, 100, 1), (2, 129, 1),
         (4, 256, 1)]                                                            # one plane


def _inst(grid, method="rk4", modes=1):
    rng = np.random.default_rng(sum(grid))
    nx, ny, nz = grid
    m = rng.normal(size=(1, 3, nz, ny, nx))
    m[:, 2] += 1.0
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    return W.Instance(grid=grid, cell=(5e-9, 4e-9, 3e-9), Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.02, 0.2),
                      demag=W.DEMAG_FFT, omega=TWO_PI * (5e9 + 1e8 * np.arange(modes)), kappa=np.full(modes, TWO_PI * 1e6),
                      g=np.full(modes, TWO_PI * 50e6), u=rng.uniform(-1, 1, (modes, nz, ny, nx)).astype(np.float32),
                      m0=m.astype(np.float32), a0=0.05 * np.exp(1j * np.arange(modes)), method=method, dt0=DT, tol=1e-6)


@pytest.mark.parametrize("grid", GRIDS)
def test_short_against_oracle(grid):
    inst = _inst(grid)
    print("short", grid, flush=True)
    st, ctx = oracle_for(inst), gpu_for(inst)
    b = mmcav.Batch([ctx])
    b.set_fft_path("short")
    run_oracle(st, STEPS * DT)
    b.run(STEPS * DT)
    assert m_err(ctx.get_m(), st) <= M_TOL
    assert np.abs(ctx.get_a() - st.a.numpy()).max() <= 1e-8


@pytest.mark.parametrize("grid,paths", [((8, 12, 4), ("short", "fused", "split", "splitx")),
                                        ((6, 20, 8), ("short", "reg", "fused", "split", "splitx")),
                                        ((5, 40, 1), ("short", "fused", "split"))])
def test_finalisation_on_every_path(grid, paths):
    """Sixteen modes over more workgroups than one: the cavity amplitudes after
    adaptive steps agree between the strategies to the rounding of the state."""
    out = {}
    for p in paths:
        inst = _inst(grid, "rk4", modes=16)
        c = gpu_for(inst)
        b = mmcav.Batch([c])
        b.set_fft_path(p)
        b.step(STEPS)
        out[p] = (c.get_m(), c.get_a())
    for p in paths[1:]:
        assert np.abs(out[p][0] - out[paths[0]][0]).max() <= M_TOL
        # a gathers g T < 1e-3 of the difference of m^-
        assert np.abs(out[p][1] - out[paths[0]][1]).max() <= 1e-3 * M_TOL
