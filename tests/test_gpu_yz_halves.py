"""The y-z convolution in two halves of the ky range, at the edges of the shapes
it takes, against the oracle: stage kernels and x kernels as readers of its
two terms, both planes of real values, ragged rows and columns."""
import math

import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for, m_err, oracle_for, run_oracle

pytestmark = pytest.mark.gpu

TWO_PI = 2 * math.pi
DT, STEPS = 0.1e-12, 10
# The state takes about four roundings of 2^-24 a step.  The convolution's own
# error, below 2^-24 log2(256 * 64 * 16) of mu0 Ms = 0.18 T, turns m by
# gamma DT of it per step: 1e-9, nothing beside them.
M_TOL = STEPS * 4 * 2.0 ** -24

GRIDS = [(2, 17, 9), (2, 32, 16), (3, 17, 17), (4, 32, 32),        # padded y 64, padded z 32 and 64
         (3, 33, 16), (2, 64, 9), (8, 64, 32), (5, 41, 20),        # 128
         (2, 65, 9), (4, 128, 16), (2, 128, 32), (3, 65, 17), (16, 100, 31)]   # 256


def _inst(grid, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = grid
    m = rng.normal(size=(1, 3, nz, ny, nx))
    m[:, 2] += 1.0
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    G = (rng.uniform(size=(nz, ny, nx)) < 0.8).astype(np.uint8)
    G[0, 0, 0] = 1
    return W.Instance(grid=grid, cell=(5e-9, 4e-9, 3e-9), Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.02, 0.2),
                      demag=W.DEMAG_FFT, geometry=G, omega=np.array([TWO_PI * 5e9]), kappa=np.array([TWO_PI * 1e6]),
                      g=np.array([TWO_PI * 50e6]), m0=(m * G).astype(np.float32), a0=np.array([0.05 + 0.02j]),
                      method="rk4", dt0=DT)


@pytest.mark.parametrize("grid", GRIDS)
def test_halves_against_oracle(grid):
    inst = _inst(grid, sum(grid))
    st = oracle_for(inst)
    run_oracle(st, STEPS * DT)
    ctx = gpu_for(inst)
    b = mmcav.Batch([ctx])
    b.set_fft_path("halves")
    start = ctx.get_state()
    for x in (["stage"] if grid[0] & (grid[0] - 1) == 0 else []) + ["lds"]:
        print("halves", grid, x, flush=True)
        ctx.set_state(start)
        b.set_fft_x(x)
        b.run(STEPS * DT)
        assert m_err(ctx.get_m(), st) <= M_TOL


def test_halves_batch_and_dp45():
    """Several instances of two shapes in one launch sequence and in two, and
    each alone: bit for bit the same; refused where the shape does not fit."""
    insts = [_inst(g, k) for k, g in enumerate([(8, 64, 32), (4, 128, 16), (8, 64, 32)])]
    for i in insts:
        i.method, i.tol = "dp45", 1e-6
    outs = []
    for groups, streams in (([[0], [1], [2]], 1), ([[0, 1, 2]], 1), ([[0, 1, 2]], 2)):
        got = {}
        for members in groups:
            ctxs = [gpu_for(insts[k]) for k in members]
            b = mmcav.Batch(ctxs)
            b.set_streams(streams)
            b.set_fft_path("halves")
            b.run(2e-12, 1e-6)
            got.update({k: c.get_m() for k, c in zip(members, ctxs)})
            b.close()
        outs.append(got)
    for o in outs[1:]:
        for k in o:
            assert np.array_equal(o[k], outs[0][k])
    small = mmcav.Batch([gpu_for(_inst((8, 16, 16), 1))])
    with pytest.raises(mmcav.MMError) as e:
        small.set_fft_path("halves")
    assert e.value.status == mmcav.MM_ERR_ARG
