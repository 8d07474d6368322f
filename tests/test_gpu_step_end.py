"""The finalisation of an RK4 step rides on the next step's first transform
where every FFT group has its x passes in the stage kernels.  Steps launched
one at a time have it in a launch of its own: bit for bit the same."""
import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for

pytestmark = pytest.mark.gpu


def _inst(grid, **kw):
    rng = np.random.default_rng(sum(grid))
    nx, ny, nz = grid
    m = rng.normal(size=(1, 3, nz, ny, nx)) * 0.2
    m[:, 2] += 1.0
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    return W.Instance(**{**dict(grid=grid, cell=(5e-9,) * 3, Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.0, 0.2),
                                demag=W.DEMAG_FFT, omega=np.full(2, 3e10), kappa=np.full(2, 1e7), g=np.full(2, 3e8),
                                u=rng.uniform(-1, 1, (2, nz, ny, nx)).astype(np.float32), m0=m.astype(np.float32),
                                a0=np.array([0.1, 0.05j]), method="rk4", dt0=0.5e-12), **kw})


CASES = {
    "stage kernels": [(12, 10, 3)],
    "two groups": [(16, 8, 4), (12, 20, 1)],
    "separate x passes": [(300, 4, 1)],                              # nx above 256: nothing rides
    "one group of each": [(16, 8, 4), (300, 4, 1)],
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("extra", [False, True])                     # beside an instance without FFT demag
def test_step_end_rides(name, extra):
    print("step end", name, extra, flush=True)
    insts = [_inst(g) for g in CASES[name]]
    if extra:
        insts.append(_inst((43, 25, 2), demag=W.DEMAG_LOCAL, n_local=(0.2, 0.3, 0.5)))
    outs = []
    for pieces in ([1] * 37, [37], [3, 34]):
        ctxs = [gpu_for(i) for i in insts]
        for c, i in zip(ctxs, insts):
            c.set_sampling(i.dt0, 60)
        b = mmcav.Batch(ctxs)
        b.begin()
        for k in pieces:
            b.advance(k)
        b.end()
        outs.append([(c.get_m(), c.get_a(), c.get_trace(60)[2], c.stats()["accepted"]) for c in ctxs])
        b.close()
    for o in outs[1:]:
        for x, y in zip(o, outs[0]):
            assert all(np.array_equal(p, q) for p, q in zip(x, y))
            assert x[3] == 37
    # a run that ends between two steps of a graph, the last step clipped, and one that goes on from it
    ctxs = [gpu_for(i) for i in insts]
    b = mmcav.Batch(ctxs)
    T = insts[0].dt0
    b.run(10.5 * T)
    assert all(c.stats()["accepted"] == 11 for c in ctxs)
    first = [(c.get_m(), c.get_a()) for c in ctxs]
    b.run(5 * T)
    for i, f, c in zip(insts, first, ctxs):
        d = gpu_for(i)
        d.run(10.5 * T)
        assert np.array_equal(d.get_m(), f[0]) and np.array_equal(d.get_a(), f[1])
        d.run(5 * T)
        assert np.array_equal(d.get_m(), c.get_m()) and np.array_equal(d.get_a(), c.get_a())
