"""The kernel that carries whole RK4 steps of small instances: the edges of its
cell counts (one wavefront, one and several blocks of 512 cells, the largest
instance it takes and the first it does not) against the oracle, and the
independence of an instance's results from the batch it runs in."""
import math

import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for, m_err, oracle_for, rel_a_err, run_oracle, variant

pytestmark = pytest.mark.gpu

TWO_PI = 2 * math.pi
DT, STEPS = 0.1e-12, 20
# Per step the state takes about four roundings of 2^-24 (the three stage
# inputs' reach the torque scaled by h |B| gamma < 0.1); 20 steps
M_TOL = STEPS * 4 * 2.0 ** -24
# a gathers i g m^- over g T < 1e-3 of an amplitude of order 0.1
A_TOL = 1e-3 / 0.1 * M_TOL


def _inst(grid, S=1, modes=1, profiled=False, mask=False, demag=W.DEMAG_NONE, method="rk4", seed=0, coupled=False):
    rng = np.random.default_rng(seed)
    nx, ny, nz = grid
    m = rng.normal(size=(S, 3, nz, ny, nx)) * 0.2
    m[:, 2] += np.array([1.0, -1.0])[:S].reshape(S, 1, 1, 1)
    m /= np.linalg.norm(m, axis=1, keepdims=True)
    G = None
    if mask:
        G = (rng.uniform(size=(nz, ny, nx)) < 0.7).astype(np.uint8)
        G[0, 0, 0] = 1
        m = m * G
    J = None
    if coupled:
        J = TWO_PI * 30e6 * (np.ones((modes, modes)) - np.eye(modes))
    return W.Instance(grid=grid, cell=(10e-9,) * 3, Ms=140e3, Aex=3.5e-12, alpha=0.01, B0=(0.01, 0.0, 0.17),
                      Ku=200.0 if S == 2 else 0.0, B_E=5.0 if S == 2 else 0.0, sublattices=S, demag=demag,
                      n_local=(0.2, 0.3, 0.5), geometry=G,
                      omega=TWO_PI * (5e9 + 0.1e9 * np.arange(modes)), kappa=np.full(modes, TWO_PI * 1e6),
                      g=np.full(modes, TWO_PI * 50e6),
                      u=rng.uniform(-1, 1, (modes, nz, ny, nx)).astype(np.float32) if profiled else None,
                      csign=np.array([1, -1], np.int8) if S == 2 else None, photon_coupling=J,
                      drive_amp=np.full(modes, 2e9 + 1e9j), drive_t0=np.full(modes, 1e-12),
                      drive_sigma=np.full(modes, 2e-12), kerr=np.full(modes, 1e8) if coupled else None,
                      m0=m.astype(np.float32), a0=0.1 * np.exp(1j * np.arange(modes)), method=method, dt0=DT)


CASES = [
    ((4, 4, 4), dict()),                                            # one wavefront, full
    ((5, 13, 1), dict(mask=True)),                                  # 65 cells: a second wavefront of one lane
    ((1, 1, 1), dict()),                                            # one cell
    ((8, 8, 8), dict(demag=W.DEMAG_LOCAL, modes=3, profiled=True)),  # 512
    ((27, 19, 1), dict(modes=2, coupled=True)),                     # 513: a second block of one cell
    ((16, 8, 8), dict(S=2, modes=16, profiled=True, mask=True)),    # 1024, most modes, profiles beside two sublattices
    ((25, 41, 1), dict(mask=True, modes=2, profiled=True)),         # 1025: four cells per thread, the last ones empty
    ((16, 16, 8), dict(S=2, demag=W.DEMAG_LOCAL)),                  # 2048, the largest
    ((16, 16, 8), dict(modes=16, profiled=True)),                   # profiles too large for LDS
    ((683, 3, 1), dict(modes=2)),                                   # 2049: the per-stage kernels
    ((9, 7, 3), dict(method="split", modes=2, profiled=True, coupled=True)),
    ((16, 8, 9), dict(method="split", S=2)),
]


@pytest.mark.parametrize("grid,kw", CASES)
def test_small_steps_against_oracle(grid, kw):
    inst = _inst(grid, seed=sum(grid), **kw)
    print("small steps", grid, kw, flush=True)
    st, ctx = oracle_for(inst), gpu_for(inst)
    st.set_sampling(2 * DT, 100)
    ctx.set_sampling(2 * DT, 100)
    T = (STEPS - 0.5) * DT                                          # the last step is clipped
    run_oracle(st, T)
    ctx.run(T)
    assert m_err(ctx.get_m(), st) <= M_TOL
    assert rel_a_err(ctx.get_a(), st.a.numpy()) <= A_TOL
    t_o, a_o, mm_o = st.trace_arrays()
    t_g, a_g, mm_g = ctx.get_trace(100)
    assert np.array_equal(t_g, t_o.numpy())
    assert rel_a_err(a_g, a_o.numpy()) <= A_TOL
    assert np.abs(mm_g - mm_o.numpy()).max() <= M_TOL
    assert ctx.stats()["accepted"] == st.accepted


def test_small_steps_independent_of_the_batch():
    """Alone, in a batch of every size class (one of them on the per-stage
    kernels) and as an open run advanced in pieces: bit for bit the same."""
    insts = [_inst(grid, seed=sum(grid), **kw) for grid, kw in CASES if kw.get("method", "rk4") == "rk4"]
    alone = []
    for inst in insts:
        c = gpu_for(inst)
        c.set_sampling(DT, 100)
        c.run(STEPS * DT)
        alone.append((c.get_m(), c.get_a(), c.get_trace(100)[2]))
    ctxs = [gpu_for(i) for i in insts]
    for c in ctxs:
        c.set_sampling(DT, 100)
    b = mmcav.Batch(ctxs)
    b.run(STEPS * DT)
    for c, ref in zip(ctxs, alone):
        for x, y in zip((c.get_m(), c.get_a(), c.get_trace(100)[2]), ref):
            assert np.array_equal(x, y)
    # open runs take whole steps (a run to an end time clips its last one onto it)
    alone = []
    for inst in insts:
        c = gpu_for(inst)
        b = mmcav.Batch([c])
        b.step(STEPS)
        alone.append((c.get_m(), c.get_a()))
        b.close()
    ctxs = [gpu_for(i) for i in insts]
    b = mmcav.Batch(ctxs)
    b.begin()
    for n in (1, 7, STEPS - 8):
        b.advance(n)
    b.end()
    for c, ref in zip(ctxs, alone):
        assert np.array_equal(c.get_m(), ref[0]) and np.array_equal(c.get_a(), ref[1])


def test_small_steps_nonfinite():
    """An overflowing Kerr cavity stops the run at the last accepted step."""
    inst = variant(_inst((8, 8, 1)), kerr=np.array([1e18]), drive_amp=None, drive_t0=None, drive_sigma=None)
    c = gpu_for(inst)
    with pytest.raises(mmcav.MMError) as e:
        c.run(200 * DT)
    assert e.value.status == mmcav.MM_ERR_NONFINITE
    n = c.stats()["accepted"]
    ref = gpu_for(inst)
    if n:
        ref.run(n * DT)
    assert np.array_equal(c.get_m(), ref.get_m()) and np.array_equal(c.get_a(), ref.get_a())
    assert np.isfinite(c.get_a()).all()
