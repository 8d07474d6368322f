"""State and trace exchanges with the host: through one kernel and a pinned
buffer up to 256 KB, by copies above.  Both routes move bytes, so everything
is compared bit for bit."""
import threading

import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for, variant

pytestmark = pytest.mark.gpu


def _inst(grid, S=1, modes=1):
    return variant(W.paper_sim1(), grid=grid, sublattices=S, B_E=1.0 if S == 2 else 0.0,
                   csign=np.array([1, -1], np.int8) if S == 2 else None, m0=W.tilted(grid, 2.0, 0.3, S),
                   omega=np.full(modes, 3e10), kappa=np.full(modes, 1e6), g=np.full(modes, 3e8),
                   drive_amp=None, drive_t0=None, drive_sigma=None, a0=0.1 + 0.01j * np.arange(modes))


# bytes of state: 12 per cell and sublattice beside the control block
@pytest.mark.parametrize("grid,S,modes", [((8, 8, 1), 1, 1), ((5, 3, 7), 2, 3), ((104, 104, 2), 1, 1),
                                          ((105, 104, 2), 1, 1), ((109, 100, 2), 1, 2)])
@pytest.mark.parametrize("steps", [2, 3])                            # the state in either buffer
def test_state_and_trace(grid, S, modes, steps):
    print("exchange", grid, S, modes, steps, flush=True)
    inst = _inst(grid, S, modes)
    c, d = gpu_for(inst), gpu_for(inst)
    c.set_sampling(inst.dt0, 20000)
    c.run(steps * inst.dt0)
    m, a = c.get_m(), c.get_a()
    # a trace within a pinned buffer, the same by copies, and one cut short
    small, large, cut = c.get_trace(steps + 1), c.get_trace(20000), c.get_trace(steps)
    assert len(small[0]) == len(large[0]) == steps + 1 and len(cut[0]) == steps
    for x, y, z in zip(small, large, cut):
        assert np.array_equal(x, y) and np.array_equal(x[:steps], z)
    assert np.array_equal(large[1][-1], a) and not np.array_equal(small[1][0], small[1][1])
    blob = c.get_state()
    assert np.array_equal(blob[-m.nbytes:].view(np.float32), m.ravel())
    # into a context with trace settings of its own, which stay
    d.set_sampling(2 * inst.dt0, 50)
    d.run(4 * inst.dt0)
    before = d.get_trace(50)
    d.set_state(blob)
    assert np.array_equal(d.get_m(), m) and np.array_equal(d.get_a(), a)
    for x, y in zip(d.get_trace(50), before):
        assert np.array_equal(x, y)
    c.run(5 * inst.dt0)
    d.run(5 * inst.dt0)
    assert np.array_equal(d.get_m(), c.get_m()) and np.array_equal(d.get_a(), c.get_a())


def test_exchanges_from_several_threads():
    """More threads than buffers are kept, each with a context of its own."""
    insts = [_inst((4 + k, 5, 1)) for k in range(8)]
    ref = []
    for inst in insts:
        c = gpu_for(inst)
        c.run(3 * inst.dt0)
        ref.append((c.get_m(), c.get_a()))
    ctxs, bad = [gpu_for(i) for i in insts], []
    start = [c.get_state() for c in ctxs]

    def work(k):
        for _ in range(20):
            ctxs[k].set_state(start[k])
            ctxs[k].run(3 * insts[k].dt0)
            if not (np.array_equal(ctxs[k].get_m(), ref[k][0]) and np.array_equal(ctxs[k].get_a(), ref[k][1])):
                bad.append(k)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(insts))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
