"""Where the x passes run for widths that are no power of two: the stage
kernels as readers of the halved strategy's two terms, and the way back to
them after another choice."""
import numpy as np
import pytest

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for, m_err, oracle_for, run_oracle
from tests.test_gpu_yz_halves import DT, M_TOL, STEPS, _inst

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,halves", [((3, 17, 17), True), ((5, 41, 20), True), ((3, 65, 17), True), ((16, 100, 31), True),
                                         ((100, 17, 9), True), ((100, 60, 20), True), ((21, 4, 2), False), ((129, 5, 1), False),
                                         ((255, 17, 9), True)])
def test_x_passes_back_in_the_stage_kernels(grid, halves):
    inst = _inst(grid, sum(grid))
    st = oracle_for(inst)
    run_oracle(st, STEPS * DT)
    ctx = gpu_for(inst)
    b = mmcav.Batch([ctx])
    if halves:
        b.set_fft_path("halves")
    start, got = ctx.get_state(), {}
    for x in ("default", "lds", "stage", "lds", "stage"):
        print("x place", grid, x, flush=True)
        ctx.set_state(start)
        if x != "default":
            b.set_fft_x(x)
        b.run(STEPS * DT)
        assert m_err(ctx.get_m(), st) <= M_TOL, x
        got.setdefault(x, []).append(ctx.get_m())
    for x in ("default", "stage"):
        assert all(np.array_equal(m, got["default"][0]) for m in got[x])


def test_x_passes_of_several_widths():
    """A mixed batch returns as a whole, and one with a width that the stage
    kernels cannot take is refused as a whole, unchanged."""
    insts = [_inst((16, 17, 9), 1), _inst((100, 9, 9), 2)]
    outs = []
    for back in (False, True):
        ctxs = [gpu_for(i) for i in insts]
        b = mmcav.Batch(ctxs)
        if back:
            b.set_fft_x("lds")
            b.set_fft_x("stage")
        b.run(STEPS * DT)
        outs.append([c.get_m() for c in ctxs])
    assert all(np.array_equal(p, q) for p, q in zip(*outs))
    wide = mmcav.Batch([gpu_for(insts[0]), gpu_for(_inst((300, 5, 2), 3))])
    wide.set_fft_x("lds")
    with pytest.raises(mmcav.MMError) as e:
        wide.set_fft_x("stage")
    assert e.value.status == mmcav.MM_ERR_ARG
