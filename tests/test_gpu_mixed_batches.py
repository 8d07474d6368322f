"""Batches of small instances of unlike kinds (sublattices, cells per thread,
profiles) with and without larger ones: the launches run beside each other."""
import time

import numpy as np
import pytest
import torch

from paper_2603_03706_amd import mmcav, workloads as W
from tests.helpers import gpu_for
from tests.test_gpu_small_steps import DT, STEPS, _inst

pytestmark = pytest.mark.gpu

KINDS = [((8, 8, 1), {}), ((16, 16, 8), dict(modes=16, profiled=True)), ((16, 16, 4), dict(S=2)),
         ((27, 19, 1), dict(modes=2, profiled=True)), ((16, 16, 8), dict(S=2, modes=4, profiled=True)), ((9, 9, 9), {})]
LARGE = [((683, 3, 1), dict(modes=2)), ((16, 12, 4), dict(demag=W.DEMAG_FFT))]


def _insts(large):
    return [_inst(g, seed=k, **kw) for k, (g, kw) in enumerate(KINDS + (LARGE if large else []))]


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("streams", [1, 2])
def test_mixed_batch_equals_each_alone(large, streams):
    insts = _insts(large)
    print("mixed", large, streams, flush=True)
    ctxs = [gpu_for(i) for i in insts]
    for c in ctxs:
        c.set_sampling(DT, 200)
    b = mmcav.Batch(ctxs)
    b.set_streams(streams)
    b.run((STEPS - 0.5) * DT)                       # the last step is clipped
    got = [[(c.get_m(), c.get_a(), *c.get_trace(200))] for c in ctxs]
    b.begin()
    for n in (1, 40, 7):
        b.advance(n)
    assert b.counts()[0] == len(insts) * (STEPS + 48)
    b.end()
    for c, g in zip(ctxs, got):
        g.append((c.get_m(), c.get_a(), *c.get_trace(200)))
    for i, g in zip(insts, got):
        c = gpu_for(i)
        c.set_sampling(DT, 200)
        c.run((STEPS - 0.5) * DT)
        want = [(c.get_m(), c.get_a(), *c.get_trace(200))]
        one = mmcav.Batch([c])
        one.step(48)
        want.append((c.get_m(), c.get_a(), *c.get_trace(200)))
        for x, y in zip(g, want):
            assert all(np.array_equal(p, q) for p, q in zip(x, y))


def _us(insts, steps=512):
    ctxs = [gpu_for(i) for i in insts]
    b = mmcav.Batch(ctxs)
    b.begin()
    b.advance(64)
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        b.advance(steps)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    b.end()
    b.close()
    return 1e6 * best / steps


@pytest.mark.parametrize("other", [((683, 3, 1), {}), ((16, 16, 8), dict(S=2, modes=16, profiled=True))])
def test_unlike_instances_run_beside_each_other(other):
    """A 2048-cell instance of sixteen profiled modes (about 96 us per step on
    one CU) beside one in per-stage launches (33 us) or of another kind (106):
    the step takes the longer of the two, not their sum."""
    a, c = _inst((16, 16, 8), modes=16, profiled=True), _inst(other[0], **other[1])
    alone = [_us([a]), _us([c])]
    # (streams of one hardware queue follow each other, whichever they are: three batches, each with its own)
    both = min(_us([a, c]) for _ in range(3))
    print("beside each other", other, alone, both, flush=True)
    assert both <= max(alone) + 0.5 * min(alone)
