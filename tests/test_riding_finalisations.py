"""Transforms that a finalisation rides on.  That of an RK4 step's last stage
sets the control block's `done` while the transform runs, so a transform that
looked at `done` itself would have wavefronts of one workgroup part ways
before a barrier: it goes by a flag of its own (transform_idle), which no
finalisation may set."""
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_03706_amd", "csrc")


def _kernels():
    """(name, body) of every __global__ function of the transform sources."""
    for f in sorted(os.listdir(CSRC)):
        if not f.startswith("kernels_fft"):
            continue
        src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())
        for m in re.finditer(r"__global__", src):
            open_ = src.index("{", src.index(")", src.index("InstDesc", m.start())))
            depth, k = 0, open_
            while True:
                depth += {"{": 1, "}": -1}.get(src[k], 0)
                if depth == 0:
                    break
                k += 1
            name = re.search(r"\b(k_\w+)\s*\(", src[m.start():open_]).group(1)
            yield name, src[m.start():k]


def test_transforms_that_carry_finalisations_do_not_read_done():
    bodies = dict(_kernels())
    riding = {n: b for n, b in bodies.items() if "final_any(" in b}
    assert {"k_fft_yz", "k_fft_yzx", "k_fft_yzh", "k_fft_yzs", "k_fft_y1", "k_fft_y"} <= set(riding)
    for name, body in riding.items():
        assert "done" not in body, name
        assert "transform_idle(D)" in body, name
    # the finalisation itself sets that flag in adaptive runs only, whose step end never rides
    rk4, dp45 = open(os.path.join(CSRC, "stage_final.h")).read().split("-- DP45\n")
    assert not re.search(r"idle\s*=", rk4) and dp45.count("C->done = C->idle = 1;") == dp45.count("C->done =")
    api = open(os.path.join(CSRC, "api.cpp")).read()
    assert re.search(r"bool merge_step_end\(const mm_batch\* b\) \{\n  if \(b->method != MM_RK4", api)


@pytest.mark.gpu
@pytest.mark.parametrize("grids", [[(16, 8, 4), (16, 8, 4), (12, 20, 1)], [(4, 100, 20), (4, 100, 20)]])
def test_instances_that_end_at_different_steps(grids):
    """RK4 instances of one batch with different steps: those that end first
    stay as they are while the others go on, and a next run starts from there."""
    from paper_2603_03706_amd import mmcav, workloads as W
    from tests.helpers import gpu_for
    insts = []
    for k, g in enumerate(grids):
        insts.append(W.Instance(grid=g, cell=(5e-9, 4e-9, 3e-9), Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.0, 0.2),
                                demag=W.DEMAG_FFT, omega=np.array([3e10]), kappa=np.array([1e7]), g=np.array([3e8]),
                                m0=W.tilted(g, 10.0, 0.3), a0=np.array([0.05 + 0.02j]), method="rk4",
                                dt0=0.4e-12 / (k + 1)))
    print("ended instances", grids, flush=True)
    ctxs = [gpu_for(i) for i in insts]
    b = mmcav.Batch(ctxs)
    for T in (15e-12, 4.9e-12):
        b.run(T)
        got = [(c.get_m(), c.get_a(), c.stats()["accepted"]) for c in ctxs]
    assert len({n for _, _, n in got}) > 1
    for i, (m, a, n) in zip(insts, got):
        c = gpu_for(i)
        c.run(15e-12)
        c.run(4.9e-12)
        assert n == c.stats()["accepted"]
        assert np.array_equal(c.get_m(), m) and np.array_equal(c.get_a(), a)


@pytest.mark.gpu
def test_finalisations_ride_where_they_cost_no_workgroups():
    """The fused y-z kernel holds fewer workgroups to a CU in the form that
    carries finalisations: one instance's 65 planes are in flight at once all
    the same, and eight instances' 520 only without.  An instance's results do
    not depend on which of the two it is in."""
    from paper_2603_03706_amd import mmcav, workloads as W
    from tests.helpers import gpu_for
    grid = (64, 200, 2)
    insts = [W.Instance(grid=grid, cell=(5e-9,) * 3, Ms=140e3, Aex=3.65e-12, alpha=0.01, B0=(0.01, 0.0, 0.2 + 0.01 * k),
                        demag=W.DEMAG_FFT, omega=np.array([3e10]), kappa=np.array([1e7]), g=np.array([3e8]),
                        m0=W.tilted(grid, 10.0, 0.3), a0=np.array([0.05 + 0.02j]), method="dp45", dt0=0.2e-12)
             for k in range(8)]
    launches, got = [], []
    for n in (1, 8):
        print("riding", n, flush=True)
        ctxs = [gpu_for(i) for i in insts[:n]]
        b = mmcav.Batch(ctxs)
        b.run(4e-12, 1e-5)
        got.append((ctxs[0].get_m(), ctxs[0].get_a()))
        launches.append({p["name"] for p in b.profile(2, 1e-5)})
        b.close()
    assert "final_dp45_2" not in launches[0] and "final_dp45_2" in launches[1]
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
