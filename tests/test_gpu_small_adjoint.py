"""The kernel that carries whole reverse steps of small instances: the edges of
its cell counts (one wavefront, one and two blocks of 512 cells, grad u
and the profiles in and out of LDS, the first instance it leaves to the
per-stage kernels) against the oracle's autograd gradient, with the relative
error of 1e-3 that the adjoint is held to everywhere (5e-3 for m0)."""
import pytest

from paper_2603_03706_amd import workloads as W
from tests.test_gpu_adjoint import _check
from tests.test_gpu_small_steps import _inst

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,kw", [
    ((1, 1, 1), dict()),                                             # one cell
    ((4, 4, 4), dict(modes=2)),                                      # one wavefront, full
    ((5, 13, 1), dict(mask=True, profiled=True)),                    # 65 cells: a second wavefront of one lane
    ((8, 8, 8), dict(demag=W.DEMAG_LOCAL, modes=3, profiled=True)),   # 512
    ((27, 19, 1), dict(modes=2, coupled=True)),                      # 513: a second block of one cell
    ((16, 8, 8), dict(S=2, modes=16, profiled=True, mask=True)),     # 1024, two sublattices; grad u outside LDS
    ((16, 16, 4), dict(modes=12, profiled=True)),                    # 1024; grad u in LDS, the profiles not
    ((25, 41, 1), dict(mask=True, modes=2, profiled=True)),          # 1025: the per-stage kernels
])
def test_small_reverse_steps_against_oracle(grid, kw):
    print("small reverse steps", grid, kw, flush=True)
    _check(_inst(grid, seed=sum(grid), **kw), steps=12, every=5, mode=0)


@pytest.mark.parametrize("grid,kw", [
    ((25, 41, 1), dict(modes=1)),                                    # one mode, uniform
    ((25, 41, 1), dict(modes=3, profiled=True, coupled=True)),       # an odd mode in a group of four, mode coupling
    ((43, 12, 2), dict(S=2, modes=4, profiled=True, mask=True)),     # 1032 cells, two sublattices, a full group
    ((25, 41, 1), dict(modes=5, profiled=True)),                     # a second group of one mode
    ((43, 25, 1), dict(modes=16, profiled=True, mask=True)),         # 1075, the most modes
])
def test_per_stage_reverse_sums_against_oracle(grid, kw):
    """The sums of the per-stage kernels, four modes at a time, on instances
    too large for the kernel above."""
    print("per-stage reverse steps", grid, kw, flush=True)
    _check(_inst(grid, seed=sum(grid), **kw), steps=6, every=4, mode=0)
