"""GPU: the step kernels' two memory orders.  A state of at most 256 MB (it
stays in the last-level cache) takes its tiles in XCD bands with cached loads,
a larger one in launch order with streaming loads; a sweep chooses by the sum
over its live cases.  Neither may change a result."""
import numpy as np
import pytest
import torch

from paper_2011_15073_amd import inputs
from pairs import gpu_for, oracle_for

pytestmark = pytest.mark.gpu

KW = dict(n=0.8, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6)


@pytest.mark.parametrize("dtype,sides", [("fp64", ((1301, 1290), (905, 900))), ("fp32", ((1700, 1800), (1501, 1499)))])
def test_sweep_above_the_cache_equals_cases_below_it(dtype, sides):
    """Two cases whose states are below 256 MB each (alone: XCD bands) and above
    it together (streaming): bitwise the same after 5 steps, ragged tiles
    included."""
    import ctypes as C

    import paper_2011_15073_amd as P
    sw = P.Sweep([dict(KW, nx=nx, ny=ny, dtype=dtype) for nx, ny in sides])
    states = []
    for i, (nx, ny) in enumerate(sides):
        f, g = inputs.random_state(nx, ny, seed=3 + i, amp=0.02, amp_T=0.1)
        states.append([torch.from_numpy(a).cuda().contiguous() for a in (f, g)])
        v = sw.case(i)
        v._c(P._lib.lib.pm_set_populations(v._h, *(C.c_void_p(t.data_ptr()) for t in states[i]), P.PM_FP64))
    torch.cuda.synchronize()
    sw.step(5)
    for i, (nx, ny) in enumerate(sides):
        one = gpu_for(nx, ny, dtype=dtype, step_kernel="single", **KW)
        one.set_populations(*states[i])
        one.step(5)
        dt = torch.float64 if dtype == "fp64" else torch.float32
        for a, b in zip(sw.case(i).populations(dt), one.populations(dt)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("size", [(1500, 1499), (1600, 1601)])
def test_fp64_step_on_both_sides_of_the_limit(size):
    """FP64 states of 252 MB and 287 MB against the oracle after 3 steps from a
    random state, every population (the 1e-13 bar of the random-state tests)."""
    nx, ny = size
    f0, g0 = inputs.random_state(nx, ny, seed=9, amp=0.02, amp_T=0.1)
    cav = gpu_for(nx, ny, dtype="fp64", step_kernel="single", **KW)
    cav.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    cav.step(3)
    orc = oracle_for(nx, ny, **KW)
    orc.set_state(f0, g0)
    orc.step(3)
    for a, b in zip(cav.populations(), orc.state()):
        assert np.abs(a.cpu().numpy() - b).max() <= 1e-13
