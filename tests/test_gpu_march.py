"""GPU: the multi-step pass of large cavities (pm_march.hip), which
PM_STEP_PAIR also takes on small ones.  Its per-node arithmetic is the
single-step kernel's, so the populations must be the same bit for bit -- on
grids narrower than a strip, with one column more or less than one, two or
several strips, with rows below, at and above one workgroup's, from an even
and an odd step count, for every remainder of a run, and through graph
replay -- and PM_STEP_AUTO must take it with FP32 and FP64 state alike on
large ragged grids."""
import pytest
import torch

import paper_2011_15073_amd as P
from paper_2011_15073_amd import inputs
from pairs import gpu_for

pytestmark = pytest.mark.gpu

# strips are 64 columns, 58 apart (three steps per pass) or 60 (two)
SIZES = [(2, 2), (3, 5), (63, 9), (64, 64), (65, 17), (122, 40), (123, 3), (124, 2), (125, 31), (290, 130), (301, 61)]


def compare(size, dtype, step_kernel, runs, n, logda, rounding):
    nx, ny = size
    kw = dict(n=n, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6, rounding=rounding, dtype=dtype)
    ld = inputs.logda_field(max(nx, ny), seed=2)[:ny, :nx].copy() if logda else None
    a = gpu_for(nx, ny, step_kernel=step_kernel, logda=ld, **kw)
    b = gpu_for(nx, ny, step_kernel="single", logda=ld, **kw)
    f0, g0 = inputs.random_state(nx, ny, seed=21, amp=0.02, amp_T=0.1)
    for c in (a, b):
        c.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    for k in runs:
        a.step(k)
        for _ in range(k):
            b.step(1)
        fa, ga = a.populations()
        fb, gb = b.populations()
        assert a.steps == b.steps
        assert torch.equal(fa, fb) and torch.equal(ga, gb), (k, a.steps)
    assert a.nu() == b.nu()


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("n,logda,rounding", [(1.0, False, "nearest"), (0.6, True, "nearest"), (0.8, False, "stochastic"),
                                              (1.0, True, "stochastic")])
def test_pass_equals_single_steps(size, n, logda, rounding):
    compare(size, "fp32", "pair", (4, 6, 1, 5, 7, 8, 9, 10, 11, 13, 131), n, logda, rounding)


@pytest.mark.parametrize("dtype,size,n", [("fp32", (2503, 2201), 0.8), ("fp64", (3001, 2701), 0.8),
                                          ("fp64", (707, 11407), 0.8), ("fp32", (1109, 1087), 1.0),
                                          ("fp64", (1301, 1303), 1.0)])
def test_large_ragged_grids_take_the_pass(dtype, size, n):
    need = {s: P.workspace_bytes(P.make_params(*size, dtype=dtype, step_kernel=s, n=n, Ra=1e5, Pr=10.0))
            for s in ("auto", "single")}
    assert need["auto"] > need["single"]
    compare(size, dtype, "auto", (6, 5, 13), n, False, "nearest")
