"""GPU: small cavities, where PM_STEP_AUTO takes several steps per launch tile by
tile (pm_tile.hip).  The per-node arithmetic is the single-step kernel's, so the
populations must be the same bit for bit -- on grids smaller than one region,
with one node more or less than a region or a whole number of them, with long
thin shapes, and up to the largest grid that takes this path -- from an even and
an odd step count, for every remainder of a run, and through graph replay."""
import numpy as np
import pytest
import torch

from paper_2011_15073_amd import inputs
from pairs import gpu_for

pytestmark = pytest.mark.gpu

SIZES = [(2, 2), (3, 5), (15, 17), (16, 16), (17, 16), (33, 21), (64, 64), (9, 700), (700, 9), (160, 160), (256, 200)]
BIG32 = [(384, 384), (520, 520)]


@pytest.mark.parametrize("dtype,size", [(d, s) for s in SIZES for d in ("fp32", "fp64")] +
                         [("fp64", s) for s in ((264, 264), (255, 333), (300, 300), (360, 360))] + [("fp32", s) for s in BIG32])
@pytest.mark.parametrize("n,logda,rounding", [(1.0, False, "nearest"), (0.6, True, "nearest"), (0.8, False, "auto")])
def test_tile_kernel_equals_single_steps(dtype, size, n, logda, rounding):
    nx, ny = size
    kw = dict(n=n, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6, rounding=rounding)
    ld = inputs.logda_field(max(nx, ny), seed=2)[:ny, :nx].copy() if logda else None
    a = gpu_for(nx, ny, dtype=dtype, logda=ld, **kw)
    b = gpu_for(nx, ny, dtype=dtype, logda=ld, step_kernel="single", **kw)
    f0, g0 = inputs.random_state(nx, ny, seed=21, amp=0.02, amp_T=0.1)
    for c in (a, b):
        c.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    for k in (2, 3, 1, 5, 6, 7, 9, 11, 13, 17, 131):
        a.step(k)
        for _ in range(k):
            b.step(1)
        fa, ga = a.populations()
        fb, gb = b.populations()
        assert a.steps == b.steps
        assert torch.equal(fa, fb) and torch.equal(ga, gb), (k, a.steps)
    assert a.nu() == b.nu()


def test_workspace_of_a_small_grid_does_not_depend_on_the_step_kernel():
    import paper_2011_15073_amd as P
    for dtype in ("fp32", "fp64"):
        sizes = {P.workspace_bytes(P.make_params(100, 77, dtype=dtype, step_kernel=s)) for s in ("auto", "single")}
        assert len(sizes) == 1


def test_tile_kernel_with_a_nan_reports_divergence():
    """A NaN in the populations reaches the residual through the tile kernel."""
    c = gpu_for(40, dtype="fp64", n=0.8, Da=1e-2, Ra=1e4, Pr=10.0, eps=0.6)
    f, g = inputs.random_state(40, 40, seed=5, amp=0.0, amp_T=0.0)
    g[2, 7, 0] = np.nan  # planted from the host
    c.set_populations(torch.from_numpy(f), torch.from_numpy(g))
    c.step(24)
    with pytest.raises(Exception) as e:
        c.residual()
    assert getattr(e.value, "code", None) == -3
