"""GPU: short runs on a small grid, one call each, from an even and an odd step
count: single steps, passes of two and more, and what remains of them -- the
populations of as many calls of one step, bit for bit."""
import pytest
import torch

from paper_2011_15073_amd import inputs
from pairs import gpu_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,size", [("fp32", (64, 64)), ("fp64", (33, 64)), ("fp32", (31, 256)), ("fp32", (32, 256)), ("fp64", (3, 900)),
                                        ("fp64", (256, 250))])
@pytest.mark.parametrize("start", [0, 1])
def test_short_runs_equal_single_steps(dtype, size, start):
    kw = dict(n=0.8, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6, dtype=dtype)
    a, b = gpu_for(*size, **kw), gpu_for(*size, step_kernel="single", **kw)
    f0, g0 = (torch.from_numpy(x) for x in inputs.random_state(*size, seed=8, amp=0.02, amp_T=0.1))
    for k in range(1, 20):
        for c in (a, b):
            c.set_populations(f0, g0)
            c.step(start)
        a.step(k)
        for _ in range(k):
            b.step(1)
        for x, y in zip(a.populations(), b.populations()):
            assert torch.equal(x, y), k
