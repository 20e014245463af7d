"""GPU: the sweep's step kernel for states beyond the last-level cache (launch order,
streaming loads).  In case and largest order a sweep is dealt to groups that fit the
cache where their sizes allow; interleaved tiles stay one group, and so does a case
that is larger than the cache by itself."""
import pytest
import torch

import paper_2011_15073_amd as P

pytestmark = pytest.mark.gpu

KW = dict(Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6)


@pytest.mark.parametrize("dtype,sides", [("fp64", ((1301, 1290), (905, 900))), ("fp32", ((1700, 1800), (1501, 1499))),
                                         ("fp64", ((1601, 1603), (70, 33))), ("fp32", ((2301, 2300), (70, 33)))])
@pytest.mark.parametrize("order", ["interleave", "case"])
@pytest.mark.parametrize("n,rounding", [(0.8, "auto"), (1.0, "nearest")])
def test_sweep_beyond_the_cache_equals_single_cases(dtype, sides, order, n, rounding):
    """From rest, bitwise, after an odd number of steps; each of the first two pairs
    is below 256 MB by itself and above it together."""
    kw = dict(KW, n=n, dtype=dtype, rounding=rounding)
    sw = P.Sweep([dict(kw, nx=nx, ny=ny) for nx, ny in sides], order=order)
    sw.step(7)
    for i, (nx, ny) in enumerate(sides):
        one = P.Cavity(nx, ny, step_kernel="single", **kw).step(7)
        for a, b in zip(sw.case(i).populations(torch.float64), one.populations(torch.float64)):
            assert torch.equal(a, b)
    sw.close()
