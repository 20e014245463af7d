"""GPU: a sweep whose states exceed the last-level cache together takes its steps
in groups of cases.  Every case must still equal the same case run alone bit for
bit -- with a case larger than a group of its own, groups that change as cases
stop, an even and an odd chunk, and every tile order."""
import pytest
import torch

import paper_2011_15073_amd as P

pytestmark = pytest.mark.gpu

SIDES = {"fp64": [(1100, 900), (70, 33), (1600, 1601), (900, 1000), (64, 64), (1000, 1100)],
         "fp32": [(1400, 1500), (2301, 2100), (33, 70), (1500, 1300), (1200, 1200)]}


@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
@pytest.mark.parametrize("order", ["case", "largest", "interleave"])
def test_grouped_sweep_equals_cases_run_alone(dtype, order):
    kws = [dict(nx=nx, ny=ny, n=(0.8, 1.0)[i % 2], Da=1e-2, Ra=1e4, Pr=10.0, eps=0.6, dtype=dtype)
           for i, (nx, ny) in enumerate(SIDES[dtype])]
    sw = P.Sweep(kws, order=order)
    sw.step(3)
    steps, res = sw.run(tol=1e-30, check_every=5, max_steps=13)
    for i, kw in enumerate(kws):
        kw = dict(kw)
        alone = P.Cavity(kw.pop("nx"), kw.pop("ny"), step_kernel="single", **kw)
        alone.step(sw.case(i).steps)
        dt = torch.float64 if dtype == "fp64" else torch.float32
        for x, y in zip(alone.populations(dt), sw.case(i).populations(dt)):
            assert torch.equal(x, y), (i, steps)
    del alone
    sw.close()


def test_groups_follow_the_cases_that_stop():
    kws = [dict(nx=1100, ny=900 + 10 * i, n=1.0, Da=1e-2, Ra=(1e2, 1e5)[i % 2], Pr=10.0, eps=0.6, dtype="fp64")
           for i in range(4)]
    alone = []
    for kw in kws:
        kw = dict(kw)
        c = P.Cavity(kw.pop("nx"), kw.pop("ny"), step_kernel="single", **kw)
        c.step(4)
        first = c.residual()
        c.step(4)
        alone.append((first, c.residual()))
    tol = sorted(r[1] for r in alone)[1] * 1.0000001  # two of the four stop at the second check
    assert tol < min(r[0] for r in alone)
    sw = P.Sweep(kws)
    steps, res = sw.run(tol=tol, check_every=4, max_steps=16)
    assert sorted(steps)[:2] == [8, 8] and sorted(steps)[2] > 8
    for i, kw in enumerate(kws):
        kw = dict(kw)
        c = P.Cavity(kw.pop("nx"), kw.pop("ny"), step_kernel="single", **kw)
        c.step(steps[i])
        for x, y in zip(c.populations(torch.float64), sw.case(i).populations(torch.float64)):
            assert torch.equal(x, y), (i, steps)
