"""GPU: the Nusselt number, the residual and the stream function where their
kernels split the work differently: rows below, at and above one wave's 64 and
one column block's, more rows than one round of the reduction's slots, row ends
inside a 64-node segment, both step parities, and contexts that take over a
destroyed context's result slots."""
import numpy as np
import pytest
import torch

from paper_2011_15073_amd import inputs
from pairs import gpu_for

pytestmark = pytest.mark.gpu

SIZES = [(2, 2), (3, 63), (64, 64), (65, 65), (70, 128), (130, 129), (2, 70001), (4099, 33), (700, 1031)]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("dtype,k", [("fp32", 1), ("fp64", 2), ("fp64", 3), ("fp16", 2)])
def test_observables_match_the_fields(size, dtype, k):
    nx, ny = size
    c = gpu_for(nx, ny, dtype=dtype, n=0.8, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6, rounding="nearest")
    f0, g0 = inputs.random_state(nx, ny, seed=3, amp=0.02, amp_T=0.1)
    c.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    c.residual()
    t0 = c.populations()[1].sum(0).cpu().numpy()
    c.step(k)
    U, _, T = (x.cpu().numpy() for x in c.fields())
    # the same values summed in another order: FP64 rounding of ny terms of size 9 nx
    nu = (nx * (8.0 - 9.0 * T[:, 0] + T[:, 1]) / 3.0).mean()
    # theta of the fields is one rounding in the compute type, of a value around 1/2, away
    e = 6e-8 if dtype != "fp64" else 2.3e-16
    assert c.nu() == pytest.approx(nu, abs=10 * nx * 2 * e)
    g1 = c.populations()[1].sum(0).cpu().numpy()
    assert c.residual() == pytest.approx(np.abs(g1 - t0).max(), abs=16 * e)
    assert c.residual() == 0.0
    psi = c.stream_function().cpu().numpy()
    ref = (np.cumsum(U, 0) - 0.5 * U) / nx
    assert np.abs(psi - ref).max() <= 1e-13 * ny * max(np.abs(U).max(), 1e-300) / nx


def test_result_slots_of_destroyed_contexts_are_taken_over():
    kw = dict(dtype="fp64", n=0.8, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6)
    ref = [gpu_for(n, n, **kw).step(6).nu() for n in (20, 33)]
    for _ in range(3):
        cs = [gpu_for(n, n, **kw) for n in (20, 33) * 40]  # more than are kept
        for c in cs:
            c.step(6)
        assert [c.nu() for c in cs] == ref * 40
        del cs, c
