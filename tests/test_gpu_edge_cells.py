"""GPU: cells at the ends of what the parameters allow, in the forward update and
the adjoint."""
import numpy as np
import pytest
import torch

import paper_2011_15073_amd as P
from paper_2011_15073_amd import inputs
from test_gpu_adjoint import torch_vjp

pytestmark = pytest.mark.gpu

PHYS = dict(Pr=10.0, eps=0.6)
CLEAR = [np.inf, 400.0, 308.5, 200.0]  # log10 Da: resistance 0, underflowing to 0, subnormal, tiny


def plane(nx, ny, cells):
    """A log10 Da plane with every seventh cell from `cells`, in turn."""
    ld = inputs.logda_field(max(nx, ny), seed=3)[:ny, :nx].copy()
    mask = np.zeros(nx * ny, bool)
    mask[::7] = True
    ld.reshape(-1)[mask] = np.resize(cells, mask.sum())
    return ld, mask.reshape(ny, nx)


@pytest.mark.parametrize("n", [0.7, 1.0, 1.4])
@pytest.mark.parametrize("grid", [(21, 13), (70, 19)])
@pytest.mark.parametrize("dtype", ["fp64", "fp32"])
def test_adjoint_step_with_clear_cells(n, grid, dtype):
    """Cells without porous resistance against autograd, whose plane holds 200
    there: the square root of 1e-200 / N^2 vanishes in every sum, and its
    derivative is finite.  The bars are those of the plane without such cells.
    An FP32 state is read back, so that both sides start from the same numbers
    (the library holds it as deviations from the rest weights rounded to FP32)."""
    nx, ny = grid
    ld, clear = plane(nx, ny, CLEAR)
    lam = np.random.default_rng(11).standard_normal((14, ny, nx))
    cav = P.Cavity(nx, ny, dtype=dtype, logda=torch.from_numpy(ld), n=n, Ra=1e4, **PHYS)
    cav.set_populations(*(torch.from_numpy(a) for a in inputs.random_state(nx, ny, seed=7, amp=0.03, amp_T=0.2)))
    f0, g0 = (x.cpu().numpy() for x in cav.populations(torch.float64))
    lam_g, gld, gn, gRa = P.vjp_step(cav, torch.from_numpy(lam))
    if dtype == "fp32":  # the library holds the plane in the compute type as well
        ld = ld.astype(np.float32).astype(np.float64)
        for x, w in ((f0, inputs.W9), (g0, 0.5 * inputs.W5)):
            x += (w - w.astype(np.float32))[:, None, None]
    tf, tg, tld, tn, tRa = torch_vjp(nx, ny, n, 1e4, f0, g0, np.where(clear, 200.0, ld), lam, 0)
    ref = np.concatenate([tf, tg])
    assert np.abs(lam_g.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()
    assert np.abs(gld.cpu().numpy() - tld).max() <= 1e-10 * np.abs(tld).max()
    assert gn == pytest.approx(tn, rel=1e-9, abs=1e-14)
    assert gRa == pytest.approx(tRa, rel=1e-9, abs=1e-14)


@pytest.mark.parametrize("T,C", [(6, 3)])
def test_backward_with_clear_cells(T, C):
    ld, clear = plane(21, 13, CLEAR)
    grads = []
    for l in (ld, np.where(clear, 200.0, ld)):
        cav = P.Cavity(21, 13, dtype="fp64", logda=torch.from_numpy(l), n=0.8, Ra=1e4, **PHYS)
        adj = P.Adjoint(cav, T, C)
        adj.forward()
        gld, gn, gRa = adj.backward()
        adj.close()
        grads.append((gld.cpu().numpy(), gn, gRa))
    (a, an, aR), (b, bn, bR) = grads
    # from rest, cells of equal resistance to rounding
    assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    assert an == pytest.approx(bn, rel=1e-12) and aR == pytest.approx(bR, rel=1e-12)
