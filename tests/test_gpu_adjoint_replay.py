"""GPU: pm_adjoint_backward against the chain of single adjoint steps it stands
for (each of which is checked against autograd elsewhere).  Up to a grid limit
the backward pass replays the next segment in the adjoint's own launches, above
it on a second stream: every split of a trajectory into segments, including
segments of one step, a short last one and a single one, on grids whose rows end
inside, at and just past a wave, on both sides of the limit."""
import pytest
import torch

import paper_2011_15073_amd as P
from paper_2011_15073_amd import inputs

pytestmark = pytest.mark.gpu

KW = dict(n=0.8, Ra=1e4, Pr=10.0, eps=0.6, rounding="nearest")


def chain(cav, T):
    """Gradients of the hot-wall Nusselt number over T steps from cav's state."""
    nx, ny = cav.nx, cav.ny
    states = []
    for _ in range(T):
        states.append([x.clone() for x in cav.populations(torch.float64)])
        cav.step(1)
    lam = torch.zeros(14, ny, nx, dtype=torch.float64, device=states[0][0].device)
    lam[9:, :, 0] = -3.0 * nx / ny
    lam[9:, :, 1] = nx / (3.0 * ny)
    gl, gn, gRa = 0.0, 0.0, 0.0
    for f, g in reversed(states):
        cav.set_populations(f, g)
        lam, l, n, r = P.vjp_step(cav, lam)
        gl, gn, gRa = gl + l, gn + n, gRa + r
    return gl, gn, gRa


@pytest.mark.parametrize("dtype,size", [("fp64", (65, 9)), ("fp32", (64, 5)), ("fp32", (63, 7)), ("fp64", (200, 21)),
                                        ("fp64", (230, 230)), ("fp32", (370, 360))])
@pytest.mark.parametrize("T,C", [(1, 1), (4, 1), (5, 2), (7, 3), (8, 4), (6, 6)])
def test_backward_is_the_chain_of_its_steps(dtype, size, T, C):
    nx, ny = size
    ld = torch.from_numpy(inputs.logda_field(max(nx, ny), seed=3)[:ny, :nx].copy())
    f0, g0 = (torch.from_numpy(x) for x in inputs.random_state(nx, ny, seed=7, amp=0.02, amp_T=0.1))
    cav = P.Cavity(nx, ny, dtype=dtype, logda=ld, **KW)
    cav.set_populations(f0, g0)
    adj = P.Adjoint(cav, T, C)
    adj.forward()
    gl, gn, gRa = adj.backward()
    adj.close()
    cav.set_populations(f0, g0)
    cl, cn, cRa = chain(cav, T)
    # the states of the chain went through f = w + df in FP64 and back: 6e-17 on
    # populations whose non-equilibrium part is about 1e-3, and up to 8 steps
    assert (gl - cl).abs().max() <= 1e-11 * cl.abs().max()
    assert gn == pytest.approx(cn, rel=1e-9)
    assert gRa == pytest.approx(cRa, rel=1e-9)
