"""GPU: cells at the ends of what the parameters allow, in the forward update and
the adjoint."""
import numpy as np
import pytest
import torch

import paper_2011_15073_amd as P
from paper_2011_15073_amd import inputs
from pairs import gpu_for, oracle_for
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


@pytest.mark.parametrize("n", [0.6, 1.0, 1.4])
@pytest.mark.parametrize("step_kernel", ["auto", "single"])
def test_solid_cells_match_the_oracle(n, step_kernel):
    """Cells whose resistance, squared, is around or beyond the largest FP64 number
    stand still: |u| < |v| / 1e153, and 0 beyond."""
    nx, ny = 70, 19
    ld, solid = plane(nx, ny, [-160.0, -200.0, -290.0])
    kw = dict(n=n, Ra=1e4, **PHYS)
    cav = gpu_for(nx, ny, logda=torch.from_numpy(ld), step_kernel=step_kernel, **kw)
    orc = oracle_for(nx, ny, logda=ld, **kw)
    f0, g0 = inputs.random_state(nx, ny, seed=7, amp=0.02, amp_T=0.1)
    cav.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    orc.set_state(f0, g0)
    for k in (1, 4):
        cav.step(k)
        orc.step(k)
        for a, b in zip(cav.populations(), orc.state()):
            assert np.abs(a.cpu().numpy() - b).max() <= 1e-13
    U = np.abs(cav.fields()[0].cpu().numpy())
    assert U[solid].max() <= 1e-150 and U[ld <= -200.0].max() == 0.0


def test_solid_scalar_darcy_number_matches_the_oracle():
    kw = dict(n=0.8, Da=1e-200, Ra=1e4, **PHYS)
    cav, orc = gpu_for(20, **kw).step(7), oracle_for(20, **kw).step(7)
    for a, b in zip(cav.populations(), orc.state()):
        assert np.abs(a.cpu().numpy() - b).max() <= 1e-13


@pytest.mark.parametrize("n", [0.7, 1.0, 1.4])
def test_adjoint_step_with_solid_cells(n):
    """Against a central difference of the oracle's step in a random direction.
    On a plane without such cells the same difference is within 3e-10 |lambda| of
    autograd's derivative (h = 1e-7: as much truncation as rounding)."""
    nx, ny = 21, 13
    ld, _ = plane(nx, ny, [-160.0, -200.0, -290.0])
    rng = np.random.default_rng(5)
    lam, d = rng.standard_normal((14, ny, nx)), rng.standard_normal((14, ny, nx))
    f0, g0 = inputs.random_state(nx, ny, seed=7, amp=0.03, amp_T=0.2)
    kw = dict(n=n, Ra=1e4, **PHYS)
    cav = gpu_for(nx, ny, logda=torch.from_numpy(ld), **kw)
    cav.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    lam_g, gld, gn, gRa = P.vjp_step(cav, torch.from_numpy(lam))
    lam_g = lam_g.cpu().numpy()

    def L(h):
        orc = oracle_for(nx, ny, logda=ld, **kw)
        orc.set_state(f0 + h * d[:9], g0 + h * d[9:])
        return (lam * np.concatenate(orc.step(1).state())).sum()

    fd = (L(1e-7) - L(-1e-7)) / 2e-7
    assert (lam_g * d).sum() == pytest.approx(fd, abs=1e-8 * np.linalg.norm(lam_g))
    assert np.isfinite(gld.cpu().numpy()).all() and np.isfinite([gn, gRa]).all()


FORCES = [1e-152, 1e-153, 1e-154, 1e-155, 1e-156, 1e-157, 1e-158, 1e-160]


@pytest.mark.parametrize("n", [0.6, 1.4])
@pytest.mark.parametrize("step_kernel", ["auto", "single"])
def test_viscosity_at_subnormal_shear(n, step_kernel):
    """A cavity at rest but for a uniform force of 1e-152 .. 1e-160: away from the
    heated walls the shear rate squared runs through the subnormal numbers, and
    the viscosity is the oracle's, the bound that weak shear lands on (FP32
    start of the FP64 solve: 2^-24 of log2 nu <= 10)."""
    for gx in FORCES:
        kw = dict(n=n, Da=1e-2, Ra=1e5, gx=gx, **PHYS)
        cav = gpu_for(64, 24, step_kernel=step_kernel, **kw).step(6)
        ref = oracle_for(64, 24, **kw).step(6).macros()["nu"][:, 8:56]
        nu = cav.viscosity().cpu().numpy()[:, 8:56]
        assert np.abs(nu / ref - 1).max() <= 1e-6, gx


def forced(nx, ny, n, gx, steps):
    """A cavity without body force in the state of one with the force gx after
    `steps` steps from rest (the adjoint takes no body force): its saved state
    behind the header of the other's, 256 bytes with the physics' hash."""
    kw = dict(n=n, Da=1e-2, Ra=1e5, **PHYS)
    cav = gpu_for(nx, ny, **kw).step(steps)
    buf = cav.save_state()
    buf[256:] = gpu_for(nx, ny, gx=gx, **kw).step(steps).save_state()[256:]
    cav.load_state(buf)
    return cav


@pytest.mark.parametrize("n", [0.6, 1.0, 1.4])
def test_adjoint_step_at_subnormal_shear(n):
    """The same states: the adjoint step differs from that of the state without
    the force by about the force's size, so not at all in FP64."""
    lam = torch.from_numpy(1e3 * np.random.default_rng(2).standard_normal((14, 24, 64)))
    out = [P.vjp_step(forced(64, 24, n, gx, 6), lam) for gx in [0.0] + FORCES]
    for gx, (l, _, gn, gRa) in zip(FORCES, out[1:]):
        assert np.isfinite(gn), gx
        assert (l - out[0][0]).abs().max() <= 1e-12 * out[0][0].abs().max(), gx
        assert gRa == pytest.approx(out[0][3], rel=1e-12), gx


def test_adjoint_step_at_subnormal_shear_next_to_newtonian():
    """n = 1 + 1e-9 has its root between the bounds at any shear: next to n = 1
    (viscosity and gradients within 1e-9 times the 1000 octaves of the shear)."""
    lam = torch.from_numpy(1e3 * np.random.default_rng(2).standard_normal((14, 4, 64)))
    for gx in FORCES[1:5]:
        a, b = (P.vjp_step(forced(64, 4, n, gx, 6), lam) for n in (1.0 + 1e-9, 1.0))
        assert (a[0] - b[0]).abs().max() <= 1e-5 * b[0].abs().max(), gx
        assert a[2] == pytest.approx(b[2], rel=1e-5) and a[3] == pytest.approx(b[3], rel=1e-5), gx
