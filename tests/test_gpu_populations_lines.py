"""GPU: pm_get_populations where a row of the output is whole 128-byte lines (its
stores go past the caches) and where it is not, and into buffers that begin
inside a line: the same values, and nothing outside the buffers."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2011_15073_amd as P
from paper_2011_15073_amd import inputs
from pairs import gpu_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [16, 31, 32, 33, 64, 96, 257])
@pytest.mark.parametrize("dtype,out", [("fp64", torch.float64), ("fp32", torch.float64), ("fp32", torch.float32),
                                       ("fp16", torch.float32)])
@pytest.mark.parametrize("steps", [0, 1])
def test_values_do_not_depend_on_lines(nx, dtype, out, steps):
    ny = 9
    cav = gpu_for(nx, ny, dtype=dtype, n=0.8, Da=1e-2, Ra=1e5, Pr=10.0, eps=0.6, rounding="nearest")
    f0, g0 = inputs.random_state(nx, ny, seed=4, amp=0.02, amp_T=0.1)
    cav.set_populations(torch.from_numpy(f0), torch.from_numpy(g0))
    cav.step(steps)
    f, g = cav.populations(out)  # torch's buffers begin at a line
    if steps == 0:
        e = {"fp64": 2e-16, "fp32": 6e-8, "fp16": 1e-3}[dtype]  # one rounding of values below 1
        assert np.abs(f.cpu().numpy() - f0).max() <= e and np.abs(g.cpu().numpy() - g0).max() <= e
    n = 14 * nx * ny
    for shift in (1, 8):
        buf = torch.full((n + 64,), -7.0, dtype=out, device="cuda")
        code = P.PM_FP64 if out == torch.float64 else P.PM_FP32
        at = buf.data_ptr() + shift * buf.element_size()
        cav._check(P._lib.lib.pm_get_populations(cav._h, C.c_void_p(at), C.c_void_p(at + 9 * nx * ny * buf.element_size()),
                                                 code))
        assert torch.equal(buf[shift:shift + n], torch.cat([f.flatten(), g.flatten()]))
        assert (buf[:shift] == -7.0).all() and (buf[shift + n:] == -7.0).all()
