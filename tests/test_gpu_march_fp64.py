"""GPU: the multi-step pass on automatically chosen grids in the variants that the
small grids of PM_STEP_PAIR (FP32) do not reach: FP64 with and without a per-cell
log10 Da plane, power law and Newtonian, with one column more or less than a whole
number of strips and one row more or less than a workgroup's, and FP32 with the
default rounding and a plane.  All bit for bit the single steps' populations."""
import pytest

import paper_2011_15073_amd as P
from test_gpu_march import compare

pytestmark = pytest.mark.gpu


# FP64 strips are 64 columns, 60 apart; at n = 1 the pass starts at 12 strips and 1.6 M nodes
@pytest.mark.parametrize("nx", [724, 725, 843, 844, 845, 905])
@pytest.mark.parametrize("ny,logda", [(2211, True), (2212, False), (2213, True)])
def test_fp64_newtonian(nx, ny, logda):
    assert P.workspace_bytes(P.make_params(nx, ny, dtype="fp64")) > P.workspace_bytes(
        P.make_params(nx, ny, dtype="fp64", step_kernel="single"))
    compare((nx, ny), "fp64", "auto", (4, 5, 7), 1.0, logda, "nearest")


@pytest.mark.parametrize("size,logda", [((3001, 2701), True), ((2704, 3000), True), ((844, 9501), False)])
def test_fp64_power_law(size, logda):
    compare(size, "fp64", "auto", (4, 5), 0.7, logda, "nearest")


@pytest.mark.parametrize("size,n,logda", [((2503, 2201), 0.8, True), ((2503, 2201), 1.4, False), ((1109, 1087), 1.0, True)])
def test_fp32_with_the_default_rounding(size, n, logda):
    compare(size, "fp32", "auto", (6, 5, 13), n, logda, "auto")
