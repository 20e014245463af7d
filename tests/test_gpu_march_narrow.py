"""GPU: the multi-step pass on grids of few strips, where its workgroups take 1, 2,
3 or 4 of them.  Narrow tall FP32 grids must take the pass (they took two steps
per pass before it, and lost a quarter to a third of their speed without), and the
populations must be those of single steps bit for bit for every number of strips."""
import pytest

import paper_2011_15073_amd as P
from test_gpu_march import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(64, 226000), (250, 58000), (500, 29000), (640, 22700)])
@pytest.mark.parametrize("n", [0.8, 1.0])
def test_narrow_tall_grids_take_the_pass(size, n):
    need = [P.workspace_bytes(P.make_params(*size, dtype="fp32", step_kernel=s, n=n)) for s in ("auto", "single")]
    assert need[0] > need[1]


# strips of 64 columns 58 apart: 64 + 58 k columns make k + 1 of them
@pytest.mark.parametrize("strips", [1, 2, 3, 4, 5, 6, 7, 9, 10, 13, 17])
@pytest.mark.parametrize("n,logda,rounding", [(0.8, True, "auto"), (1.0, False, "nearest")])
def test_every_number_of_strips_equals_single_steps(strips, n, logda, rounding):
    for nx in (64 + 58 * (strips - 1), 64 + 58 * (strips - 1) - 57):
        compare((nx, 41), "fp32", "pair", (6, 5, 13), n, logda, rounding)


@pytest.mark.parametrize("n,logda", [(0.8, True), (1.0, False)])
def test_a_narrow_grid_equals_single_steps(n, logda):
    compare((251, 23003), "fp32", "auto", (6, 13), n, logda, "auto")
