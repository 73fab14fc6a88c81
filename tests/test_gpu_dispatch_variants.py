"""Kernels that the choices of the update and the adjoint lead to only on some
grids, one step each against the oracle, with the bars and inputs of
test_gpu_tiled_edges."""
import pytest

import workloads as W
from test_gpu_tiled_edges import _check

pytestmark = pytest.mark.gpu

P, X, O = W.PERIODIC, W.WALL, W.OUTLET


# D2Q9: one column per lane on segments of many rows (one, three and five
# spans), two columns per lane on two, six and nine halves, the last empty or
# not, with segments that FP32 doubles (r2 <= 16) or not; up to four rows
# uncut, with one column per lane and with two
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("nx,ny", [(3, 20000), (64, 40000), (130, 20000), (256, 14400), (384, 13000), (570, 8000), (256, 35000),
                                   (65600, 3), (66000, 4), (524300, 3)])
@pytest.mark.parametrize("xface", [P, X, O])
def test_d2q9(kind, nx, ny, xface):
    if xface != P and nx * ny > 4_000_000:
        pytest.skip("walls and ghosts on the smaller grids")
    _check(kind, nx, ny, 1, xface, lattice=9)
