"""Narrow grids, whose bricks or tiles are mostly empty, at sizes beyond what
one launch of the brick kernel takes: they step, as the same state on a small
grid does."""
import pytest

import workloads as W
from helpers import gpu_solver, to_device_state

pytestmark = pytest.mark.gpu


def _step(nz, st):
    import torch
    s = gpu_solver(W.Case("narrow", st.shape[3], st.shape[2], nz, 0.62, force=(2e-6, 1e-6, 0.0)))
    s.set_state(st.repeat(1, nz // st.shape[1], 1, 1))
    s.step(1)
    out = s.get_state()
    s.close()
    torch.cuda.empty_cache()
    return out


@pytest.mark.parametrize("nx,nz", [(1, 24_800_000), (3, 1 << 20)])
def test_narrow_grid_steps(nx, nz):
    import torch
    st = torch.from_numpy(to_device_state(W.random_state((8, 1, nx), seed=71))).cuda()
    one, many = _step(8, st), _step(nz, st)
    assert torch.equal(many.view(10, nz // 8, 8, 1, nx), one.unsqueeze(1).expand(-1, nz // 8, -1, -1, -1))
