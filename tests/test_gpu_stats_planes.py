"""Plane profiles where a block's nodes, its remainders of four and the runs of
planes per XCD meet an edge, against FP64 sums of the stored velocities; and
more planes than a launch of one wavefront each takes."""
import numpy as np
import pytest

import workloads as W
from helpers import gpu_solver, to_device_state

pytestmark = pytest.mark.gpu

P, X, O = W.PERIODIC, W.WALL, W.OUTLET


# planes along y of nx x nz nodes in one block: 1 to 5 and 7 nodes per thread,
# with and without a rest; several blocks per plane; along x fewer, as many and
# more planes than XCDs, in one block per plane and in several
@pytest.mark.parametrize("dims,axis", [((255, 5, 1), 1), ((16, 5, 32), 1), ((64, 6, 12), 1), ((33, 3, 31), 1), ((40, 4, 32), 1),
                                       ((60, 3, 30), 1), ((150, 3, 150), 1), ((7, 40, 5), 0), ((8, 100, 3), 0), ((9, 64, 20), 0),
                                       ((333, 41, 3), 0), ((17, 90, 60), 0), ((3, 5, 70), 2), ((130, 70, 3), 2)])
@pytest.mark.parametrize("bc", ["periodic", "walls"])
def test_profile_sums(dims, axis, bc):
    faces = (P,) * 6 if bc == "periodic" else tuple(f for n in dims for f in ((X, X) if n >= 3 else (P, P)))
    case = W.Case("planes", *dims, 0.6, faces=faces)
    st = to_device_state(W.random_state(case.shape, seed=81))
    s = gpu_solver(case)
    s.set_state(st)
    s.stats_begin(profile_axis=axis)
    s.stats_sample()
    s.stats_sample()
    rows, ns = s.stats_profile()
    s.close()
    fluid = np.ones(case.shape, bool)
    for d in range(3):
        if faces[2 * d] == X:
            ax = np.moveaxis(fluid, 2 - d, 0)
            ax[0] = ax[-1] = False
    u = st[1:4].astype(np.float64)
    terms = [np.ones(case.shape)] + [u[a] for a in range(3)] + [u[a] * u[b] for a, b in
                                                                ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))] + [u[a] ** 3 for a in range(3)]
    over = tuple(a for a in range(3) if a != 2 - axis)
    want = 2 * np.stack([(t * fluid).sum(over) for t in terms], 1)
    size = 2 * np.stack([(np.abs(t) * fluid).sum(over) for t in terms], 1)
    # at most 2e4 terms of a plane, each sum's rounding within half their number of ulps of the magnitudes
    assert ns == 2 and rows.shape == want.shape
    assert np.all(np.abs(rows.numpy() - want) <= 2e4 * 2.0 ** -53 * size)


def test_more_planes_than_wavefronts_of_a_launch():
    """68 million planes of one node: 2^32 threads at a wavefront each."""
    import torch
    n = 68_000_000
    s = gpu_solver(W.Case("line", 1, 1, n, 0.6))
    st = torch.zeros((10, n, 1, 1), device="cuda")
    st[1, :, 0, 0] = torch.arange(n, device="cuda") % 1024 / 2 ** 16
    s.set_state(st)
    del st
    s.stats_begin(profile_axis=2)
    s.stats_sample()
    rows, ns = s.stats_profile()
    s.close()
    torch.cuda.empty_cache()
    assert ns == 1 and bool((rows[:, 0] == 1.0).all())
    assert torch.equal(rows[:, 1], (torch.arange(n, dtype=torch.float64) % 1024) / 2 ** 16)
