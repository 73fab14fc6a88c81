"""Kernels that the choices of the update and the adjoint lead to only on some
grids, one step each against the oracle, with the bars and inputs of
test_gpu_tiled_edges."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import from_device_state, gpu_solver, oracle_grid, to_device_state
from test_gpu_tiled_edges import EMIN, EPS32, FRAC_BITS, SCALES, _check, _scaled, _stored, test_adjoint as _adjoint_check

pytestmark = pytest.mark.gpu

P, X, O = W.PERIODIC, W.WALL, W.OUTLET


def _check_more(kind, dims, faces, order=3, lattice=27, field=False):
    """_check for any order, lattice, faces and a force field."""
    case = W.Case("variant", *dims, 0.61, faces=faces, force=(2e-6, 1e-6, 0.0), order=order, lattice=lattice)
    G, sc = oracle_grid(case), SCALES[kind]
    kinds = oracle.node_kinds(G)
    st0 = _stored(G, W.to_fp32(W.random_state(case.shape, seed=91, u_amp=0.05, pi_amp=2e-3)), kind, sc)
    st0[:, kinds == 1] = W.rest_state((1,))[:, 0:1]
    g = W.random_force(case.shape, seed=92, amp=1e-5).astype(np.float32).astype(np.float64) if field else None
    s = gpu_solver(case, storage=kind)
    if field:
        s.set_force_field(g)
    s.set_state(to_device_state(st0))
    start = from_device_state(s.get_state())  # ghosts refilled
    s.step(1)
    got = from_device_state(s.get_state())
    s.close()
    want = oracle.step(G, start, g)
    fl = kinds == 0
    w, v = _scaled(_stored(G, want, kind, sc), sc)[:, fl], _scaled(got, sc)[:, fl]
    ulp = 0.0
    if kind:
        ax = np.abs(w)
        ulp = 2.0 ** (np.maximum(np.floor(np.log2(np.where(ax > 0, ax, 1.0))), EMIN[kind]) - FRAC_BITS[kind])
    u, u2 = np.abs(want[1:4][:, fl]).max(), (want[1:4][:, fl] ** 2).sum(axis=0).max()
    size = [max(np.abs(want[0][fl] - 1.0).max(), u) * sc[0]] + [u * sc[1]] * 3 + \
        [max(np.abs(want[4:][:, fl]).max(), u2) * sc[2]] * 6
    bar = 1.0000001 * ulp + 16 * EPS32 * np.array(size)[:, None]
    assert np.all(np.abs(v - w) <= bar), float((np.abs(v - w) - bar).max())


PER, WALLS, GHOSTS = (P,) * 6, (P, P, X, X, X, X), (O,) * 6


# FP32 tiles of 12 rows with loads two planes ahead (275 MB in two levels), and
# of 8 rows (287 MB)
@pytest.mark.parametrize("dims", [(64, 130, 413), (64, 8, 7000)])
@pytest.mark.parametrize("faces,order,lattice,field", [(WALLS, 3, 27, True), (PER, 3, 19, False), (WALLS, 3, 19, True),
                                                       (PER, 2, 27, True), (WALLS, 2, 19, False), (GHOSTS, 2, 27, False),
                                                       (GHOSTS, 3, 27, True)])
def test_streamed(dims, faces, order, lattice, field):
    _check_more(0, dims, faces, order, lattice, field)


# 16-bit tiles of 13 rows (39 rows are 3 of them, 4 of 12) whose levels exceed
# the Infinity Cache, rows of whole lines (non-temporal stores, ghosts on x
# written by the update) and not
@pytest.mark.parametrize("kind,nx", [(1, 64), (2, 65)])
@pytest.mark.parametrize("faces,order,lattice,field", [(PER, 3, 27, False), (WALLS, 3, 27, True), (GHOSTS, 3, 27, False),
                                                       (PER, 3, 19, True), (GHOSTS, 2, 27, False)])
def test_thirteen_rows(kind, nx, faces, order, lattice, field):
    _check_more(kind, (nx, 39, 2750), faces, order, lattice, field)


# 16-bit tiles of 12 rows that share cache lines: loads with the exchange, a
# plane ahead with a force field
@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("faces,order,lattice,field", [(PER, 3, 27, False), (WALLS, 3, 27, False), (GHOSTS, 3, 19, False),
                                                       (PER, 2, 27, False), (PER, 3, 27, True)])
def test_late_loads(kind, faces, order, lattice, field):
    _check_more(kind, (70, 37, 203), faces, order, lattice, field)


# adjoint in tiles of 12 rows, of whole cache lines (non-temporal stores)
@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("xface", [P, X, O])
def test_adjoint_of_whole_lines(field, xface):
    _adjoint_check((64, 37, 607), field, xface)


@pytest.mark.parametrize("dims", [(33, 17, 9), (32, 16, 9), (101, 97, 91)])
def test_rollout_checkpoints(dims):
    """The checkpoints of a rollout are the states themselves: sizes of no
    multiple of 16 bytes, and beyond 32 MB."""
    import torch
    from paper_2401_17074_amd import _binding as C
    case = W.Case("ckpt", *dims, 0.7, force=(1e-5, 0.0, 0.0))
    s = gpu_solver(case)
    s.set_state(to_device_state(W.random_state(case.shape, seed=93)))
    ws = torch.zeros(C.tslb_rollout_workspace_bytes(s.h, 5, 2), dtype=torch.uint8, device="cuda")
    levels = [s.save_raw()]
    for _ in range(2):
        s.step(2)
        levels.append(s.save_raw())
    s.load_raw(levels[0])
    C.tslb_rollout_forward(s.h, 5, 2, ws)
    n = s.state_bytes()
    for k, want in enumerate(levels):
        assert torch.equal(ws[k * n:(k + 1) * n], want), k
    # an odd number of adjoint steps: the result is copied out of the workspace
    lam = torch.randn((10,) + case.shape, device="cuda")
    s.load_raw(levels[2])
    states = [levels[2]]
    s.step(1)
    states.append(s.save_raw())
    want = s.adjoint_step(states[0], states[1], lam.clone())
    s.load_raw(levels[2])
    C.tslb_rollout_forward(s.h, 1, 2, ws)
    C.tslb_rollout_backward(s.h, 1, 2, ws, lam, None)
    s.close()
    assert torch.equal(lam, want)


# D2Q9: one column per lane on segments of many rows (one, three and five
# spans), two columns per lane on two, six and nine halves, the last empty or
# not, with segments that FP32 doubles (r2 <= 16) or not; up to four rows
# uncut, with one column per lane and with two
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("nx,ny", [(3, 20000), (64, 40000), (130, 20000), (256, 14400), (384, 13000), (570, 8000), (256, 34900),
                                   (65600, 3), (66000, 4), (524300, 3)])
@pytest.mark.parametrize("xface", [P, X, O])
def test_d2q9(kind, nx, ny, xface):
    if xface != P and nx * ny > 4_000_000:
        pytest.skip("walls and ghosts on the smaller grids")
    _check(kind, nx, ny, 1, xface, lattice=9)
