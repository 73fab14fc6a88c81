"""The tiled and the brick update where their tiles, segments, bricks and wave
roles meet an edge: rows narrower than a tile or a brick, one or two columns
past one, rows of whole cache lines and not; segments of a single plane (only
their two halo planes and one output plane) and of several; walls and ghost
faces on x.  Small grids run the brick kernel, the larger ones here the tiled.

One step from a state that is representable in the storage format, against
the oracle's FP64 step rounded to storage.  Bar: one storage ulp of the
expected value (16-bit storage) plus 16 binary32 ulps of the largest
magnitude of the field (for rho - 1 also of |u|, for Pi also of |u|^2: the
terms that cancel in them).  Walls must stay at rest and ghosts hold their
neighbour's values, bit for bit."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import from_device_state, gpu_solver, oracle_grid, to_device_state

pytestmark = pytest.mark.gpu

SCALES = {0: (1.0, 1.0, 1.0), 1: (2.0 ** 12, 2.0 ** 12, 2.0 ** 16), 2: (1.0, 1.0, 1.0)}
FRAC_BITS, EMIN = {1: 10, 2: 7}, {1: -14, 2: -126}
EPS32 = float(np.finfo(np.float32).eps)
P, X, O = W.PERIODIC, W.WALL, W.OUTLET


def _scaled(st, sc):
    out = st.copy()
    out[0] = (st[0] - 1.0) * sc[0]
    out[1:4] *= sc[1]
    out[4:] *= sc[2]
    return out


def _stored(G, st, kind, sc):
    return oracle.round_storage(G, st, kind, sc) if kind else st


def _check(kind, nx, ny, nz, xface, lattice=27):
    # y walls with x walls, ghosts on z with x ghosts
    faces = {P: (P,) * 6, X: (X, X, X, X, P, P), O: (O, O, P, P, O, O) if lattice == 27 else (O, O, P, P, P, P)}[xface]
    case = W.Case("edges", nx, ny, nz, 0.61, faces=faces, force=(2e-6, 1e-6, 0.0), lattice=lattice)
    G, sc = oracle_grid(case), SCALES[kind]
    kinds = oracle.node_kinds(G)
    st0 = W.to_fp32(W.random_state(case.shape, seed=41 + nx, u_amp=0.05, pi_amp=2e-3))
    if lattice == 9:
        st0[[3, 6, 8, 9]] = 0.0
    st0 = _stored(G, st0, kind, sc)
    st0[:, kinds == 1] = W.rest_state((1,))[:, 0:1]
    s = gpu_solver(case, storage=kind)
    s.set_state(to_device_state(st0))
    start = from_device_state(s.get_state())  # ghosts refilled
    s.step(1)
    got = from_device_state(s.get_state())
    s.close()
    want = oracle.step(G, start)
    fl = kinds == 0
    w, g = _scaled(_stored(G, want, kind, sc), sc)[:, fl], _scaled(got, sc)[:, fl]
    ulp = 0.0
    if kind:
        ax = np.abs(w)
        ulp = 2.0 ** (np.maximum(np.floor(np.log2(np.where(ax > 0, ax, 1.0))), EMIN[kind]) - FRAC_BITS[kind])
    u, u2 = np.abs(want[1:4][:, fl]).max(), (want[1:4][:, fl] ** 2).sum(axis=0).max()
    size = [max(np.abs(want[0][fl] - 1.0).max(), u) * sc[0]] + [u * sc[1]] * 3 + \
        [max(np.abs(want[4:][:, fl]).max(), u2) * sc[2]] * 6
    bar = 1.0000001 * ulp + 16 * EPS32 * np.array(size)[:, None]
    assert np.all(np.abs(g - w) <= bar), float((np.abs(g - w) - bar).max())
    assert np.array_equal(got[:, kinds == 1], np.broadcast_to(W.rest_state((1,))[:, 0:1], got[:, kinds == 1].shape))
    if xface == O:
        assert np.array_equal(got[:, :, :, 0], got[:, :, :, 1]) and np.array_equal(got[:, :, :, -1], got[:, :, :, -2])


# bricks of 16 x 4 x 4: 13 rows and 5 planes are one past a brick
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("nx", [1, 3, 15, 16, 17, 33])
@pytest.mark.parametrize("xface", [P, X, O])
def test_bricks(kind, nx, xface):
    if xface != P and nx < 3:
        pytest.skip("a non-periodic axis needs 3 nodes")
    _check(kind, nx, 13, 5, xface)


# tiles of 64 x 12 (FP32: x 8), 37 rows one past a tile, segments of a few planes
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("nx", [63, 64, 65, 130])
@pytest.mark.parametrize("xface", [P, X, O])
def test_tiles(kind, nx, xface):
    _check(kind, nx, 37, 101, xface)


# 12 tile columns on 256 blocks: segments of 9, 8 and fewer planes
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("xface", [P, X, O])
def test_longer_segments(kind, xface):
    _check(kind, 66, 70, 203, xface)


# D2Q9: spans of 64 columns and segments of one row, then spans of 128 columns
# (two per lane) with segments of 16 rows (FP32) and 8
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("nx,ny", [(1, 7), (3, 5), (63, 4), (64, 33), (65, 9), (128, 12), (129, 14341), (260, 9600)])
@pytest.mark.parametrize("xface", [P, X, O])
def test_d2q9_spans(kind, nx, ny, xface):
    if xface != P and nx < 3:
        pytest.skip("a non-periodic axis needs 3 nodes")
    _check(kind, nx, ny, 1, xface, lattice=9)


@pytest.mark.parametrize("lattice,order", [(19, 3), (27, 2), (19, 2)])
@pytest.mark.parametrize("dims", [(17, 13, 9), (66, 37, 101)])
def test_other_lattice_and_order(lattice, order, dims):
    """Force field and walls with D3Q19 and order 2."""
    faces = (P, P, X, X, X, X)
    case = W.Case("lat", *dims, 0.61, faces=faces, lattice=lattice, order=order)
    G = oracle_grid(case)
    kinds = oracle.node_kinds(G)
    st0 = W.to_fp32(W.random_state(case.shape, seed=7, u_amp=0.05, pi_amp=2e-3))
    st0[:, kinds == 1] = W.rest_state((1,))[:, 0:1]
    g = W.random_force(case.shape, seed=8, amp=2e-6).astype(np.float32).astype(np.float64)
    s = gpu_solver(case)
    s.set_force_field(g)
    s.set_state(to_device_state(st0))
    s.step(1)
    got, want = from_device_state(s.get_state()), oracle.step(G, st0, g)
    s.close()
    fl = kinds == 0
    u, u2 = np.abs(want[1:4][:, fl]).max(), (want[1:4][:, fl] ** 2).sum(axis=0).max()
    size = [max(np.abs(want[0][fl] - 1.0).max(), u)] + [u] * 3 + [max(np.abs(want[4:][:, fl]).max(), u2)] * 6
    assert np.all(np.abs(got - want)[:, fl] <= 16 * EPS32 * np.array(size)[:, None])


# tiles of 64 x 12: 37 rows one past a tile
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("nx", [64, 65])
@pytest.mark.parametrize("xface", [P, X, O])
def test_larger_tiles(kind, nx, xface):
    _check(kind, nx, 37, 607, xface)


# FP32 levels larger than the Infinity Cache (268 MB): non-temporal stores and
# loads two planes ahead, segments of odd and even length
@pytest.mark.parametrize("xface", [P, X, O])
def test_streamed_tiles(xface):
    _check(0, 64, 130, 413, xface)


# tiles of 64 x 13 (16-bit levels larger than the Infinity Cache, 270 MB): 40
# rows one past a tile
@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("xface", [P, X])
def test_thirteen_row_tiles(kind, xface):
    _check(kind, 65, 40, 2600, xface)


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("dims", [(1, 13, 5), (63, 12, 9), (64, 25, 4), (130, 37, 101), (66, 70, 203), (65, 37, 607)])
@pytest.mark.parametrize("xface", [P, X, O])
def test_adjoint(dims, field, xface):
    """One adjoint step where tiles, segments and roles meet an edge, with and
    without a force field and its gradient.  Every result is a sum of at most
    a few hundred products of values of the same size: 64 binary32 ulps of
    the largest."""
    import torch
    if xface != P and min(dims) < 3:
        pytest.skip("a non-periodic axis needs 3 nodes")
    faces = {P: (P,) * 6, X: (X, X, X, X, P, P), O: (O, O, P, P, O, O)}[xface]
    case = W.Case("adj", *dims, 0.62, faces=faces, force=(2e-6, 1e-6, 0.0))
    G = oracle_grid(case)
    st0 = W.random_state(case.shape, seed=51, u_amp=0.05, pi_amp=2e-3)
    st0 = W.to_fp32(oracle.ghost_fill(G, st0, 0) if xface == O else st0)
    g = W.random_force(case.shape, seed=52, amp=1e-4).astype(np.float32).astype(np.float64) if field else None
    lam1 = np.random.default_rng(53).standard_normal(st0.shape).astype(np.float32).astype(np.float64)
    if xface != O:
        lam1[:, oracle.node_kinds(G) != 0] = 0.0
    s = gpu_solver(case)
    if field:
        s.set_force_field(g)
    s.set_state(to_device_state(st0))
    raw0 = s.save_raw()
    s.step(1)
    raw1 = s.save_raw()
    dg = torch.zeros((3,) + case.shape, dtype=torch.float32, device="cuda") if field else None
    lam0 = s.adjoint_step(raw0, raw1, torch.tensor(lam1, dtype=torch.float32, device="cuda"), dg)
    lam0 = lam0.double().cpu().numpy()
    s.close()
    want, want_dg = oracle.adjoint_step(G, st0, lam1, g)
    assert np.abs(lam0 - want).max() <= 64 * EPS32 * np.abs(want).max()
    if field:
        assert np.abs(dg.double().cpu().numpy() - want_dg).max() <= 64 * EPS32 * np.abs(want_dg).max()
