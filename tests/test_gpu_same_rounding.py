"""A node's update does not depend on the kernel, tile height or brick that
does it: every D3Q27 population is evaluated in the same form on any grid.

A state repeated along a periodic z axis stays repeated, bit for bit, so a
small grid (bricks, tiles of 8 rows; 16-bit storage: 12 rows) is compared with
many copies of it stacked along z, which are updated in tiles of 12 rows
(16-bit storage: 13).  The FP64 loss of checkpointed rollouts on small grids
is compared with values recorded from tiles of 12 rows."""
import json
import os

import numpy as np
import pytest

import workloads as W
from helpers import gpu_solver, to_device_state

pytestmark = pytest.mark.gpu

P, X, O = W.PERIODIC, W.WALL, W.OUTLET
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "rollout_loss_rows12.json")


def _stepped(case, st, g, copies, kind):
    import torch
    big = W.Case(case.name, case.nx, case.ny, case.nz * copies, case.tau, faces=case.faces, force=case.force,
                 order=case.order, lattice=case.lattice)
    s = gpu_solver(big, storage=kind)
    s.set_state(torch.from_numpy(st).cuda().repeat(1, copies, 1, 1))
    if g is not None:
        s.set_force_field(torch.from_numpy(g).cuda().repeat(1, copies, 1, 1))
    s.step(3)
    out = s.get_state()
    s.close()
    return out


def _check(dims, copies, faces, kind=0, order=3, lattice=27, field=False):
    import torch
    case = W.Case("same", *dims, 0.62, faces=faces + (P, P), force=(2e-6, 1e-6, 0.0), order=order, lattice=lattice)
    st = to_device_state(W.random_state(case.shape, seed=61, u_amp=0.05, pi_amp=2e-3))
    g = W.random_force(case.shape, seed=62, amp=1e-5).astype(np.float32) if field else None
    one, many = _stepped(case, st, g, 1, kind), _stepped(case, st, g, copies, kind)
    assert torch.equal(one, many[:, :dims[2]])
    assert torch.equal(many, one.repeat(1, copies, 1, 1))


XY = {"periodic": (P,) * 4, "walls_y": (P, P, X, X), "walls_xy": (X,) * 4, "ghosts": (O,) * 4}


# bricks: 32^3, 40^3, 17 x 90 (two bricks wide); 8 rows: 64^3, 130 x 37
@pytest.mark.parametrize("dims,copies", [((32, 32, 32), 64), ((40, 40, 40), 50), ((17, 90, 16), 80),
                                         ((64, 64, 64), 16), ((130, 37, 50), 30)])
@pytest.mark.parametrize("faces", sorted(XY))
def test_small_grids_as_tiles_of_12_rows(dims, copies, faces):
    _check(dims, copies, XY[faces])


@pytest.mark.parametrize("dims,copies", [((40, 40, 40), 50), ((130, 37, 50), 30)])
@pytest.mark.parametrize("order,lattice", [(2, 27), (3, 19), (2, 19)])
def test_other_orders_and_lattice(dims, copies, order, lattice):
    _check(dims, copies, XY["walls_y"], order=order, lattice=lattice, field=True)


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("nx", [64, 65])
@pytest.mark.parametrize("faces", sorted(XY))
def test_16_bit_tiles_of_13_rows_as_12(kind, nx, faces):
    _check((nx, 39, 26), 104, XY[faces], kind=kind)


def rollout_loss(dims, steps, every):
    """Kinetic energy after `steps` steps of a box at tau 0.8 under a force field."""
    import torch
    from paper_2401_17074_amd import Solver, TslbRollout
    nx, ny, nz = dims
    shape = (nz, ny, nx)
    s = Solver(nx, ny, nz, 0.8)
    u0 = W.random_state(shape, seed=63, u_amp=0.02)[1:4].astype(np.float32)
    g = W.random_force(shape, seed=64, amp=1e-6).astype(np.float32)
    loss = TslbRollout.apply(torch.from_numpy(g).cuda(), torch.from_numpy(u0).cuda(), s, steps, every)
    s.close()
    return float(loss)


def test_rollout_loss_as_recorded():
    """The loss is a sum of positive FP64 terms: only the order of its at most
    5e5 additions is free, a few thousand in a chain and rounding up and down
    alike: 1e-12."""
    for rec in json.load(open(GOLDEN)):
        got, want = rollout_loss(rec["dims"], rec["steps"], rec["every"]), float.fromhex(rec["loss"])
        print(rec["dims"], got.hex(), rec["loss"], flush=True)
        assert abs(got - want) <= 1e-12 * want, (rec["dims"], got, want)


if __name__ == "__main__":  # PYTHONPATH=<tree of the library to record from> python ...
    recs = [{"dims": d, "steps": n, "every": e, "loss": rollout_loss(d, n, e).hex()}
            for d, n, e in (((32, 32, 32), 30, 10), ((40, 40, 40), 20, 7), ((64, 64, 64), 40, 20), ((77, 33, 64), 30, 10),
                            ((24, 90, 70), 20, 10))]
    with open(GOLDEN, "w") as f:
        f.write("[" + ",\n ".join(json.dumps(r) for r in recs) + "]\n")
