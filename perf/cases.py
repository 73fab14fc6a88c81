"""The work a user of this library has it do, as cases whose passes can be timed and checked.

A case is a dict of plain values.  Its "kind" says which public entry points a pass goes through:

  loop      the main loop of a simulation: Solver.step(steps) on a handle whose state buffers are PyTorch
            tensors (bind_state_to_torch); the state after the steps is read in place
  run       a whole small run on new fields: set_state, step(steps), get_state
  grad      a gradient: TslbRollout forward and backward (checkpointed rollout and discrete adjoint)
  adjoint   one discrete adjoint step (Solver.adjoint_step), as a program with its own checkpointing calls it
  stats     monitoring: stats_sample, the sums read back, the conservation check (reduce); with "field" the
            per-node sums, their moments and the jet diagnostics as well

Boundary kinds ("bc"): "periodic"; "channel" (walls on y, forced along x); "duct" (walls on y and z, forced along x);
"jet" (inlet disc on x = 0, outflow elsewhere); "zjet" (inlet disc on z = 0 with Gaussian noise, periodic sides,
outflow on top, viscosity growing over the last planes).
"""
import math

import numpy as np
import torch

from paper_2401_17074_amd import Solver, TslbRollout

PERIODIC, WALL, INLET, OUTLET = 0, 1, 2, 3
FACES = {
    "periodic": (PERIODIC,) * 6,
    "channel": (PERIODIC, PERIODIC, WALL, WALL, PERIODIC, PERIODIC),
    "duct": (PERIODIC, PERIODIC, WALL, WALL, WALL, WALL),
    "jet": (INLET, OUTLET, OUTLET, OUTLET, OUTLET, OUTLET),
    "zjet": (PERIODIC, PERIODIC, PERIODIC, PERIODIC, INLET, OUTLET),
}
STORAGE = {"fp32": (0, torch.float32), "fp16": (1, torch.float16), "bf16": (2, torch.bfloat16)}
SCALE = {"fp32": (1.0, 1.0, 1.0), "fp16": (4096.0, 4096.0, 65536.0), "bf16": (1.0, 1.0, 1.0)}  # the library's defaults
JET_U, JET_NOISE = 0.05, 0.02
BIG_STATE = 34_000_000  # nodes of the largest drawn grid


def _case(name, kind, nx, ny, nz, bc="periodic", lattice=27, storage="fp32", order=3, tau=0.8, field=False, steps=0,
          every=0):
    return {"name": name, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "bc": bc, "lattice": lattice,
            "storage": storage, "order": order, "tau": tau, "field": field, "steps": steps, "every": every}


def listed():
    return [
        # the smallest calls: a 32^3 Taylor-Green run on new fields, where launches and latency count
        _case("run_box_32", "run", 32, 32, 32, steps=10),
        # the differentiable box's forward with its force field, one checkpoint interval
        _case("run_forced_box_64", "run", 64, 64, 64, field=True, steps=20),
        # its gradient: forward, recomputation and adjoint of two checkpoint intervals
        _case("grad_forced_box_64", "grad", 64, 64, 64, field=True, steps=40, every=20),
        # an adjoint step where bytes rather than launches bound it
        _case("adjoint_box_256", "adjoint", 256, 256, 256, field=True),
        # the ordinary channel, and the large one in single precision and with 16-bit moments
        _case("loop_channel_384x192x192", "loop", 384, 192, 192, "channel", tau=0.5045, steps=10),
        _case("loop_channel_512x256x256", "loop", 512, 256, 256, "channel", tau=0.5045, steps=4),
        _case("loop_channel_512x256x256_fp16", "loop", 512, 256, 256, "channel", tau=0.5045, storage="fp16", steps=4),
        # inflow and outflow ghost layers on every face
        _case("loop_jet_512x256x256", "loop", 512, 256, 256, "jet", tau=0.50043, steps=4),
        # the largest: the paper's jet grid, rows that are no whole cache lines, sponge, bfloat16 moments
        _case("loop_zjet_440x440x600_bf16", "loop", 440, 440, 600, "zjet", tau=0.50043, storage="bf16", steps=4),
        # the other lattices: D3Q19 on ragged sizes, D2Q9
        _case("loop_d3q19_channel_333x101x77", "loop", 333, 101, 77, "channel", lattice=19, tau=0.5045, steps=10),
        _case("loop_channel2d_8192x4096", "loop", 8192, 4096, 1, "channel", lattice=9, tau=0.5045, steps=4),
        # monitoring a channel run: plane profiles and the conservation sums
        _case("stats_channel_384x192x192", "stats", 384, 192, 192, "channel", tau=0.5045),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi, most):
    while True:
        n = [_log(rng, lo, hi) for _ in range(3)]
        if rng.random() < 0.4:  # many grids in use have sides that are multiples of 32
            n = [max(lo, 32 * round(v / 32)) for v in n]
        if n[0] * n[1] * n[2] <= most:
            return n


def draw(rng):
    pick = rng.random()
    if pick < 0.12:
        n = _grid(rng, 16, 96, 500_000)
        return _drawn("run", n, rng.choice(("periodic", "channel", "jet")), rng.choice((27, 27, 19)),
                      rng.choice(("fp32", "fp32", "fp16", "bf16")), rng, steps=rng.choice((2, 10, 20)))
    if pick < 0.62:
        n = _grid(rng, 48, 512, BIG_STATE)
        nodes = n[0] * n[1] * n[2]
        return _drawn("loop", n, rng.choice(("periodic", "channel", "channel", "duct", "jet", "zjet")),
                      rng.choice((27, 27, 27, 19)), rng.choice(("fp32", "fp32", "fp16", "bf16")), rng,
                      steps=4 if nodes > 4_000_000 else 10)
    if pick < 0.72:
        return _drawn("loop", [_log(rng, 128, 8192), _log(rng, 128, 4096), 1], rng.choice(("periodic", "channel")), 9,
                      rng.choice(("fp32", "fp32", "fp16", "bf16")), rng, steps=4)
    if pick < 0.81:
        return _drawn("grad", _grid(rng, 24, 96, 500_000), "periodic", 27, "fp32", rng, steps=rng.choice((20, 30, 40)),
                      every=rng.choice((7, 10, 20)))
    if pick < 0.90:
        return _drawn("adjoint", _grid(rng, 48, 288, 17_000_000), rng.choice(("periodic", "channel")), 27, "fp32", rng)
    bc = rng.choice(("channel", "zjet"))
    return _drawn("stats", _grid(rng, 64, 448, 16_000_000), bc, 27, rng.choice(("fp32", "fp32", "fp16")), rng)


def _drawn(kind, n, bc, lattice, storage, rng, steps=0, every=0):
    c = _case("", kind, n[0], n[1], n[2], bc, lattice, storage, steps=steps, every=every,
              tau=0.50043 if bc in ("jet", "zjet") else rng.choice((0.5045, 0.8)))
    del c["name"]
    c["order"] = 2 if kind in ("run", "loop") and rng.random() < 0.15 else 3
    c["field"] = kind in ("grad", "adjoint") or (kind == "stats" and bc == "zjet") or (
        kind in ("run", "loop") and bc in ("periodic", "channel") and rng.random() < 0.2)
    return c


# ------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _noise(shape, amp, gen):
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-amp, amp, generator=gen)


def _force(case):
    if case["bc"] in ("channel", "duct"):  # friction Reynolds number 180 across the half-width
        nu, h = (case["tau"] - 0.5) / 3.0, (case["ny"] - 2) / 2.0
        return (float(np.float32(min(1e-4, (180.0 * nu / h) ** 2 / h))), 0.0, 0.0)
    return (0.0, 0.0, 0.0)


def _center(case):
    n = (case["nx"], case["ny"], case["nz"])
    a = (1, 2) if case["bc"] == "jet" else (0, 1)
    return ((n[a[0]] - 1) / 2.0, (n[a[1]] - 1) / 2.0)


def _radius(case):
    n = (case["nx"], case["ny"], case["nz"])
    return float(min(10, min(n[1:] if case["bc"] == "jet" else n[:2]) // 4))


def _inlet(case):
    u = (JET_U, 0.0, 0.0) if case["bc"] == "jet" else (0.0, 0.0, JET_U)
    return {"inlet_u": u, "inlet_center": _center(case), "inlet_radius": _radius(case), "inlet_noise": JET_NOISE,
            "seed": 4321, "inlet_noise_kind": 1 if case["bc"] == "zjet" else 0}


def _tau_z(case):
    """Outlet sponge of the jet along z: the viscosity grows over the last planes."""
    width = min(50, case["nz"] // 4)
    xi = np.clip((np.arange(case["nz"]) - (case["nz"] - 1 - width)) / width, 0.0, 1.0)
    return [float(np.float32(v)) for v in 0.5 + (case["tau"] - 0.5) * (1.0 + 1000.0 * xi ** 3)]


def _state(case, seed):
    """Moments (rho - 1, u, Pi) of a developed flow: the mean profile of the boundary kind plus fluctuations."""
    gen = _gen(seed)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    shape = (nz, ny, nx)
    st = torch.zeros((10,) + shape, dtype=torch.float32, device="cuda")
    x = torch.arange(nx, device="cuda", dtype=torch.float32)[None, None, :]
    y = torch.arange(ny, device="cuda", dtype=torch.float32)[None, :, None]
    z = torch.arange(nz, device="cuda", dtype=torch.float32)[:, None, None]
    amp = 0.0025
    if case["bc"] in ("channel", "duct"):
        h = (ny - 2) / 2.0
        st[1] = 0.05 * (1.0 - ((y - (ny - 1) / 2.0) / h) ** 2).clamp_(min=0.0)
    elif case["bc"] == "periodic":
        kx, ky = 2.0 * math.pi / nx, 2.0 * math.pi / ny
        st[1] = 0.02 * torch.sin(kx * x) * torch.cos(ky * y)
        st[2] = -0.02 * torch.cos(kx * x) * torch.sin(ky * y)
    else:
        c, along = _center(case), (0 if case["bc"] == "jet" else 2)
        a, b = (y, z) if along == 0 else (x, y)
        st[1 + along] = JET_U * torch.exp(-((a - c[0]) ** 2 + (b - c[1]) ** 2) / (2.0 * (_radius(case) + 2.0) ** 2))
    two_d = case["lattice"] == 9
    st[0] += _noise(shape, 1e-3, gen)
    for a in range(2 if two_d else 3):
        st[1 + a] += _noise(shape, amp, gen)
    for k in ((0, 1, 3) if two_d else range(6)):
        st[4 + k] = _noise(shape, 1e-4, gen)
    return st


def _force_field(case, seed):
    gen = _gen(seed + 500_000)
    g = torch.empty((3, case["nz"], case["ny"], case["nx"]), dtype=torch.float32, device="cuda")
    g.normal_(0.0, 1e-6, generator=gen)
    if case["lattice"] == 9:
        g[2] = 0.0
    return g


def _solver(case):
    more = _inlet(case) if case["bc"] in ("jet", "zjet") else {}
    s = Solver(case["nx"], case["ny"], case["nz"], case["tau"], force=_force(case), faces=FACES[case["bc"]],
               storage=STORAGE[case["storage"]][0], order=case["order"], lattice=case["lattice"], **more)
    if case["bc"] == "zjet":
        s.set_relaxation_profile(_tau_z(case))
    return s


def prepare(case, seed):
    kind = case["kind"]
    s = _solver(case)
    p = {"case": case, "solver": s}
    if kind == "grad":
        st = _state(case, seed)
        p["u0"] = st[1:4].clone().requires_grad_(True)
        p["g"] = _force_field(case, seed).requires_grad_(True)
        return p
    st = _state(case, seed)
    if case["field"] and kind != "stats":
        s.set_force_field(_force_field(case, seed))
    if kind == "run":
        p["st"] = st
        return p
    s.set_state(st)
    if kind == "loop":
        s.bind_state_to_torch()
        dtype = STORAGE[case["storage"]][1]
        # steps is even: the level after a pass is in the buffer it started from
        p["view"] = s.state_buffers[0].view(dtype).view((10,) + s.shape)
    elif kind == "adjoint":
        p["raw0"] = s.save_raw()
        s.step(1)
        p["raw1"] = s.save_raw()
        p["lam"] = _lambda(case, seed)
        p["dg"] = torch.zeros((3,) + s.shape, dtype=torch.float32, device="cuda")
    else:
        s.stats_begin(profile_axis=_axis(case), field=case["field"])
        s.stats_sample()
        s.set_state(_state(case, seed + 250_000))
    return p


def _lambda(case, seed):
    """Sensitivities as a later adjoint step leaves them: of the size of u, zero on walls."""
    lam = _noise((10, case["nz"], case["ny"], case["nx"]), 0.02, _gen(seed + 750_000))
    if case["bc"] == "channel":
        lam[:, :, 0] = 0.0
        lam[:, :, -1] = 0.0
    return lam


def _axis(case):
    return 2 if case["bc"] == "zjet" else 1


def run(state):
    case, s = state["case"], state["solver"]
    kind = case["kind"]
    if kind == "loop":
        s.step(case["steps"])
        return state["view"]
    if kind == "run":
        s.t = 0
        s.set_state(state["st"])
        s.step(case["steps"])
        return s.get_state()
    if kind == "grad":
        loss = TslbRollout.apply(state["g"], state["u0"], s, case["steps"], case["every"])
        dg, du = torch.autograd.grad(loss, (state["g"], state["u0"]))
        return {"loss": loss.detach(), "dg": dg, "du": du}
    if kind == "adjoint":
        return {"lam": s.adjoint_step(state["raw0"], state["raw1"], state["lam"], state["dg"]), "dg": state["dg"]}
    s.stats_sample()
    rows, _ = s.stats_profile()
    sums, _ = s.reduce()
    out = {"profile": rows, "sums": np.array(sums)}
    if case["field"]:
        mean, cov = s.stats_field()
        uc, rhalf = s.stats_jet(2, _center(case))
        out.update(mean=mean, cov=cov, uc=uc, rhalf=rhalf)
    return out


def work(case):
    """Bytes and operations of a pass.  An update reads the stored fields of a node and writes them (ten fields, six
    on D2Q9), plus a force field; its operations are those of the separable evaluation and summation of the
    populations.  An adjoint step reads the ten moments, (rho, u) of the next level, ten sensitivities and the force,
    and writes ten sensitivities and the three force gradients it has read."""
    n = case["nx"] * case["ny"] * case["nz"]
    size = 4 if case["storage"] == "fp32" else 2
    step = (2 * (6 if case["lattice"] == 9 else 10) * size + (12 if case["field"] else 0)) * n
    ops = {9: 120, 19: 330, 27: 380}[case["lattice"]] * n
    adj, adj_ops = (160 + (12 if case["field"] else 0)) * n, 700 * n
    kind, steps = case["kind"], case["steps"]
    if kind == "loop":
        return {"bytes": steps * step, "flops": steps * ops}
    if kind == "run":  # fields in, state written; state read, fields out
        return {"bytes": steps * step + 2 * (40 + 10 * size) * n, "flops": steps * ops}
    if kind == "grad":
        return {"bytes": steps * (2 * step + adj), "flops": steps * (2 * ops + adj_ops)}
    if kind == "adjoint":
        return {"bytes": adj, "flops": adj_ops}
    # the sample reads the velocity, the conservation check every moment; the per-node sums are read and written
    # once and read again for the moments
    return {"bytes": (13 * size + (2 * 72 + 72 + 36 if case["field"] else 0)) * n, "flops": 60 * n}


# ------------------------------------------------------------------------------------- 64-bit values
def _velocities(lattice):
    out = []
    for cz in (-1, 0, 1):
        for cy in (-1, 0, 1):
            for cx in (-1, 0, 1):
                n = abs(cx) + abs(cy) + abs(cz)
                if lattice == 9:
                    if cz == 0:
                        out.append((cx, cy, cz, (4 / 9, 1 / 9, 1 / 36)[n]))
                elif lattice == 19:
                    if n < 3:
                        out.append((cx, cy, cz, (1 / 3, 1 / 18, 1 / 36)[n]))
                else:
                    out.append((cx, cy, cz, (8 / 27, 2 / 27, 1 / 54, 1 / 216)[n]))
    return out


def _dot(c, v):
    s = 0.0
    for k in range(3):
        if c[k]:
            s = s + c[k] * v[k]
    return s


def _emitted(m, g, omo, v, order, lattice):
    """Deviation from its rest value of the population that nodes with moments m (rho - 1, u, Pi) emit along v."""
    c, w = v[:3], v[3]
    rho, u, p = 1.0 + m[0], m[1:4], m[4:10]
    rows = ((p[0], p[3], p[4]), (p[3], p[1], p[5]), (p[4], p[5], p[2]))
    u2, tr = u[0] * u[0] + u[1] * u[1] + u[2] * u[2], p[0] + p[1] + p[2]
    cu, pc = _dot(c, u), [_dot(c, rows[a]) for a in range(3)]
    cpc = _dot(c, pc)
    eq = 3.0 * cu + 4.5 * cu * cu - 1.5 * u2
    neq = 4.5 * cpc - 1.5 * tr
    out = m[0] + 3.0 * rho * _dot(c, g)
    if order == 3 and lattice != 19:
        eq = eq + 4.5 * cu * cu * cu - 4.5 * cu * u2
        neq = neq + 13.5 * cpc * cu - 4.5 * tr * cu - 9.0 * (pc[0] * u[0] + pc[1] * u[1] + pc[2] * u[2])
    if order == 3 and lattice == 19:
        # the pairs (aab, bcc) of the third-order coefficient, on their sums and differences
        def a3(a, b):  # a_aab
            return rho * u[a] * u[a] * u[b] + omo * (rows[a][a] * u[b] + 2.0 * rows[a][b] * u[a])
        for a, b, k in ((0, 1, 2), (2, 0, 1), (1, 2, 0)):
            if c[b]:
                plus, minus = a3(a, b) + a3(k, b), a3(a, b) - a3(k, b)
                out = out + c[b] * ((c[a] ** 2 + c[k] ** 2) * 13.5 * plus + (c[a] ** 2 - c[k] ** 2) * 4.5 * minus - 9.0 * plus)
    return w * (out + rho * eq + omo * neq)


def _shift(t, c):
    s = [c[2 - d] for d in range(3) if c[2 - d]]
    return torch.roll(t, s, [d for d in range(3) if c[2 - d]]) if s else t


def _solid(case):
    m = torch.zeros((case["nz"], case["ny"], case["nx"]), dtype=torch.bool, device="cuda")
    f = FACES[case["bc"]]
    for d in range(3):
        for hi in (0, 1):
            if f[2 * d + hi] == WALL:
                m.select(2 - d, -hi)[...] = True
    return m if bool(m.any()) else None


def _step64(case, m, g, omo, solid):
    vs, order, lat = _velocities(case["lattice"]), case["order"], case["lattice"]
    D, J, S = 0.0, [0.0] * 3, [0.0] * 6
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
    for i, v in enumerate(vs):
        f = _shift(_emitted(m, g, omo, v, order, lat), v)
        if solid is not None and any(v[:3]):
            from_wall = _shift(solid, v)
            f = torch.where(from_wall, _emitted(m, g, omo, vs[len(vs) - 1 - i], order, lat), f)
        D = D + f
        for a in range(3):
            if v[a]:
                J[a] = J[a] + v[a] * f
        for k, (a, b) in enumerate(pairs):
            if v[a] * v[b]:
                S[k] = S[k] + v[a] * v[b] * f
    out = torch.zeros_like(m)
    out[0] = D
    dims = 2 if lat == 9 else 3
    for a in range(dims):
        out[1 + a] = J[a] / (1.0 + D)
    for k, (a, b) in enumerate(pairs):
        if a < dims and b < dims:
            out[4 + k] = S[k] - J[a] * out[1 + b] - (D / 3.0 if a == b else 0.0)
    if solid is not None:
        out[:, solid] = 0.0
    return out


def _mix(seed, k):
    z = np.uint64(seed) + k * np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _ghosts64(case, m, t):
    """The ghost layers copy their interior neighbour; the inlet disc has the imposed velocity and its noise."""
    f, n = FACES[case["bc"]], (case["nx"], case["ny"], case["nz"])
    ghost = [(d, hi) for d in range(3) for hi in (0, 1) if f[2 * d + hi] in (INLET, OUTLET)]
    if not ghost:
        return
    for d, hi in ghost:  # one axis after another: edges and corners end up with their diagonal neighbour
        m.select(3 - d, n[d] - 1 if hi else 0).copy_(m.select(3 - d, n[d] - 2 if hi else 1))
    inlet = _inlet(case)
    d = [f[2 * a] for a in range(3)].index(INLET)
    e1, e2 = [a for a in range(3) if a != d]
    b, a = np.meshgrid(np.arange(n[e2]), np.arange(n[e1]), indexing="ij")
    c = inlet["inlet_center"]
    on = (a - c[0]) ** 2 + (b - c[1]) ** 2 <= inlet["inlet_radius"] ** 2
    a, b = a[on].astype(np.int64), b[on].astype(np.int64)
    stride = (1, n[0], n[0] * n[1])
    node = a * stride[e1] + b * stride[e2]
    at = torch.from_numpy(node).cuda()
    amp = float(np.float32(JET_NOISE)) * float(np.float32(JET_U))
    tn = (np.uint64(t) * np.uint64(n[0] * n[1] * n[2]) + node.astype(np.uint64))
    for q in range(3):
        if inlet["inlet_noise_kind"] == 1:
            k = np.uint64(1 + 2 * q) + np.uint64(6) * tn
            v1 = ((_mix(inlet["seed"], k) >> np.uint64(40)).astype(np.float64) + 1.0) * 2.0 ** -24
            v2 = (_mix(inlet["seed"], k + np.uint64(1)) >> np.uint64(40)).astype(np.float64) * 2.0 ** -24
            xi = np.sqrt(-2.0 * np.log(v1)) * np.cos(2.0 * np.pi * v2)
        else:
            xi = (_mix(inlet["seed"], np.uint64(1 + q) + np.uint64(3) * tn) >> np.uint64(40)).astype(np.float64) * 2.0 ** -23 - 1.0
        m[1 + q].view(-1)[at] = torch.from_numpy(float(np.float32(inlet["inlet_u"][q])) + amp * xi).cuda()


def _setup64(case, seed):
    g = [torch.tensor(v, dtype=torch.float64, device="cuda") for v in _force(case)]
    if case["field"] and case["kind"] != "stats":
        g = list(_force_field(case, seed).double())
    tau = torch.tensor(float(np.float32(case["tau"])), dtype=torch.float64, device="cuda")
    if case["bc"] == "zjet":
        tau = torch.tensor(_tau_z(case), dtype=torch.float64, device="cuda")[:, None, None]
    return g, 1.0 - 1.0 / tau, _solid(case)


def _start64(case, seed, solid):
    m = _state(case, seed).double()
    if solid is not None:
        m[:, solid] = 0.0
    _ghosts64(case, m, 0)
    return m


def _vjp64(case, m, m1, lam, g, omo, solid):
    """Transpose of one update, linearised at m with the new level m1: (sensitivities of m, of g)."""
    vs, u1 = _velocities(27), m1[1:4]
    fluid = 1.0 if solid is None else (~solid).double()
    at = [x.detach().clone().requires_grad_(True) for x in m]
    gg = [(x if x.dim() else x.expand(m.shape[1:])).detach().clone().requires_grad_(True) for x in g]

    def arrival(v):
        r = [v[a] - u1[a] for a in range(3)]
        s = lam[0] + (lam[1] * r[0] + lam[2] * r[1] + lam[3] * r[2]) / (1.0 + m1[0])
        for k, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
            s = s + lam[4 + k] * (r[a] * r[b] - (1.0 / 3.0 if a == b else 0.0))
        return s * fluid

    total = [torch.zeros_like(m[0]) for _ in range(13)]
    for i, v in enumerate(vs):
        back = tuple(-x for x in v[:3])
        a = arrival(v)
        if solid is None:
            a = _shift(a, back)
        else:
            opp = vs[len(vs) - 1 - i]
            own = arrival(opp) * _shift(solid, opp).double() if any(back) else 0.0
            a = _shift(a * (~_shift(solid, v)).double(), back) + own
        f = _emitted(at, gg, omo, v, 3, 27)
        for k, x in enumerate(torch.autograd.grad(f, at + gg, a, allow_unused=True)):
            if x is not None:
                total[k] += x
    if solid is not None:
        for x in total:
            x[solid] = 0.0
    return torch.stack(total[:10]), torch.stack(total[10:])


def exact(case, seed):
    kind = case["kind"]
    g, omo, solid = _setup64(case, seed)
    if kind == "stats":
        return _stats64(case, seed, solid)
    if kind == "grad":
        st = _state(case, seed).double()
        m = torch.zeros_like(st)
        m[1:4] = st[1:4]
        levels = [m]
        for _ in range(case["steps"]):
            levels.append(_step64(case, levels[-1], g, omo, solid))
        m = levels[-1]
        u2 = m[1] ** 2 + m[2] ** 2 + m[3] ** 2
        lam = torch.zeros_like(m)
        lam[0], lam[1:4] = 0.5 * u2, (1.0 + m[0]) * m[1:4]
        dg = torch.zeros_like(m[:3])
        for k in range(case["steps"] - 1, -1, -1):
            lam, d = _vjp64(case, levels[k], levels[k + 1], lam, g, omo, solid)
            dg += d
        return {"loss": (0.5 * (1.0 + m[0]) * u2).sum(), "dg": dg, "du": lam[1:4]}
    m = _start64(case, seed, solid)
    if kind == "adjoint":
        lam, dg = _vjp64(case, m, _step64(case, m, g, omo, solid), _lambda(case, seed).double(), g, omo, solid)
        return {"lam": lam, "dg": dg}
    for t in range(case["steps"]):
        m = _step64(case, m, g, omo, solid)
        _ghosts64(case, m, t + 1)
    if kind == "loop":
        s = SCALE[case["storage"]]
        m[0] *= s[0]
        m[1:4] *= s[1]
        m[4:10] *= s[2]
    return m


def _stats64(case, seed, solid):
    """Sums over two samples; the values summed are the stored ones (16-bit storage rounds them on the way in)."""
    dtype, sc = STORAGE[case["storage"]][1], SCALE[case["storage"]]
    f = FACES[case["bc"]]
    states = []
    for sd in (seed, seed + 250_000):
        m = _state(case, sd)
        for k in range(10):
            s = sc[0 if k == 0 else 1 if k < 4 else 2]
            m[k] = (m[k] * s).to(dtype).float() / s
        m = m.double()
        if solid is not None:
            m[:, solid] = 0.0
        _ghosts64(case, m, 0)
        if dtype != torch.float32 and case["bc"] == "zjet":
            m[1:4, 0] = (m[1:4, 0] * sc[1]).to(dtype).double() / sc[1]
        states.append(m)
    fluid = torch.ones((case["nz"], case["ny"], case["nx"]), dtype=torch.float64, device="cuda")
    for d in range(3):
        for hi in (0, 1):
            if f[2 * d + hi] != PERIODIC:
                fluid.select(2 - d, -hi)[...] = 0.0
    axis = _axis(case)
    over = [d for d in range(3) if d != 2 - axis]
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
    rows = 0.0
    for m in states:
        u = m[1:4]
        q = [torch.ones_like(fluid)] + list(u) + [u[a] * u[b] for a, b in pairs] + [x ** 3 for x in u]
        rows = rows + torch.stack([(x * fluid).sum(over) for x in q], 1)
    m = states[1]
    rho = (1.0 + m[0]) * fluid
    sums = torch.stack([rho.sum()] + [(rho * m[1 + a]).sum() for a in range(3)] +
                       [(0.5 * rho * (m[1] ** 2 + m[2] ** 2 + m[3] ** 2)).sum()])
    out = {"profile": rows, "sums": sums}
    if case["field"]:
        mean = (states[0][1:4] + states[1][1:4]) / 2.0
        cov = torch.stack([(states[0][1 + a] * states[0][1 + b] + states[1][1 + a] * states[1][1 + b]) / 2.0 -
                           mean[a] * mean[b] for a, b in pairs])
        uc, rhalf = _jet64(case, mean[2])
        out.update(mean=mean, cov=cov, uc=uc, rhalf=rhalf)
    return out


def _jet64(case, w):
    """Centreline velocity and half-width of every cross-section from the ring averages of the axial velocity."""
    c = _center(case)
    y, x = torch.meshgrid(torch.arange(case["ny"], device="cuda", dtype=torch.float64),
                          torch.arange(case["nx"], device="cuda", dtype=torch.float64), indexing="ij")
    r = torch.sqrt((x - c[0]) ** 2 + (y - c[1]) ** 2).reshape(-1)
    k = r.floor().long()
    nb = int(k.max()) + 1
    count = torch.bincount(k, minlength=nb).double()
    radius = (torch.zeros(nb, dtype=torch.float64, device="cuda").index_add_(0, k, r) / count).tolist()
    ring = torch.zeros((case["nz"], nb), dtype=torch.float64, device="cuda").index_add_(1, k, w.reshape(case["nz"], -1))
    mean, full = (ring / count).tolist(), (count > 0).tolist()
    uc, rh = [row[0] for row in mean], []
    for row in mean:
        prev, got = 0, -1.0
        for b in range(1, nb):
            if not full[b]:
                continue
            if row[b] <= 0.5 * row[0]:
                got = radius[prev] + (radius[b] - radius[prev]) * (row[prev] - 0.5 * row[0]) / (row[prev] - row[b])
                break
            prev = b
        rh.append(got)
    return torch.tensor(uc, dtype=torch.float64), torch.tensor(rh, dtype=torch.float64)
