"""Performance cases of the WCSPH hot path, through its public entry points.

A case is a scene (a tank with fluid and wall particles, its resolution and its
formulation) and the path that a program takes through it: a symplectic or
Verlet step of a Simulation, steps replayed from a HIP graph, a step of the
serving engine's batch, or one stage of the step (binning, interaction, wall
densities) through the calls of the C ABI.

The particles are what a running simulation holds: disordered positions, a
smooth flow with small-scale noise, near-hydrostatic densities, stored in the
cell order that the step before left.  Except for the graph replay, whose
buffers advance, every pass starts from the same state.
"""
import functools
import math

import numpy as np
import torch

DEV = "cuda"
G = 9.81
FLUID, FIXED, MOVING, EXCLUDED = 0, 1, 2, 0x80


# -------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest request of a solver's users and of the serving stream: a
        # 2-D dam break of 3.2k fluid particles, two steps from a HIP graph
        dict(name="replay_dam_2d_4k", path="replay", scene="dam2", m=80),
        # the smallest 3-D dam break of the throughput sweep, eager steps: a
        # parameter study, or a case under development
        dict(name="step_dam_3d_26k", path="step", scene="dam3", m=27),
        # a laptop-sized 3-D case, the upper third of the serving range
        dict(name="step_dam_3d_168k", path="step", scene="dam3", m=58),
        # the benchmark: 3-D dam break with 1.0M fluid particles
        dict(name="step_dam_3d_1m", path="step", scene="dam3", m=126),
        # a production run: sloshing in a closed moving tank, 8M fluid particles
        dict(name="step_slosh_3d_9m", path="step", scene="slosh3", m=200),
        # the interaction by itself, in 2-D at the top of the serving range, with
        # every per-particle output a program can ask for
        dict(name="interact_dam_2d_500k", path="interact", scene="dam2", m=994),
        # formulation options: cubic spline, laminar viscosity, Fourtakas DDT
        dict(name="interact_options_3d_442k", path="interact", scene="dam3", m=84,
             kernel=1, viscosity=1, ddt=2),
        # the neighbour-list stage by itself, on an odd-sized case
        dict(name="bin_dam_3d_3m", path="bin", scene="dam3", m=181),
        # the cheaper integrator, one interaction per step
        dict(name="verlet_dam_3d_442k", path="verlet", scene="dam3", m=84),
        # modified DBC: binning, wall densities and the interaction after them
        dict(name="mdbc_dam_3d_442k", path="mdbc", scene="dam3", m=84),
        # a periodic channel with particle shifting
        dict(name="step_channel_shift_3d", path="step", scene="channel3", m=48, shift=2.0),
        # serving: eight requests of mixed size and dimension, one batched step
        dict(name="batch_8_mixed", path="batch", slots=8, n_lo=2000, n_hi=300000, mix=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    path = rng.choice(("replay", "step", "step", "step", "interact", "interact", "bin", "verlet",
                       "mdbc", "batch", "batch"))
    if path == "batch":
        return dict(path="batch", slots=_log(rng, 2, 24), n_lo=2000,
                    n_hi=_log(rng, 5000, 120000), mix=rng.randrange(1 << 20))
    if path == "replay":
        return dict(path=path, scene="dam2", m=_log(rng, 40, 300))
    if path in ("bin", "mdbc", "verlet"):
        if path == "mdbc" and rng.random() < 0.3:
            return dict(path=path, scene="dam2", m=_log(rng, 60, 700))
        return dict(path=path, scene="dam3", m=_log(rng, 20, 130))
    c = dict(path=path, scene=rng.choice(("dam3", "dam3", "dam2", "slosh3", "channel3")))
    c["m"] = {"dam3": _log(rng, 20, 180), "dam2": _log(rng, 60, 1000), "slosh3": _log(rng, 24, 130),
              "channel3": _log(rng, 16, 56)}[c["scene"]]
    if rng.random() < 0.3:
        c.update(rng.choice((dict(kernel=1), dict(viscosity=1), dict(ddt=2), dict(ddt=0),
                             dict(kernel=1, viscosity=1))))
    if path == "step" and c["scene"] != "dam2" and rng.random() < 0.25:
        c["shift"] = 2.0
    return c


# ------------------------------------------------------------------- scenes
def _grid(*ranges):
    axes = [torch.arange(lo, hi, dtype=torch.int64, device=DEV) for lo, hi in ranges]
    return torch.stack([g.reshape(-1) for g in torch.meshgrid(*axes, indexing="ij")])


def _walls(tank, closed):
    """Two wall layers around a tank of tank[k] lattice cells (open on top
    unless closed)."""
    dim, nz = len(tank), tank[-1]
    foot = [(-2, t + 2) for t in tank[:-1]]
    parts = [_grid(*foot, (-2, 0))]
    if closed:
        parts.append(_grid(*foot, (nz, nz + 2)))
    for k in range(dim - 1):
        for lo, hi in ((-2, 0), (tank[k], tank[k] + 2)):
            r = [(0, tank[j]) if j < k else (-2, tank[j] + 2) for j in range(dim - 1)]
            r[k] = (lo, hi)
            parts.append(_grid(*r, (0, nz)))
    return torch.cat(parts, 1)


@functools.lru_cache(maxsize=1)
def _scene(scene, m, opts):
    """(constants, lattice indices of fluid then walls, fluid count) of a
    scene; independent of the seed."""
    o = dict(opts)
    moving, per = False, ()
    if scene == "dam2":
        dp = 0.8 / m
        nf, tank = (max(2, round(0.4 / dp)), m), (round(1.6 / dp), round(1.0 / dp))
    elif scene == "dam3":
        dp = 0.6 / m
        nf, tank = (m, m, max(2, round(0.3 / dp))), (round(1.6 / dp), m, m)
    elif scene in ("slosh2", "slosh3"):
        dp, moving = 1.0 / m, True
        tank = (2 * m, m, m) if scene == "slosh3" else (2 * m, m)
        nf = tank[:-1] + (max(2, round(o.get("fill", 0.5) * m)),)
    elif scene == "channel3":
        dp, per = 1.0 / m, (0, 1)
        nf = (4 * m, 2 * m, m)  # even: whole cells of 2 dp along x and y
        tank = nf
    else:
        raise ValueError(scene)
    dim = len(tank)
    fluid = _grid(*[(0, n) for n in nf])
    if per:
        walls = torch.cat([_grid((0, nf[0]), (0, nf[1]), (-2, 0)),
                           _grid((0, nf[0]), (0, nf[1]), (nf[2], nf[2] + 2))], 1)
    else:
        walls = _walls(tank, closed=moving)
    idx = torch.cat([fluid, walls], 1)
    h, height = math.sqrt(dim) * dp, nf[-1] * dp
    cell_div, x_sub = 2, 4
    accel, omega = 0.05 * G, math.pi
    period = [0.0] * 3
    if per:
        cs = 2 * dp
        mz = 2.001 * dp + 2 * cs
        origin = [0.0, 0.0, -mz]
        ncell = [nf[0] // 2, nf[1] // 2, math.ceil((nf[2] * dp + 2 * mz) / cs)]
        period = [nf[0] * dp, nf[1] * dp, 0.0]
    else:
        cs, mg = 2.0 * h / cell_div, 2.001 * dp
        hi = [t * dp + mg for t in tank]
        if moving:
            hi[0] += 2.0 * accel / omega ** 2
        else:
            hi[-1] = max(tank[-1], 2.5 * nf[-1]) * dp + mg
        origin = [-mg] * dim + [0.0] * (3 - dim)
        ncell = [math.ceil((e + mg) / cs) for e in hi] + [1] * (3 - dim)
    ncell[0] *= x_sub
    grav = [0.0] * 3
    grav[dim - 1] = -G
    c = dict(name=scene, dim=dim, dp=dp, h=h, rho0=1000.0, gamma=7.0, c0=10.0 * math.sqrt(G * height),
             alpha=0.01, delta=0.1, eta2=0.001 * h * h, cfl=0.2, mass_fluid=1000.0 * dp ** dim,
             mass_bound=1000.0 * dp ** dim, gravity=tuple(grav), ddt=o.get("ddt", 1),
             kernel=o.get("kernel", 0), viscosity=o.get("viscosity", 0), visc_nu=1e-6,
             boundary=o.get("boundary", 0), period=tuple(period), shift_coef=o.get("shift", 0.0),
             shift_fs=0.0, cell_div=cell_div, x_sub=x_sub, origin=tuple(origin), cell_size=cs,
             inv_cell_size=1.0 / cs, ncell=tuple(ncell), motion_amp=accel if moving else 0.0,
             motion_omega=omega if moving else 0.0, fluid_height=height)
    normal = None
    if o.get("boundary"):
        mid = idx.double() + 0.5
        top = torch.tensor(tank, device=DEV)[:, None]
        normal = torch.where(idx < 0, -2.0 * mid, torch.where(idx >= top, 2.0 * (top - mid), 0.0))
        normal = (normal * dp).float()
        normal[:, :fluid.shape[1]] = 0.0
    return c, idx, fluid.shape[1], normal


def _opts(case):
    o = {k: case[k] for k in ("kernel", "viscosity", "ddt", "shift", "fill") if k in case}
    if case.get("path") == "mdbc":
        o["boundary"] = 1
    return tuple(sorted(o.items()))


def _keys(c, pos):
    """Cell keys (x fastest) and whether each position lies in the grid."""
    key = torch.zeros(pos.shape[1], dtype=torch.int64, device=pos.device)
    ok = torch.ones(pos.shape[1], dtype=torch.bool, device=pos.device)
    mul = 1
    for k in range(c["dim"]):
        inv = c["inv_cell_size"] * (c["x_sub"] if k == 0 else 1)
        x = pos[k]
        if c["period"][k] > 0:
            x = _wrap(c, k, x)
        f = torch.floor((x - c["origin"][k]) * inv)
        if c["period"][k] > 0:
            f = torch.where(f == c["ncell"][k], f - 1, f)
        ok &= (f >= 0) & (f < c["ncell"][k])
        key += f.clamp(0, c["ncell"][k] - 1).long() * mul
        mul *= c["ncell"][k]
    return torch.where(ok, key, torch.full_like(key, mul)), mul


def _wrap(c, k, x):
    o, L = c["origin"][k], c["period"][k]
    x = torch.where(x >= o + L, x - L, torch.where(x < o, x + L, x))
    return torch.where(x >= o + L, torch.full_like(x, o), x)


def _inputs(case, seed):
    """The particles of a case as the step before left them, on the GPU:
    (constants, dict of pos, vel, rho, type, id[, normal])."""
    c, idx, nf, normal = _scene(case["scene"], case["m"], _opts(case))
    dim, dp, n = c["dim"], c["dp"], idx.shape[1]
    gen = torch.Generator(device=DEV).manual_seed(seed * 1000003 + case["m"])
    pos = (idx.double() + 0.5) * dp
    jit = torch.rand(pos.shape, generator=gen, device=DEV, dtype=torch.float64) * 2 - 1
    amp = torch.full((n,), 1e-4 * dp, dtype=torch.float64, device=DEV)
    amp[:nf] = 0.15 * dp
    pos += jit * amp
    del jit
    # a smooth flow of about a third of the surge speed, and noise
    ph = torch.rand((dim, dim), generator=gen, device=DEV, dtype=torch.float64) * 6.28
    wave = 4.0 / c["fluid_height"]
    vel = torch.empty((dim, n), dtype=torch.float32, device=DEV)
    for k in range(dim):
        s = sum(torch.sin(wave * pos[j] + ph[k, j]) for j in range(dim))
        vel[k] = (0.3 * math.sqrt(G * c["fluid_height"]) * s / dim).float()
    vel += (0.01 * math.sqrt(G * c["fluid_height"])
            * torch.randn((dim, n), generator=gen, device=DEV, dtype=torch.float32))
    vel[:, nf:] = 0.0
    depth = (c["fluid_height"] - pos[-1]).clamp_min(0.0)
    b = c["c0"] ** 2 * c["rho0"] / c["gamma"]
    rho = c["rho0"] * (1.0 + c["rho0"] * G * depth / b) ** (1.0 / c["gamma"])
    rho = (rho * (1.0 + 5e-4 * (torch.rand((n,), generator=gen, device=DEV,
                                           dtype=torch.float64) * 2 - 1))).float()
    typ = torch.full((n,), MOVING if c["motion_omega"] else FIXED, dtype=torch.uint8, device=DEV)
    typ[:nf] = FLUID
    # the order of the step before: sorted where the particles were then
    dt = 0.2 * c["h"] / c["c0"]
    order = torch.sort(_keys(c, pos - dt * vel.double())[0], stable=True)[1]
    out = dict(pos=pos[:, order].contiguous(), vel=vel[:, order].contiguous(), rho=rho[order],
               type=typ[order], id=torch.arange(n, dtype=torch.int32, device=DEV))
    if normal is not None:
        out["normal"] = normal[:, order].contiguous()
    return c, out


def _slots(case):
    """The requests of a batch: dam breaks and sloshing tanks in 2-D and 3-D
    with log-uniform sizes."""
    rng = np.random.default_rng(case["mix"])
    out = []
    for _ in range(case["slots"]):
        n = math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))
        scene = ("dam2", "dam3", "slosh2", "slosh3")[int(rng.integers(4))]
        per_m = {"dam2": 0.5, "dam3": 0.5, "slosh2": 1.0, "slosh3": 1.0}[scene]
        m = max(8, round((n / per_m) ** (1.0 / int(scene[-1]))))
        out.append(dict(path="batch", scene=scene, m=m))
    return out


def _case_object(c, d):
    from paper_2104_00537_amd import cases as K
    host = {k: v.cpu().numpy() for k, v in d.items()}
    return K.Case(params=K.CaseParams(**c), pos=host["pos"], vel=host["vel"], rho=host["rho"],
                  type=host["type"], normal=host.get("normal"))


# -------------------------------------------------------------- entry points
def prepare(case, seed):
    from paper_2104_00537_amd import sph as S
    from paper_2104_00537_amd.runner import Simulation
    path = case["path"]
    if path == "batch":
        from paper_2104_00537_amd import serve
        reqs = []
        for k, sl in enumerate(_slots(case)):
            c, d = _inputs(sl, seed + 101 * k)
            reqs.append(serve.Request(rid=k, case=_case_object(c, d), steps=1000, arrival=0.0))
        cells = sum(r.case.params.ncell_total() + 1 for r in reqs) + 1
        eng = serve.BatchEngine(sum(serve.padded(r.n) for r in reqs), cells, max_slots=len(reqs),
                                cell_div=2)
        eng.repack([], reqs)
        cur, t = eng.cur, eng.t.clone()
        eng.run(1)  # (captures the step's graph, as the engine's first step does)
        eng.cur = cur
        eng.t.copy_(t)
        return dict(path=path, eng=eng, cur=cur)
    c, d = _inputs(case, seed)
    sim = Simulation(_case_object(c, d), DEV, integrator="verlet" if path == "verlet" else "symplectic")
    st = dict(path=path, sim=sim, S=S, bufs=list(sim.states), saved=list(sim.saved))
    if path == "replay":
        sim.step()
        sim.step()  # (both buffers used once before the capture)
        sim.capture(2)
    elif path == "verlet":
        # the step before the present one
        sim.saved[0].pos.copy_(sim.state.pos)
        sim.saved[0].vel.copy_(sim.state.vel * 0.999)
        sim.saved[0].rho.copy_(sim.state.rho * (1.0 - 1e-6))
    elif path == "interact":
        a, b = sim.states
        S.sph_bin_cells(sim.params, sim.n, a, b, sim.key, sim.perm, sim.cell_start, sim.ws)
        st["visc"] = torch.empty(sim.n, dtype=torch.float32, device=DEV)
        st["nbr"] = torch.empty(sim.n, dtype=torch.int32, device=DEV)
        st["maxima"] = torch.empty(2, dtype=torch.float32, device=DEV)
    return st


def run(state):
    if state["path"] == "batch":
        eng = state["eng"]
        eng.cur = state["cur"]
        eng.run(1)
        n = eng.offsets[-1]
        s = eng._dev_state(eng.cur, n)
        return dict(pos=s.pos, vel=s.vel, rho=s.rho, type=s.type, id=s.id)
    S, sim, path = state["S"], state["sim"], state["path"]
    a, b = state["bufs"]
    if path == "replay":
        sim.replay(1)
        s = sim.state
        return dict(pos=s.pos, vel=s.vel, rho=s.rho, id=s.id)
    if path == "interact":
        S.sph_interact(sim.params, sim.n, b, sim.key, sim.cell_start, sim.ace, sim.arho, sim.ws,
                       visc=state["visc"], nbr=state["nbr"])
        S.sph_reduce_dt(sim.params, sim.n, sim.dt, sim.ws, maxima=state["maxima"])
        return dict(ace=sim.ace, arho=sim.arho, visc=state["visc"], nbr=state["nbr"],
                    maxima=state["maxima"])
    if path == "bin":
        S.sph_bin_cells(sim.params, sim.n, a, b, sim.key, sim.perm, sim.cell_start, sim.ws)
        return dict(key=sim.key, perm=sim.perm, cell_start=sim.cell_start, pos=b.pos, vel=b.vel,
                    rho=b.rho, type=b.type, id=b.id)
    if path == "mdbc":
        S.sph_bin_cells(sim.params, sim.n, a, b, sim.key, sim.perm, sim.cell_start, sim.ws)
        S.sph_mdbc(sim.params, sim.n, b, sim.key, sim.cell_start, sim.ws)
        S.sph_interact(sim.params, sim.n, b, sim.key, sim.cell_start, sim.ace, sim.arho, sim.ws)
        return dict(rho=b.rho, ace=sim.ace, arho=sim.arho, id=b.id)
    # a whole step from the same state: the result goes to the other buffer
    sim.states = [a, b]
    if path == "verlet":
        sim.saved = list(state["saved"])
        sim.steps_done = 1  # (not the first step: Eq. 30)
    sim.step()
    s = sim.state
    out = dict(pos=s.pos, vel=s.vel, rho=s.rho, type=s.type, id=s.id, ace=sim.ace, arho=sim.arho)
    if path == "verlet":
        p = sim.saved[0]
        out.update(prev_vel=p.vel, prev_rho=p.rho)
    return out


# ---------------------------------------------------------------------- work
def _pairs(c, n_all, n_fluid):
    """About the pairs of one interaction: every particle with a full support
    of fluid and walls, half of one for a wall particle."""
    dim = c["dim"]
    s = 2.0 * c["h"] / c["dp"]
    full = math.pi * s * s if dim == 2 else 4.0 / 3.0 * math.pi * s ** 3
    return 0.85 * full * n_fluid + 0.25 * full * (n_all - n_fluid)


def _counts(scene, m):
    """(particles, fluid particles) of a scene, without building it."""
    def box(*e):
        return math.prod(e)
    if scene == "dam2":
        dp = 0.8 / m
        f, t, closed = (max(2, round(0.4 / dp)), m), (round(1.6 / dp), round(1.0 / dp)), 0
    elif scene == "dam3":
        dp = 0.6 / m
        f, t, closed = (m, m, max(2, round(0.3 / dp))), (round(1.6 / dp), m, m), 0
    elif scene == "channel3":
        return box(4 * m, 2 * m, m + 4), box(4 * m, 2 * m, m)
    else:
        t = (2 * m, m, m) if scene == "slosh3" else (2 * m, m)
        f, closed = t[:-1] + (max(2, round(0.5 * m)),), 1
    foot = box(*[e + 4 for e in t[:-1]])
    walls = 2 * foot * (1 + closed) + (foot - box(*t[:-1])) * t[-1]
    return box(*f) + walls, box(*f)


def work(case):
    if case["path"] == "batch":
        w = [work(dict(sl, path="step")) for sl in _slots(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    scene, dim = case["scene"], int(case["scene"][-1])
    n, nf = _counts(scene, case["m"])
    dp = {"dam2": 0.8, "dam3": 0.6}.get(scene, 1.0) / case["m"]
    c = dict(dim=dim, h=math.sqrt(dim) * dp, dp=dp)
    pairs = 50.0 * _pairs(c, n, nf)
    state = 12 * dim + 4  # FP64 positions, FP32 velocities and densities
    path = case["path"]
    if path == "interact":
        return dict(bytes=n * (32.0 + 4 * dim + 12), flops=pairs)
    if path == "bin":
        return dict(bytes=n * (2.0 * (state + 5) + 8), flops=10.0 * n)
    if path == "mdbc":
        return dict(bytes=n * (2.0 * (state + 5 + 4 * dim) + 8 + 4 * dim + 4),
                    flops=pairs + 2.0 * 50.0 * 0.4 * 174 * (n - nf))
    if path == "verlet":
        return dict(bytes=n * (2.0 * (state + 5) + 3.0 * (4 * dim + 4)), flops=pairs)
    one = dict(bytes=n * (2.0 * (state + 5) + 4 * dim + 4), flops=2 * pairs)
    if case.get("shift"):
        one["flops"] += 1.2 * pairs
    return {k: v * (2 if path == "replay" else 1) for k, v in one.items()}


# --------------------------------------------------------------------- exact
class _Search:
    """Sources binned in cells of 2h (plain torch, FP64); periodic components
    get copies of the sources near their ends."""

    def __init__(self, c, pos):
        self.c, dim, h2 = c, c["dim"], 2.0 * c["h"]
        src = torch.arange(pos.shape[1], device=pos.device)
        x = pos
        for k in range(dim):
            L = c["period"][k]
            if L > 0:
                lo, hi = c["origin"][k], c["origin"][k] + L
                parts, ids = [x], [src]
                for sel, s in ((x[k] < lo + 1.01 * h2, L), (x[k] > hi - 1.01 * h2, -L)):
                    y = x[:, sel].clone()
                    y[k] += s
                    parts.append(y)
                    ids.append(src[sel])
                x, src = torch.cat(parts, 1), torch.cat(ids)
        self.lo = x.min(dim=1).values - h2
        self.nc = ((x.max(dim=1).values - self.lo) / h2).long() + 3
        key = self._key(((x - self.lo[:, None]) / h2).long())
        self.key, o = torch.sort(key)
        self.x, self.src = x[:, o].contiguous(), src[o]

    def _key(self, cell):
        k = cell[self.c["dim"] - 1]
        for d in range(self.c["dim"] - 2, -1, -1):
            k = k * self.nc[d] + cell[d]
        return k

    def each(self, tpos, f, chunk=1 << 18):
        """Calls f(target, source, r_ab [dim, pairs], r2) for all pairs within
        2h, in pieces."""
        c, dim, h2 = self.c, self.c["dim"], 2.0 * self.c["h"]
        rows = [(0,)] if dim == 1 else [(y,) for y in (-1, 0, 1)] if dim == 2 else \
            [(y, z) for y in (-1, 0, 1) for z in (-1, 0, 1)]
        order = torch.argsort(self._key(self._cell(tpos)))
        for t0 in range(0, tpos.shape[1], chunk):
            t = order[t0:t0 + chunk]
            p = tpos[:, t]
            cell = self._cell(p)
            for row in rows:
                q = cell.clone()
                q[0] -= 1
                for k, d in enumerate(row):
                    q[1 + k] += d
                ok = torch.ones_like(q[0], dtype=torch.bool)
                for k in range(1, dim):
                    ok &= (q[k] >= 0) & (q[k] < self.nc[k])
                k0 = self._key(q)
                j0 = torch.searchsorted(self.key, k0)
                num = torch.where(ok, torch.searchsorted(self.key, k0 + 3) - j0, 0)
                w = int(num.max()) if num.numel() else 0
                if not w:
                    continue
                j = j0[:, None] + torch.arange(w, device=p.device)
                inside = torch.arange(w, device=p.device) < num[:, None]
                j.clamp_(max=self.key.numel() - 1)
                r2 = torch.zeros(j.shape, dtype=torch.float64, device=p.device)
                for k in range(dim):
                    r2 += (p[k][:, None] - self.x[k][j]) ** 2
                a, b = torch.nonzero(inside & (r2 < h2 * h2), as_tuple=True)
                jj = j[a, b]
                f(t[a], self.src[jj], p[:, a] - self.x[:, jj], r2[a, b])

    def _cell(self, p):
        cell = ((p - self.lo[:, None]) / (2.0 * self.c["h"])).floor().long()
        return torch.maximum(torch.minimum(cell, (self.nc - 1)[:, None]),
                             torch.zeros_like(cell))


def _alpha_d(c):
    h = c["h"]
    if c["kernel"] == 1:
        return 10.0 / (7.0 * math.pi * h * h) if c["dim"] == 2 else 1.0 / (math.pi * h ** 3)
    return 7.0 / (4.0 * math.pi * h * h) if c["dim"] == 2 else 21.0 / (16.0 * math.pi * h ** 3)


def _fab(c, r2):
    q = r2.sqrt() / c["h"]
    if c["kernel"] == 0:
        return -5.0 * _alpha_d(c) / c["h"] ** 2 * (1.0 - 0.5 * q) ** 3
    far = -0.75 * (2.0 - q) ** 2 / q.clamp_min(1e-300)
    return _alpha_d(c) / c["h"] ** 2 * torch.where(q <= 1, -3.0 + 2.25 * q, far)


def _w(c, r2):
    q = r2.sqrt() / c["h"]
    if c["kernel"] == 0:
        return _alpha_d(c) * (1.0 - 0.5 * q) ** 4 * (2.0 * q + 1.0)
    return _alpha_d(c) * torch.where(q <= 1, 1.0 - 1.5 * q ** 2 + 0.75 * q ** 3,
                                     0.25 * (2.0 - q) ** 3)


def _mass(c, fluid):
    return torch.where(fluid, torch.full(fluid.shape, c["mass_fluid"], dtype=torch.float64,
                                         device=fluid.device), c["mass_bound"])


def _tait(c, rho):
    return c["c0"] ** 2 * c["rho0"] / c["gamma"] * ((rho / c["rho0"]) ** c["gamma"] - 1.0)


def _rates(c, pos, vel, rho, fluid, vel_src=None):
    """Eq. 15, 17-23, 28, 36: ace, arho, visc, pair counts, in FP64.
    vel_src: the velocities that neighbours are seen with (modified DBC)."""
    dim, n, h = c["dim"], pos.shape[1], c["h"]
    vs = vel if vel_src is None else vel_src
    P = _tait(c, rho)
    ace = torch.zeros((dim, n), dtype=torch.float64, device=pos.device)
    cont = torch.zeros(n, dtype=torch.float64, device=pos.device)
    diff, visc = torch.zeros_like(cont), torch.zeros_like(cont)
    cnt = torch.zeros(n, dtype=torch.int64, device=pos.device)
    g = abs(c["gravity"][dim - 1])
    b_tait = c["c0"] ** 2 * c["rho0"] / c["gamma"]

    def pair(a, b, r, r2):
        keep = (a != b) & (fluid[a] | fluid[b])
        a, b, r, r2 = a[keep], b[keep], r[:, keep], r2[keep]
        fa, fb = fluid[a], fluid[b]
        mb = _mass(c, fb)
        f = _fab(c, r2)
        dv = vel[:, a] - vs[:, b]
        vr = (dv * r).sum(0)
        ra, rb = rho[a], rho[b]
        cont.index_add_(0, a, mb / rb * f * vr)
        cnt.index_add_(0, a, torch.ones_like(a))
        mu = h * vr / (r2 + c["eta2"])
        coef = (P[a] + P[b]) / (ra * rb)
        if c["viscosity"] == 0:
            coef = coef - torch.where(vr < 0, c["alpha"] * c["c0"] * mu / (0.5 * (ra + rb)), 0.0)
        coef = torch.where(fa, -mb * coef * f, 0.0)
        if c["viscosity"] == 1:
            lam = mb * 4.0 * c["visc_nu"] * f * r2 / ((ra + rb) * (r2 + c["eta2"]))
            lam = torch.where(fa, lam, 0.0)
        for k in range(dim):
            t = coef * r[k]
            if c["viscosity"] == 1:
                t = t + lam * dv[k]
            ace[k].index_add_(0, a, t)
        visc.index_reduce_(0, a, torch.where(fa, mu.abs(), 0.0), "amax")
        if c["ddt"]:
            dr = rb - ra
            if c["ddt"] == 2:
                e = c["rho0"] * g * r[dim - 1] / b_tait
                dr = dr - c["rho0"] * ((1.0 + e) ** (1.0 / c["gamma"]) - 1.0)
            diff.index_add_(0, a, torch.where(fa & fb, -2.0 * dr * f * mb / rb, 0.0))

    _Search(c, pos).each(pos, pair)
    for k in range(dim):
        ace[k] += c["gravity"][k]
    arho = rho * cont + c["delta"] * h * c["c0"] * diff
    arho = torch.where(fluid, arho, rho * cont)
    return torch.where(fluid, ace, 0.0), arho, torch.where(fluid, visc, 0.0), cnt


def _dt(c, ace, visc, fluid):
    f = float((ace ** 2).sum(0).sqrt()[fluid].max())
    v = float(visc[fluid].max())
    return c["cfl"] * min(math.sqrt(c["h"] / f), c["h"] / (c["c0"] + v)), f, v


def _sorted_state(c, d):
    order = torch.sort(_keys(c, d["pos"])[0], stable=True)[1]
    s = {k: (v[..., order]) for k, v in d.items()}
    for k in range(c["dim"]):
        if c["period"][k] > 0:
            s["pos"][k] = _wrap(c, k, s["pos"][k])
    return order, s


def _exact_step(c, d):
    """A symplectic step (Eq. 33-35, 37, shifting of Section 2.8) in FP64."""
    _, s = _sorted_state(c, d)
    pos, vel, rho = s["pos"], s["vel"].double(), s["rho"].double()
    fluid, moving = s["type"] == FLUID, s["type"] == MOVING
    ace, arho, visc, _ = _rates(c, pos, vel, rho, fluid)
    dt, _, _ = _dt(c, ace, visc, fluid)
    A, w = c["motion_amp"], c["motion_omega"]

    def disp(t):
        return A / w ** 2 * (1.0 - math.cos(w * t)) if w else 0.0

    def wall_v(t):
        return A / w * math.sin(w * t) if w else 0.0

    ph, vh = pos.clone(), vel.clone()
    ph[:, fluid] += 0.5 * dt * vel[:, fluid]
    vh[:, fluid] += 0.5 * dt * ace[:, fluid]
    ph[0, moving] += disp(0.5 * dt)
    vh[0, moving] = wall_v(0.5 * dt)
    rh = rho + 0.5 * dt * arho
    ace2, arho2, _, _ = _rates(c, ph, vh, rh, fluid)
    p1, v1 = pos.clone(), vel.clone()
    v1[:, fluid] = vel[:, fluid] + dt * ace2[:, fluid]
    p1[:, fluid] = pos[:, fluid] + 0.5 * dt * (v1 + vel)[:, fluid]
    p1[0, moving] = pos[0, moving] + disp(dt)
    v1[0, moving] = wall_v(dt)
    eps = -(arho2 / rh) * dt
    r1 = rho * (2.0 - eps) / (2.0 + eps)
    if c["shift_coef"] > 0:
        n = pos.shape[1]
        vol = _mass(c, fluid) / rh
        conc = torch.zeros(n, dtype=torch.float64, device=pos.device)
        grad = torch.zeros_like(pos)
        S = _Search(c, ph)
        S.each(ph, lambda a, b, r, r2: conc.index_add_(0, a, vol[b] * _w(c, r2)))

        def pair(a, b, r, r2):
            t = vol[b] * (conc[b] - conc[a]) * _fab(c, r2)
            for k in range(c["dim"]):
                grad[k].index_add_(0, a, t * r[k])

        S.each(ph, pair)
        dr = -c["shift_coef"] * c["h"] * (vh ** 2).sum(0).sqrt() * dt * grad
        p1 += torch.where(fluid, dr, 0.0)
    return dict(pos=p1, vel=v1, rho=r1, ace=ace2, arho=arho2, type=None, id=None)


def _exact_mdbc(c, s):
    """Eq. 38-39: wall densities and the velocities the fluid sees, FP64."""
    dim = c["dim"]
    pos, vel, rho = s["pos"], s["vel"].double(), s["rho"].double()
    fluid = s["type"] == FLUID
    wall = torch.nonzero(~fluid)[:, 0]
    src = torch.nonzero(fluid)[:, 0]
    ghost = pos[:, wall] + s["normal"][:, wall].double()
    m, nw = dim + 1, wall.numel()
    A = torch.zeros((nw, m, m), dtype=torch.float64, device=pos.device)
    b = torch.zeros((nw, m), dtype=torch.float64, device=pos.device)
    sv = torch.zeros((dim, nw), dtype=torch.float64, device=pos.device)

    def pair(a, j, r, r2):
        j = src[j]
        r = -r  # r_b - r_G
        w, f = _w(c, r2), _fab(c, r2)
        vb = c["mass_fluid"] / rho[j]
        A[:, 0, 0].index_add_(0, a, vb * w)
        b[:, 0].index_add_(0, a, c["mass_fluid"] * w)
        for p in range(dim):
            A[:, 0, 1 + p].index_add_(0, a, vb * w * r[p])
            A[:, 1 + p, 0].index_add_(0, a, vb * f * r[p])
            b[:, 1 + p].index_add_(0, a, c["mass_fluid"] * f * r[p])
            sv[p].index_add_(0, a, vb * w * vel[p, j])
            for q in range(dim):
                A[:, 1 + p, 1 + q].index_add_(0, a, vb * f * r[p] * r[q])

    _Search(c, pos[:, src]).each(ghost, pair)
    wet = A[:, 0, 0] > 0
    good = wet & (torch.linalg.det(A).abs() >= 1e-3)
    eye = torch.eye(m, dtype=torch.float64, device=pos.device)
    x = torch.linalg.solve(torch.where(good[:, None, None], A, eye), b)
    lin = x[:, 0] - (s["normal"][:, wall].double() * x[:, 1:].T).sum(0)
    shep = b[:, 0] / torch.where(wet, A[:, 0, 0], 1.0)
    rho, seen = rho.clone(), vel.clone()
    rho[wall] = torch.where(good, lin, torch.where(wet, shep, c["rho0"]))
    vg = sv / torch.where(wet, A[:, 0, 0], 1.0)
    seen[:, wall] = torch.where(wet, 2.0 * vel[:, wall] - vg, vel[:, wall])
    return rho, seen, fluid


def exact(case, seed):
    """What run() returns, in FP64 (None for whole numbers)."""
    path = case["path"]
    if path == "batch":
        parts = []
        for k, sl in enumerate(_slots(case)):
            c, d = _inputs(sl, seed + 101 * k)
            e, n = _exact_step(c, d), d["pos"].shape[1]
            pad = -(-n // 64) * 64 - n
            if c["dim"] == 2:
                z = torch.zeros_like(e["pos"][0])
                for f in ("pos", "vel"):
                    e[f] = torch.stack([e[f][0], z, e[f][1]])
            e = {f: torch.nn.functional.pad(e[f], (0, pad), value=c["rho0"] if f == "rho" else 0.0)
                 for f in ("pos", "vel", "rho")}
            parts.append(e)
        out = {f: torch.cat([e[f] for e in parts], -1) for f in ("pos", "vel", "rho")}
        return dict(out, type=None, id=None)
    c, d = _inputs(case, seed)
    if path == "step":
        return _exact_step(c, d)
    if path == "replay":
        # four steps from the prepared state (two before the capture)
        keep = d["id"]
        for _ in range(4):
            _, s = _sorted_state(c, dict(d, id=keep))
            e = _exact_step(c, d)
            keep = s["id"]
            d = dict(pos=e["pos"], vel=e["vel"], rho=e["rho"], type=s["type"], id=keep)
        return dict(pos=d["pos"], vel=d["vel"], rho=d["rho"], id=None)
    order, s = _sorted_state(c, d)
    pos, vel, rho = s["pos"], s["vel"].double(), s["rho"].double()
    fluid = s["type"] == FLUID
    if path == "bin":
        return dict(key=None, perm=None, cell_start=None, pos=pos, vel=vel, rho=rho, type=None,
                    id=None)
    if path == "mdbc":
        rho, seen, fluid = _exact_mdbc(c, s)
        ace, arho, _, _ = _rates(c, pos, vel, rho, fluid, vel_src=seen)
        return dict(rho=rho, ace=ace, arho=torch.where(fluid, arho, 0.0), id=None)
    ace, arho, visc, _ = _rates(c, pos, vel, rho, fluid)
    dt, fm, vm = _dt(c, ace, visc, fluid)
    if path == "interact":
        return dict(ace=ace, arho=arho, visc=visc, nbr=None,
                    maxima=torch.tensor([fm, vm], dtype=torch.float64))
    # Verlet, Eq. 30
    v0, r0 = (s["vel"] * 0.999).double(), (s["rho"] * (1.0 - 1e-6)).double()
    p1, v1 = pos.clone(), vel.clone()
    p1[:, fluid] += (dt * vel + 0.5 * dt * dt * ace)[:, fluid]
    v1[:, fluid] = (v0 + 2.0 * dt * ace)[:, fluid]
    r1 = r0 + 2.0 * dt * arho
    return dict(pos=p1, vel=v1, rho=r1, type=None, id=None, ace=ace, arho=arho, prev_vel=vel,
                prev_rho=rho)
