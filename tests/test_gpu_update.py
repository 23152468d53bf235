"""The one-call update (time step, predictor or corrector, view refresh) against
the separate calls it stands for, at sizes around a block, with fixed and moving
walls, particles that leave the grid and a case above the size up to which
every block sums the partial results itself.

The same FP64 expressions are evaluated on both sides: whole numbers and the
time step must be equal, positions may differ by one rounding of FP64 and
velocities and densities by one of FP32 where a compiler fuses differently."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2104_00537_amd import cases

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2104_00537_amd import sph as S
    from paper_2104_00537_amd.runner import Simulation

DEV = "cuda:0"


def _case(kind):
    if kind == "moving":
        c = cases.sloshing_3d(dp=0.05, seed=3, cell_div=2, x_sub=4)
        assert c.params.motion_omega != 0.0
    elif kind == "2d":
        c = cases.dam_break_2d(cell_div=2, x_sub=4)
    elif kind == "large":
        c = cases.block_case(3, (70, 66, 62), walls=False, cell_div=2, x_sub=2, seed=5)
    else:
        c = cases.block_case(3, (15, 14, 9), walls=True, cell_div=2, x_sub=4, seed=5)
    rng = np.random.default_rng(11)
    fluid = c.type == cases.FLUID
    c.vel[:, fluid] += rng.uniform(-0.3, 0.3, (c.params.dim, fluid.sum())).astype(np.float32)
    if kind == "leaving":  # three particles below the grid's upper end, on their way out
        out = np.flatnonzero(fluid)[:3]
        cp = c.params
        c.pos[-1, out] = cp.origin[-1] + cp.ncell[-1] * cp.cell_size - 1e-9 * cp.dp
        c.vel[-1, out] = np.float32(1.0)
    return c


def _run(c, n, fused):
    """Binning, then two half steps with an interaction before each."""
    cp = c.params
    P = S.make_params(cp)
    src = S.DeviceState.from_case(c, DEV)
    b = S.DeviceState.empty(cp.dim, n, DEV)
    saved = S.DeviceState.empty(cp.dim, n, DEV)
    key = torch.empty(n, dtype=torch.int32, device=DEV)
    perm = torch.empty_like(key)
    start = torch.empty(cp.ncell_total() + 1, dtype=torch.int32, device=DEV)
    ws = torch.zeros(S.sph_workspace_bytes(P, n), dtype=torch.uint8, device=DEV)
    ace = torch.zeros((cp.dim, n), dtype=torch.float32, device=DEV)
    arho = torch.zeros(n, dtype=torch.float32, device=DEV)
    nbr = torch.zeros(n, dtype=torch.int32, device=DEV)
    dt, dth = (torch.zeros(1, dtype=torch.float64, device=DEV) for _ in range(2))
    t = torch.full((1,), 0.37, dtype=torch.float64, device=DEV)
    inter = torch.zeros(2, dtype=torch.int64, device=DEV)
    S.sph_bin_cells(P, n, src, b, key, perm, start, ws)
    S.sph_interact(P, n, b, key, start, ace, arho, ws)
    if fused:
        S.sph_symplectic_update(P, n, 0, dt, dth, inter, t, saved, b, ace, arho, key, ws)
    else:
        S.sph_reduce_dt(P, n, dt, ws, interactions=inter)
        S.sph_symplectic_step(P, n, 0, dt, t, saved, b, ace, arho, ws)
        S.sph_refresh_view(P, n, b, key, ws)
    S.sph_interact(P, n, b, key, start, ace, arho, ws, nbr=nbr, flags=S.SPH_INTERACT_REUSE_CELLS)
    half = [x.cpu().numpy().copy() for x in (b.pos, b.vel, b.rho, b.type, saved.pos, saved.vel,
                                             saved.rho, ace, arho, nbr)]
    if fused:
        S.sph_symplectic_update(P, n, 1, dt, dth, inter, t, saved, b, ace, arho, key, ws)
    else:
        S.sph_reduce_dt(P, n, dth, ws, interactions=inter)
        S.sph_symplectic_step(P, n, 1, dt, t, saved, b, ace, arho, ws)
    torch.cuda.synchronize()
    full = [x.cpu().numpy().copy() for x in (b.pos, b.vel, b.rho, b.type)]
    return half, full, (dt.item(), dth.item(), t.item(), inter.tolist(), S.sph_read_error(ws))


@pytest.mark.parametrize("kind,n", [("fixed", None), ("fixed", 1), ("fixed", 256), ("fixed", 257),
                                    ("moving", None), ("2d", None), ("leaving", None),
                                    ("large", None)])
def test_one_call_matches_the_separate_calls(kind, n):
    c = _case(kind)
    if n is not None:
        sel = np.random.default_rng(n).permutation(c.n)[:n]
        c = cases.Case(c.params, np.ascontiguousarray(c.pos[:, sel]),
                       np.ascontiguousarray(c.vel[:, sel]), c.rho[sel].copy(), c.type[sel].copy(),
                       dict(c.meta))
    if kind == "large":
        assert c.n > 262144
    ha, fa, sa = _run(c, c.n, False)
    hb, fb, sb = _run(c, c.n, True)
    assert sa[0] == sb[0] and sa[2:] == sb[2:]
    assert sa[1] == pytest.approx(sb[1], rel=1e-5)
    if kind == "leaving":
        assert np.count_nonzero(hb[3] & 0x80) == 3 and sb[4] != 0
    for a, b, tol in zip(ha + fa, hb + fb, [4e-16, 2e-7, 2e-7, 0, 0, 0, 0, 1e-5, 1e-5, 0,
                                            4e-16, 1e-5, 2e-7, 0]):
        assert a.dtype == b.dtype
        ok = np.isfinite(a)
        assert np.array_equal(ok, np.isfinite(b))
        if ok.any():
            scale = np.abs(a[ok].astype(np.float64)).max()
            err = np.abs(a[ok].astype(np.float64) - b[ok].astype(np.float64)).max()
            assert err <= tol * scale, (kind, tol, err, scale)


def test_timing_other_calls_leaves_the_step_as_it_is():
    """Events around the interactions alone, as the benchmark records them: the
    step takes the one-call update and the fused concentration as without, bit for
    bit (a size at which shifting by itself would sum C over another number of
    lanes).  Timed call by call, the update's parts run apart: one rounding of
    FP32 in the velocities, of which positions take a time step's share."""
    out = []
    for timed in ("none", "interact", "all"):
        c = cases.block_case(3, (34, 32, 26), walls=True, cell_div=2, x_sub=4, seed=5)
        c.params = dataclasses.replace(c.params, shift_coef=2.0, shift_fs=0.9)
        rng = np.random.default_rng(3)
        c.vel[:] = rng.uniform(-0.3, 0.3, c.vel.shape).astype(np.float32)
        sim = Simulation(c, DEV)
        timing = None if timed == "none" else {}
        sim.timed_calls = ("interact",) if timed == "interact" else None
        for _ in range(3):
            sim.step(timing=timing)
        torch.cuda.synchronize()
        assert sim.error() == 0
        if timed == "interact":
            assert {k: len(v) for k, v in timing.items()} == {"interact": 6}
        if timed == "all":
            assert "update" not in timing and len(timing["shifting"]) == 3
        out.append((sim.state.pos, sim.state.vel, sim.state.rho))
    assert all(torch.equal(x, y) for x, y in zip(out[0], out[1]))
    for x, y, tol in zip(out[0], out[2], (1e-9, 1e-5, 1e-5)):
        assert (x - y).abs().max().item() <= tol * y.abs().max().item()


def test_one_buffer_for_both_time_steps():
    """dt_half = dt: the second pass's time step is written before the corrector
    reads it, as in the separate calls; every result equals theirs."""
    c = _case("fixed")
    P, n, dim = S.make_params(c.params), c.n, c.params.dim
    out = []
    for fused in (False, True):
        src, b = S.DeviceState.from_case(c, DEV), S.DeviceState.empty(dim, n, DEV)
        saved = S.DeviceState.empty(dim, n, DEV)
        key, perm = (torch.empty(n, dtype=torch.int32, device=DEV) for _ in range(2))
        start = torch.empty(c.params.ncell_total() + 1, dtype=torch.int32, device=DEV)
        ws = torch.zeros(S.sph_workspace_bytes(P, n), dtype=torch.uint8, device=DEV)
        ace, arho = torch.zeros((dim, n), device=DEV), torch.zeros(n, device=DEV)
        dt, t = (torch.zeros(1, dtype=torch.float64, device=DEV) for _ in range(2))
        inter = torch.zeros(2, dtype=torch.int64, device=DEV)
        S.sph_bin_cells(P, n, src, b, key, perm, start, ws)
        S.sph_interact(P, n, b, key, start, ace, arho, ws)
        S.sph_reduce_dt(P, n, dt, ws)
        first = dt.item()
        S.sph_symplectic_step(P, n, 0, dt, t, saved, b, ace, arho, ws)
        S.sph_refresh_view(P, n, b, key, ws)
        S.sph_interact(P, n, b, key, start, ace, arho, ws, flags=S.SPH_INTERACT_REUSE_CELLS)
        if fused:
            S.sph_symplectic_update(P, n, 1, dt, dt, inter, t, saved, b, ace, arho, key, ws)
        else:
            S.sph_reduce_dt(P, n, dt, ws, interactions=inter)
            S.sph_symplectic_step(P, n, 1, dt, t, saved, b, ace, arho, ws)
        assert dt.item() != first and t.item() == dt.item()
        out.append((dt.clone(), t.clone(), inter, b.pos, b.vel, b.rho, b.type))
    assert all(torch.equal(x, y) for x, y in zip(*out))


def test_step_of_a_floating_case_without_bodies():
    """floating = 1 and an empty body list: the step takes the separate calls,
    timed or not, with the same results."""
    out = []
    for timing in (None, {}):
        c = dataclasses.replace(cases.floating_box(2, dp=0.04), bodies=None)
        c.vel[:, c.type == cases.FLUID] = np.float32(0.1)
        sim = Simulation(c, DEV)
        assert sim.reuse_cells and sim.params.floating == 1
        for _ in range(3):
            sim.step(timing=timing)
        assert sim.error() == 0
        out.append((sim.state.pos, sim.state.vel, sim.state.rho, sim.t))
    assert all(torch.equal(x, y) for x, y in zip(*out))
