"""The list of wall particles and the lanes per wall of the modified dynamic
boundary condition, at numbers of particles around the 2048 that one block of
the list takes, with walls and fluid in random places, against the CPU oracle.
Both sides sum in FP64, in different orders, and round to FP32: wall densities
within 2e-4 kg/m^3 (two FP32 ulps at 1000)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2104_00537_amd import cases

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2104_00537_amd import sph as S

DEV = "cuda:0"


@pytest.mark.parametrize("dim,n", [(3, 1), (3, 2047), (3, 2048), (3, 2049), (3, 4097),
                                   (2, 63), (2, 2049)])
def test_walls_of_any_count_match_the_oracle(dim, n):
    if dim == 3:
        full = cases.block_case(3, (15, 13, 11), walls=True, seed=4, cell_div=2, x_sub=4)
    else:
        full = cases.block_case(2, (60, 40), walls=True, seed=4, cell_div=2, x_sub=4)
    rng = np.random.default_rng(n)
    sel = rng.permutation(full.n)[:n] if n > 1 else np.flatnonzero(full.type != cases.FLUID)[:1]
    normal = rng.uniform(-1.5, 1.5, (dim, n)).astype(np.float32) * np.float32(full.params.dp)
    c = cases.Case(dataclasses.replace(full.params, boundary=1),
                   np.ascontiguousarray(full.pos[:, sel]), np.ascontiguousarray(full.vel[:, sel]),
                   full.rho[sel].copy(), full.type[sel].copy(), dict(full.meta), normal)
    assert c.n == n
    cp = c.params
    P = S.make_params(cp)
    src = S.DeviceState.from_case(c, DEV, with_normal=True)
    dst = S.DeviceState.empty(dim, n, DEV, with_normal=True)
    key = torch.empty(n, dtype=torch.int32, device=DEV)
    perm = torch.empty_like(key)
    start = torch.empty(cp.ncell_total() + 1, dtype=torch.int32, device=DEV)
    ws = torch.zeros(S.sph_workspace_bytes(P, n), dtype=torch.uint8, device=DEV)
    S.sph_bin_cells(P, n, src, dst, key, perm, start, ws)
    rho_in = dst.rho.cpu().numpy().astype(np.float64)
    S.sph_mdbc(P, n, dst, key, start, ws)
    torch.cuda.synchronize()
    typ = dst.type.cpu().numpy()
    rho_o, _ = oracle.mdbc(cp, dst.pos.cpu().numpy(), dst.vel.cpu().numpy().astype(np.float64),
                           rho_in, typ, dst.normal.cpu().numpy())
    rho_g = dst.rho.cpu().numpy().astype(np.float64)
    walls = typ != cases.FLUID
    assert walls.sum() > 0
    assert np.abs(rho_g - rho_o)[walls].max() <= 2e-4
    assert np.array_equal(rho_g[~walls], rho_in[~walls])
