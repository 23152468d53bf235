"""The counting sort of the binning at the sizes where it can go wrong: inputs
of one particle, of whole wavefronts, blocks and scan tiles and one beside;
grids of one cell, of a scan tile of cells and one beside, and of more cells
than one tile per scan block; cells of hundreds of members; particles excluded
before and by the call, scattered over the input; slots of a batch that begin
inside a wavefront.  Keys, permutation and ranges are the oracle's (a stable
sort), bit for bit, in two calls on one workspace."""
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


def _case(n, ncell, seed, excluded, outside):
    """n particles at random places of a 2-D grid of ncell cells, a share of
    them excluded before the call and a share outside the grid."""
    rng = np.random.default_rng(seed)
    p = cases.block_case(2, (4, 4)).params
    p = dataclasses.replace(p, ncell=(ncell[0], ncell[1], 1), origin=(0.0, 0.0, 0.0))
    size = np.array(ncell, np.float64)[:, None] * p.cell_size
    pos = rng.uniform(0.0, 1.0, (2, n)) * size * (1.0 - 1e-9)
    pos[0, rng.random(n) < outside] = -p.cell_size
    typ = rng.integers(0, 2, n).astype(np.uint8)
    typ[rng.random(n) < excluded] |= cases.EXCLUDED
    vel = rng.standard_normal((2, n)).astype(np.float32)
    return cases.Case(p, pos, vel, rng.uniform(990, 1010, n).astype(np.float32), typ)


def _reference(c):
    key = oracle.cell_keys(c.params, c.pos).astype(np.uint32)
    key[(c.type & cases.EXCLUDED) != 0] = c.params.ncell_total()
    perm = np.argsort(key, kind="stable").astype(np.uint32)
    return key[perm], perm


def _u32(t):
    return t.cpu().numpy().view(np.uint32)


GRIDS = [(1, (1, 1), 0.0, 0.0), (1, (1, 1), 1.0, 0.0), (63, (3, 3), 0.2, 0.1),
         (64, (5, 2), 0.0, 0.5), (65, (2048, 1), 0.1, 0.1), (256, (2047, 1), 0.1, 0.0),
         (257, (2049, 1), 0.3, 0.3), (700, (2, 1), 0.1, 0.1), (2049, (40, 50), 0.9, 0.05),
         (3000, (2100, 2100), 0.1, 0.1), (100000, (300, 200), 0.02, 0.02)]


@pytest.mark.parametrize("n,ncell,excluded,outside", GRIDS)
def test_counting_sort(n, ncell, excluded, outside):
    print("counting sort", n, ncell, excluded, outside, flush=True)
    ws = None
    for seed in (1, 2):
        c = _case(n, ncell, seed, excluded, outside)
        P = S.make_params(c.params)
        src = S.DeviceState.from_case(c, DEV)
        dst = S.DeviceState.empty(2, n, DEV)
        key, perm = (torch.full((n,), -1, dtype=torch.int32, device=DEV) for _ in range(2))
        total = c.params.ncell_total()
        start = torch.full((total + 1,), -1, dtype=torch.int32, device=DEV)
        if ws is None:
            ws = torch.zeros(S.sph_workspace_bytes(P, n), dtype=torch.uint8, device=DEV)
        S.sph_bin_cells(P, n, src, dst, key, perm, start, ws)
        rkey, rperm = _reference(c)
        assert np.array_equal(_u32(key), rkey)
        assert np.array_equal(_u32(perm), rperm)
        assert np.array_equal(_u32(start), oracle.cell_start(rkey, total))
        assert np.array_equal(dst.pos.cpu().numpy(), c.pos[:, rperm])
        assert np.array_equal(_u32(dst.id), rperm)


def test_counting_sort_of_a_batch():
    print("counting sort of a batch", flush=True)
    cs = [_case(65, (3, 3), 3, 0.2, 0.1), _case(1, (1, 1), 4, 1.0, 0.0),
          _case(130, (7, 5), 5, 0.5, 0.2), _case(900, (40, 60), 6, 0.1, 0.1),
          _case(300, (2, 2), 7, 0.0, 0.9)]
    params = [S.make_params(c.params) for c in cs]
    offs = np.concatenate([[0], np.cumsum([c.n for c in cs])])
    n = int(offs[-1])
    b, host = S.sph_batch_describe(params, offs)
    table = torch.from_numpy(host).to(DEV)
    b.table = table.data_ptr()
    src, dst = (S.DeviceState.empty(3, n, DEV) for _ in range(2))
    src.pos.zero_()
    src.vel.zero_()
    keys, perms, base = [], [], 0
    for c, o in zip(cs, offs):
        e = o + c.n
        for k, comp in ((0, 0), (2, 1)):
            src.pos[k, o:e] = torch.from_numpy(c.pos[comp]).to(DEV)
            src.vel[k, o:e] = torch.from_numpy(c.vel[comp]).to(DEV)
        src.rho[o:e] = torch.from_numpy(c.rho).to(DEV)
        src.type[o:e] = torch.from_numpy(c.type).to(DEV)
        rkey, rperm = _reference(c)
        keys.append(rkey + np.uint32(base))
        perms.append(rperm + np.uint32(o))
        base += c.params.ncell_total() + 1
    src.id.copy_(torch.arange(n, dtype=torch.int32))
    keys, perms = np.concatenate(keys), np.concatenate(perms)
    key, perm = (torch.full((n,), -1, dtype=torch.int32, device=DEV) for _ in range(2))
    start = torch.full((base + 1,), -1, dtype=torch.int32, device=DEV)
    ws = torch.zeros(S.sph_batch_workspace_bytes(b), dtype=torch.uint8, device=DEV)
    for _ in range(2):
        S.sph_batch_bin_cells(b, src, dst, key, perm, start, ws)
        assert np.array_equal(_u32(key), keys)
        assert np.array_equal(_u32(perm), perms)
        assert np.array_equal(_u32(start), oracle.cell_start(keys, base))
        assert np.array_equal(_u32(dst.id), perms)
