"""sph_interact_noalloc (the interaction without a workspace, for callers that
cannot allocate) against sph_interact on the same sorted state: the same
kernels, so every output must be identical.  Two calls in a row, the second
with a smaller input, so that what the first call left in the library's
device array cannot leak into the second."""
import numpy as np
import pytest
import torch

from paper_2104_00537_amd import cases

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2104_00537_amd import sph as S

DEV = "cuda:0"


def _say(*a):
    print(*a, flush=True)


def _binned(case, seed):
    """The case binned by sph_bin_cells, with velocities of a developed flow
    (so that every term of the pass is non-zero)."""
    rng = np.random.default_rng(seed)
    case.vel[:] = rng.uniform(-0.5, 0.5, case.vel.shape).astype(np.float32)
    P = S.make_params(case.params)
    n = case.n
    src = S.DeviceState.from_case(case, DEV)
    dst = S.DeviceState.empty(case.params.dim, n, DEV)
    key = torch.empty((n,), dtype=torch.int32, device=DEV)
    perm = torch.empty((n,), dtype=torch.int32, device=DEV)
    start = torch.empty((case.params.ncell_total() + 1,), dtype=torch.int32, device=DEV)
    ws = torch.zeros(S.sph_workspace_bytes(P, n), dtype=torch.uint8, device=DEV)
    S.sph_bin_cells(P, n, src, dst, key, perm, start, ws)
    return P, n, dst, key, start, ws


def _outputs(dim, n):
    return (torch.full((dim, n), float("nan"), dtype=torch.float32, device=DEV),
            torch.full((n,), float("nan"), dtype=torch.float32, device=DEV),
            torch.full((n,), float("nan"), dtype=torch.float32, device=DEV),
            torch.full((n,), -1, dtype=torch.int32, device=DEV))


def _compare(case, seed, flags):
    P, n, dst, key, start, ws = _binned(case, seed)
    dim = case.params.dim
    a_ace, a_arho, a_visc, a_nbr = _outputs(dim, n)
    S.sph_interact(P, n, dst, key, start, a_ace, a_arho, ws, visc=a_visc, nbr=a_nbr, flags=flags)
    b_ace, b_arho, b_visc, b_nbr = _outputs(dim, n)
    S.sph_interact_noalloc(P, n, dst, key, start, b_ace, b_arho, visc=b_visc, nbr=b_nbr,
                           flags=flags)
    torch.cuda.synchronize()
    assert S.sph_read_error(ws) == 0
    assert torch.isfinite(a_ace).all() and torch.isfinite(a_arho).all()
    assert torch.equal(a_ace, b_ace)
    assert torch.equal(a_arho, b_arho)
    assert torch.equal(a_visc, b_visc)
    assert torch.equal(a_nbr, b_nbr)
    assert int(b_nbr.max()) > 0


@pytest.mark.parametrize("flags", [0, "diag", "one_lane"])
def test_noalloc_matches_interact_on_two_calls(flags):
    fl = {0: 0, "diag": S.SPH_DIAG_COUNT_F64, "one_lane": S.SPH_INTERACT_ONE_LANE}[flags]
    big = cases.dam_break_3d(dp=0.6 / 60, cell_div=2, x_sub=4)   # one lane per target
    small = cases.dam_break_2d(dp=0.02, cell_div=2, x_sub=4)     # four lanes per target
    assert big.n > 131072 >= small.n
    _say(f"noalloc: flags={flags} n={big.n} then n={small.n}")
    _compare(big, 1, fl)
    _compare(small, 2, fl)


def test_noalloc_rejects_sizes_beyond_its_array():
    case = cases.dam_break_2d(dp=0.02)
    P = S.make_params(case.params)
    n = S.SPH_NOALLOC_MAX_N + 1
    x = torch.zeros(1, dtype=torch.float32, device=DEV)
    st = S.DeviceState(pos=torch.zeros((2, 1), dtype=torch.float64, device=DEV),
                       vel=torch.zeros((2, 1), dtype=torch.float32, device=DEV),
                       rho=x, type=torch.zeros(1, dtype=torch.uint8, device=DEV))
    k = torch.zeros(1, dtype=torch.int32, device=DEV)
    with pytest.raises(S.SphError, match="invalid argument"):
        S.sph_interact_noalloc(P, n, st, k, k, x, x)


@pytest.mark.parametrize("diag", [False, True])
def test_noalloc_matches_interact_with_one_lane_by_size(diag):
    """A case above the 266,240 particles up to which 3-D cases get several lanes
    per target: the one-lane kernels, without a flag that asks for them."""
    big = cases.dam_break_3d(dp=0.6 / 70, cell_div=2, x_sub=4)
    assert 266_240 < big.n <= S.SPH_NOALLOC_MAX_N
    _say(f"noalloc: diag={diag} n={big.n}")
    _compare(big, 3, S.SPH_DIAG_COUNT_F64 if diag else 0)
