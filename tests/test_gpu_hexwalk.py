"""Walking stage kernel of p = 3 hexahedra (FP64 storage, BF16 increments).

A work-group walks a tile of elements of one z-layer in the upwind directions
of its velocity chunk and hands the x and y outflow traces from element to
element; at tile entries, and for velocities of the other sign, the traces
come from the neighbour's nodes by the same sum. BGK_WALK_TILE=XxY (read when
a solver is created) forces the tile. Checked against the FP64 oracle after
two RK3 steps (FP64 1e-12 max|f|; BF16 increments within the bound of the
parity tests), and bit for bit between tiles:

  * tiles of one element (nothing carried), tiles that do and do not divide
    the mesh, and the whole mesh;
  * grids whose 64-velocity chunks are uniform in the signs (8^3), straddle
    sign changes (7 x 5 x 6), are mostly padding (3^3) and need more row
    entries than the first batch of row loads (30 x 29 x 2);
  * periodic and specular boundaries on every axis, a single element per axis,
    and collisions off.
"""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2308_06196_amd import workloads as wl
from tests.helpers import initial_state, oracle_problem, rel_max

pytestmark = pytest.mark.gpu

# nelem, nvel, specular walls, tiles, collisions
CASES = {
    "uniform": ((5, 3, 2), (8, 8, 8), False, ("1x1", "2x2", "4x3", "5x3"), True),
    "straddling": ((4, 5, 3), (7, 5, 6), False, ("1x1", "3x2", "4x5"), True),
    "walls": ((3, 4, 2), (8, 6, 7), True, ("1x1", "2x3", "3x4"), True),
    "padding": ((3, 2, 2), (3, 3, 3), False, ("1x1", "3x2"), False),
    "rows": ((2, 2, 1), (30, 29, 2), False, ("1x1", "2x2"), False),
    "rows_collide": ((2, 1, 1), (30, 29, 4), False, ("1x1", "2x1"), True),
    "one_element": ((1, 1, 1), (8, 8, 8), True, ("1x1",), True),
    "collisionless": ((4, 3, 2), (8, 7, 6), True, ("1x1", "3x3", "4x3"), False),
}


def _problem(nelem, nvel, walls, collide):
    bc = [(1, 1)] * 3 if walls else None
    pb = wl.problem(3, 3, list(nelem), [0.0] * 3, [2 * np.pi] * 3, list(nvel), [-5.0] * 3,
                    [5.0] * 3, 1e-2, bc=bc)
    if not collide:
        pb["mu_ref"] = 0.0
    return pb


def _bf16_bound(pr, f0, dt, n):
    # as in test_gpu_parity: 1e-5 max|f| + 2 n 2^-8 max_k dt |L(f^k)|
    traj, inc = [f0], 0.0
    for _ in range(n):
        L, _ = orc.residual(pr, traj[-1])
        inc = max(inc, dt * float(np.abs(L).max()))
        traj.append(orc.rk3_step(pr, traj[-1], dt, 1)[0])
    return traj[-1], 1e-5 * float(np.abs(traj[-1]).max()) + 2.0 * n * 2.0 ** -8 * inc


@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("name", list(CASES))
def test_walk_matches_oracle_for_every_tile(monkeypatch, name, precision):
    import torch

    from paper_2308_06196_amd import bgk
    nelem, nvel, walls, tiles, collide = CASES[name]
    pb = _problem(nelem, nvel, walls, collide)
    print("[case] hex walk", name, ["fp64", "fp32", "bf16"][precision], flush=True)
    sys.stdout.flush()
    pr = oracle_problem(pb)
    f0 = initial_state(pb, "tgv3d", seed=17, amp=0.2)
    dt = orc.stable_dt(pr, f0, 0.1)
    if precision == 2:
        ref, bound = _bf16_bound(pr, f0, dt, 2)
    else:
        ref, _ = orc.rk3_step(pr, f0, dt, 2)
        bound = 1e-12 * float(np.abs(ref).max())
    first = None
    for tile in (None,) + tiles:
        if tile is None:
            monkeypatch.delenv("BGK_WALK_TILE", raising=False)
        else:
            monkeypatch.setenv("BGK_WALK_TILE", tile)
        s = bgk.Solver(pb, precision=precision)
        s.set_state(torch.from_numpy(np.ascontiguousarray(f0)).to("cuda:0"))
        s.rk3_step(dt, 2)
        f = s.get_state().cpu().numpy()
        Q = s.moments().cpu().numpy()
        d = s.diagnostics()
        assert d["newton_fail"] == 0 and d["stages"] == 6
        assert float(np.abs(f - ref).max()) <= bound, tile
        # the stage's moment partials against the oracle's moments of its own state
        assert rel_max(Q, orc.moments(pr, f)) < 1e-13
        if first is None:
            first = f, d
        else:
            assert np.array_equal(f, first[0]), tile
            assert d["limiter_hits"] == first[1]["limiter_hits"], tile
