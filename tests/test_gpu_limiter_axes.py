"""Positivity limiter on hexahedra whose state varies along every axis.

The limiter contracts a slice towards its Gauss-weighted mean over all (p+1)^3
nodes; a jump along one axis only (tests/test_gpu_hex_limiter.py) does not
tell a mean over the wrong nodes from the right one. Here the state has jumps
along x, y and z: FP64 states and contraction counts against the oracle for
every kernel family, the elements' means kept by the limiter through the
conserved total mass (periodic box, collisions on).
"""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2308_06196_amd import workloads as wl
from tests.helpers import oracle_problem, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("order", [1, 2, 3])
def test_limiter_with_jumps_along_every_axis(order, precision):
    import torch

    from paper_2308_06196_amd import bgk
    print("[case] limiter axes", order, bgk.PRECISION_NAME[precision], flush=True)
    sys.stdout.flush()
    pb = wl.problem(3, order, [3, 3, 3], [0.0] * 3, [1.0] * 3, [8] * 3, [-6.0] * 3, [6.0] * 3, 1e-3)
    pr = oracle_problem(pb)
    x = orc.node_coords(pr)
    prim = np.zeros((len(x), 5))
    prim[:, 0] = np.prod(np.where(x < 0.45, 1.0, 0.3), axis=1)
    prim[:, 4] = 0.8 + 0.2 * (x[:, 1] < 0.45) * (x[:, 2] < 0.45)
    f0 = orc.maxwellian(pr, prim)
    dt = orc.stable_dt(pr, f0, 0.1)
    ref, d_orc = orc.rk3_step(pr, f0, dt, 3)
    assert d_orc["limiter_hits"] > 1000
    s = bgk.Solver(pb, precision=precision)
    s.set_state(torch.from_numpy(f0).to("cuda:0"))
    s.rk3_step(dt, 3)
    f, d = s.get_state().cpu().numpy(), s.diagnostics()
    scale = float(np.abs(ref).max())
    _, w1 = orc.gauss_legendre(order + 1)
    W = np.tile(np.einsum("k,j,i->kji", w1, w1, w1).ravel(), s.ne)
    Q = s.moments().cpu().numpy()
    mass, mass0 = float((W * Q[:, 0]).sum()), float((W * orc.moments(pr, f0)[:, 0]).sum())
    if precision == 0:
        assert rel_max(f, ref) < 1e-12
        assert d["limiter_hits"] == d_orc["limiter_hits"]
        assert d["limiter_bad"] == d_orc["limiter_bad"]
        assert abs(mass - mass0) < 1e-13 * mass0
    elif precision == 1:
        assert rel_max(f, ref) < 1e-5
        assert abs(mass - mass0) < 1e-6 * mass0
    else:  # the increment rounding of the parity tests
        traj, inc = [f0], 0.0
        for _ in range(3):
            L, _ = orc.residual(pr, traj[-1])
            inc = max(inc, dt * float(np.abs(L).max()))
            traj.append(orc.rk3_step(pr, traj[-1], dt, 1)[0])
        assert float(np.abs(f - ref).max()) < 1e-5 * scale + 6.0 * 2.0 ** -8 * inc
    assert d["limiter_hits"] > 1000
