"""Exchange between the canonical and the internal layout, and the Maxwellian
sampler, at the edges of their work items (16 nodes x 256 velocities): node
counts below, at and beyond 16, elements that straddle a work item, velocity
counts below, at and beyond 256, and host buffers staged in windows that begin
and end inside a node. FP64 states come back bit for bit, FP32 storage rounded
to FP32; sampled Maxwellians match numpy's to rounding."""
import sys

import numpy as np
import pytest

from paper_2308_06196_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [(1, 1, (1,), (3, 2, 2)), (1, 2, (5,), (16, 16, 1 + 1)), (1, 3, (4,), (8, 8, 4)),
         (1, 2, (11,), (17, 5, 4)), (2, 2, (3, 2), (7, 9, 5)), (2, 3, (2, 1), (16, 16, 16)),
         (3, 1, (3, 1, 2), (5, 7, 9)), (3, 2, (1, 2, 1), (8, 8, 8)), (3, 3, (2, 1, 1), (6, 5, 11))]


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("dim,order,nelem,nvel", CASES)
def test_state_round_trip(dim, order, nelem, nvel, precision):
    import torch

    from paper_2308_06196_amd import bgk
    print("[case] exchange", dim, order, nelem, nvel, precision, flush=True)
    sys.stdout.flush()
    pb = wl.problem(dim, order, list(nelem), [0.0] * dim, [1.0] * dim, list(nvel), [-4.0] * 3,
                    [4.0] * 3, 1e-2)
    s = bgk.Solver(pb, precision=precision)
    rng = np.random.default_rng(dim * 100 + order)
    f = rng.uniform(0.0, 1.0, s.shape)
    want = f if precision == 0 else f.astype(np.float32).astype(np.float64)
    s.set_state(torch.from_numpy(f).to("cuda:0"))
    assert np.array_equal(s.get_state().cpu().numpy(), want)
    assert np.array_equal(s.get_state(np.empty(s.shape)), want)  # host: staged in windows
    s.set_state(np.ascontiguousarray(f))
    assert np.array_equal(s.get_state().cpu().numpy(), want)
    u, _ = s.velocity_grid()
    prim = np.column_stack([rng.uniform(0.5, 1.5, s.nx), rng.uniform(-0.5, 0.5, (s.nx, 3)),
                            rng.uniform(0.7, 1.3, s.nx)])
    s.set_maxwellian(prim)
    d2 = ((u[None] - prim[:, None, 1:4]) ** 2).sum(-1)
    g = (prim[:, 0] / (2 * np.pi * prim[:, 4]) ** 1.5)[:, None] * np.exp(-d2 / (2 * prim[:, 4:5]))
    got = s.get_state().cpu().numpy().reshape(g.shape)
    tol = 1e-13 if precision == 0 else 1.2e-7
    assert float(np.abs(got - g).max()) <= tol * float(g.max())
