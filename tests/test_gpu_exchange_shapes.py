"""Exchange kernels and Maxwellian sampler over the shapes their launches choose:
1, 4 and 16 nodes per lane (few entries, from 4e5, from 4e6), work-groups of 256
velocities and, where those leave gaps (8, 27, 64, 288, 600 velocities), lanes that
run on into the next nodes; node counts that do not divide, and host buffers staged
in windows. States come back bit for bit (FP32 storage rounded), sampled
Maxwellians match numpy's to rounding."""
import sys

import numpy as np
import pytest

from paper_2308_06196_amd import workloads as wl

pytestmark = pytest.mark.gpu

# nelem (p = 2 line elements), velocities
CASES = [(5, (2, 2, 2)), (16667, (2, 2, 2)), (166669, (2, 2, 2)), (4999, (3, 3, 3)), (49999, (3, 3, 3)),
         (2083, (4, 4, 4)), (20837, (4, 4, 4)), (463, (6, 6, 8)), (4631, (6, 6, 8)),
         (523, (16, 16, 1 + 1)), (2609, (16, 16, 2)), (223, (10, 10, 6)), (2227, (10, 10, 6)),
         (31, (17, 17, 17)), (277, (17, 17, 17))]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ne,nvel", CASES)
def test_round_trip_and_sampling(ne, nvel, precision):
    import torch

    from paper_2308_06196_amd import bgk
    print("[case] exchange shape", ne, nvel, precision, flush=True)
    sys.stdout.flush()
    pb = wl.problem(1, 2, [ne], [0.0], [1.0], list(nvel), [-4.0] * 3, [4.0] * 3, 1e-2)
    s = bgk.Solver(pb, precision=precision)
    rng = np.random.default_rng(ne)
    f = rng.uniform(0.0, 1.0, s.shape)
    want = f if precision == 0 else f.astype(np.float32).astype(np.float64)
    s.set_state(torch.from_numpy(f).to("cuda:0"))
    guard = torch.full((f.size + 512,), -7.0, dtype=torch.float64, device="cuda:0")
    out = guard[256:-256].view(s.shape)
    assert np.array_equal(s.get_state(out).cpu().numpy(), want)
    assert bool((guard[:256] == -7.0).all()) and bool((guard[-256:] == -7.0).all())
    s.set_state(np.ascontiguousarray(f))  # host: staged in windows
    assert np.array_equal(s.get_state(np.empty(s.shape)), want)
    u, _ = s.velocity_grid()
    prim = np.column_stack([rng.uniform(0.5, 1.5, s.nx), rng.uniform(-0.5, 0.5, (s.nx, 3)),
                            rng.uniform(0.7, 1.3, s.nx)])
    s.set_maxwellian(prim)
    got = s.get_state().cpu().numpy().reshape(s.nx, -1)
    norm = (prim[:, 0] / (2 * np.pi * prim[:, 4]) ** 1.5)[:, None]
    d2 = sum((u[None, :, c] - prim[:, None, 1 + c]) ** 2 for c in range(3))
    g = norm * np.exp(-d2 / (2 * prim[:, 4:5]))
    tol = 1e-13 if precision == 0 else 1.2e-7
    assert float(np.abs(got - g).max()) <= tol * float(g.max())
