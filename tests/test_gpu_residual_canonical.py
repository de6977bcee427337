"""Residual of a device array read in place (canonical layout).

bgk_residual and bgk_residual_noalloc read a device f_in where it is, in
lexicographic velocity order, unless r_out overlaps it; then f_in is copied to
the internal layout first, as for host buffers. Every kernel that reads the
canonical array is checked against the FP64 oracle (the parity tests' bound,
relative to max|T| + max|C|) and against the in-place call (r_out = f_in),
which takes the copying path: the two differ only by the order of the moment
sums (1e-13 of the same scale in FP64; FP32 arithmetic 1e-6). Chunks that wrap
rows, planes or neither; one velocity row; periodic, specular and diffuse
boundaries; collisions off.
"""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2308_06196_amd import workloads as wl
from tests.helpers import initial_state, oracle_problem

pytestmark = pytest.mark.gpu


def _problem(dim, order, nelem, nvel, walls=0, mu=1e-2):
    bc = [(walls, walls)] * dim
    pb = wl.problem(dim, order, list(nelem), [0.0] * dim, [1.0] * dim, list(nvel), [-6.0] * 3,
                    [6.0] * 3, mu, bc=bc)
    pb["wall_theta"] = [(0.9, 1.1), (1.2, 0.8), (1.0, 1.0)]
    if mu == 0.0:
        pb["mu_ref"] = 0.0
    return pb


CASES = {}
for _p in (1, 2, 3):
    CASES[f"d1p{_p}"] = _problem(1, _p, (5,), (9, 8, 7), 1)
    CASES[f"d1p{_p}_diffuse"] = _problem(1, _p, (3,), (8, 8, 8), 2)
    CASES[f"d2p{_p}"] = _problem(2, _p, (3, 2), (7, 6, 9))
    CASES[f"d2p{_p}_diffuse"] = _problem(2, _p, (2, 3), (8, 7, 6), 2)
    CASES[f"d3p{_p}"] = _problem(3, _p, (2, 3, 2), (7, 8, 6), 1)
CASES["long_rows"] = _problem(2, 3, (2, 2), (300, 3, 3), 1, mu=0.0)
CASES["long_planes"] = _problem(2, 1, (2, 2), (20, 30, 4))
CASES["small"] = _problem(1, 2, (2,), (5, 6, 5))
CASES["free"] = _problem(3, 3, (2, 1, 2), (5, 6, 4), 0, mu=0.0)


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("name", list(CASES))
def test_canonical_residual(name, precision):
    import torch

    from paper_2308_06196_amd import bgk
    pb = CASES[name]
    diffuse = any(s == 2 for b in pb["bc"] for s in b)
    if precision == 2 and diffuse:
        pytest.skip("diffuse walls are built for FP64 and FP32 storage")
    print("[case] canonical residual", name, ["fp64", "fp32", "bf16"][precision], flush=True)
    sys.stdout.flush()
    pr = oracle_problem(pb)
    f = initial_state(pb, ["", "sod1d", "box2d", "tgv3d"][pb["dim"]], seed=len(name), amp=0.2)
    if precision:  # FP32 storage rounds f_in first
        f = f.astype(np.float32).astype(np.float64)
    L, _ = orc.residual(pr, f)
    scale = float(np.abs(orc.transport(pr, f)).max())
    if pb["mu_ref"] > 0.0:
        scale += float(np.abs(orc.collision(pr, f)[0]).max())
    tol = 1e-12 if precision == 0 else 1e-5
    t = torch.from_numpy(np.ascontiguousarray(f)).to("cuda:0")
    keep = t.clone()
    s = bgk.Solver(pb, precision=precision)
    s.set_state(t)
    state = s.get_state().clone()
    r = s.residual(t)
    assert torch.equal(t, keep) and torch.equal(s.get_state(), state)  # inputs unchanged
    assert float(np.abs(r.cpu().numpy() - L).max()) < tol * scale
    both = s.residual(t, t).cpu().numpy()  # in place: through the copy
    assert float(np.abs(both - r.cpu().numpy()).max()) < (1e-13 if precision == 0 else 1e-6) * scale
    s.diagnostics()
    if not diffuse and precision < 2:
        n = bgk.residual_noalloc(pb, keep, precision=precision)
        assert torch.equal(n, r)
        m = keep.clone()
        bgk.residual_noalloc(pb, m, out=m, precision=precision)
        assert np.array_equal(m.cpu().numpy(), both)
