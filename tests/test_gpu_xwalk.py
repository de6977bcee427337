"""Stage kernel that walks runs of elements along x (one lane per velocity).

p = 3 quadrilaterals in FP32 and with BF16 increments, p = 1 hexahedra in every
precision and p = 2 hexahedra with BF16 increments walk once the mesh is large enough; BGK_XWALK
(read when a solver is created) forces the run length (0: one work-group per
element). The sums and their order are those of the per-element kernels, so
every length must give their bits and counters: runs of one element, lengths
that do and do not divide the row, the whole row; velocity chunks that are
uniform in the signs, straddle sign changes or are mostly padding, and more row
entries than the first batch of row loads; periodic and specular boundaries;
collisions on and off; the limiter contracting slices across the walk.
"""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2308_06196_amd import workloads as wl
from tests.helpers import initial_state, oracle_problem

pytestmark = pytest.mark.gpu

FAMILIES = [(2, 3, 1), (2, 3, 2), (3, 1, 0), (3, 1, 1), (3, 1, 2), (3, 2, 2)]
# nelem, nvel, walls, collisions, run lengths
SHAPES = {
    "uniform": ((5, 3, 2), (8, 8, 8), 0, True, (1, 2, 3, 5)),
    "straddling": ((4, 2, 3), (11, 9, 7), 0, True, (1, 3, 4)),
    "walls": ((3, 4, 2), (10, 8, 6), 1, True, (1, 2, 3)),
    "padding": ((3, 2, 2), (5, 4, 4), 0, True, (2, 3)),
    "rows": ((3, 2, 1), (40, 30, 8), 0, True, (1, 3)),
    "one": ((1, 1, 1), (8, 8, 8), 1, True, (1,)),
    "free": ((4, 3, 2), (8, 7, 6), 1, False, (1, 3, 4)),
}


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("dim,order,precision", FAMILIES)
def test_walk_gives_the_bits_of_single_elements(monkeypatch, dim, order, precision, name):
    import torch

    from paper_2308_06196_amd import bgk
    nelem, nvel, walls, collide, lengths = SHAPES[name]
    print("[case] x walk", f"d{dim}p{order}", ["fp64", "fp32", "bf16"][precision], name, flush=True)
    sys.stdout.flush()
    pb = wl.problem(dim, order, list(nelem)[:dim], [0.0] * dim, [1.0] * dim, list(nvel),
                    [-6.0] * 3, [6.0] * 3, 1e-2, bc=[(walls, walls)] * dim)
    if not collide:
        pb["mu_ref"] = 0.0
    pr = oracle_problem(pb)
    # a strong modulation: some slices turn negative within the steps
    f0 = initial_state(pb, "box2d" if dim == 2 else "tgv3d", seed=29, amp=0.8)
    dt = orc.stable_dt(pr, f0, 0.3)
    first = None
    for length in (0,) + lengths:
        monkeypatch.setenv("BGK_XWALK", str(length))
        s = bgk.Solver(pb, precision=precision)
        s.set_state(torch.from_numpy(np.ascontiguousarray(f0)).to("cuda:0"))
        s.rk3_step(dt, 2)
        f, Q = s.get_state().cpu().numpy(), s.moments().cpu().numpy()
        d = s.diagnostics()
        assert d["newton_fail"] == 0 and d["stages"] == 6
        if first is None:
            first = f, Q, d
            assert name == "one" or d["limiter_hits"] > 0
        assert np.array_equal(f, first[0]), length
        assert np.array_equal(Q, first[1]), length
        assert d == first[2], length
