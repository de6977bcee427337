"""Equilibrium solve on velocity grids with one or two long axes, whose sums run
over the three axes together up to the shortest one and over each rest alone:
every axis as the long one, rests that do and do not fill a team, teams of 16, 4
and 2 lanes (few, some and many nodes). One step against the FP64 oracle on a few
elements; on many copies of one element the result of the few to rounding; the
collision term's moments vanish; batch members get the bits they get alone."""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2308_06196_amd import workloads as wl
from tests.helpers import oracle_problem

pytestmark = pytest.mark.gpu

GRIDS = [(34, 8, 8), (8, 61, 9), (7, 8, 50), (33, 32, 7), (100, 8, 8)]


def _problem(ne, nvel):
    return wl.problem(1, 3, [ne], [0.0], [float(ne)], list(nvel), [-6.0] * 3, [6.0] * 3, 1e-2)


def _prim(ne):
    rng = np.random.default_rng(3)
    one = np.column_stack([rng.uniform(0.5, 1.5, 8), rng.uniform(-0.3, 0.3, (8, 3)),
                           rng.uniform(0.8, 1.2, 8)])  # two elements, repeated
    return np.ascontiguousarray(np.tile(one, (ne // 2, 1)))


@pytest.mark.parametrize("nvel", GRIDS)
def test_long_axes(nvel):
    import torch

    from paper_2308_06196_amd import bgk
    print("[case] newton split", nvel, flush=True)
    sys.stdout.flush()
    pb = _problem(4, nvel)
    pr = oracle_problem(pb)
    f0 = orc.maxwellian(pr, _prim(4))
    dt = orc.stable_dt(pr, f0, 0.1)
    ref, _ = orc.rk3_step(pr, f0, dt, 1)
    first = None
    for ne in (4, 2048, 32768):  # teams of 16, 4, 2
        s = bgk.Solver(_problem(ne, nvel))
        s.set_maxwellian(_prim(ne))
        Cm, Q = s.collision_moments(), s.moments()
        # C = (g - f) / tau with 1 / tau = P / mu < 300
        assert float(Cm.abs().max()) < 1e-12 * 300 * float(Q.abs().max())
        s.rk3_step(dt, 1)
        f = s.get_state()
        assert s.diagnostics()["newton_fail"] == 0
        if first is None:
            first = f
            assert float(np.abs(f.cpu().numpy() - ref).max()) < 1e-12 * float(np.abs(ref).max())
        else:
            d = f.view(ne // 4, *first.shape) - first
            assert float(d.abs().max()) < 1e-13 * float(first.abs().max()), ne
        del s, f
        torch.cuda.empty_cache()


def test_batch_members():
    import torch

    from paper_2308_06196_amd import bgk
    stream = torch.cuda.current_stream()
    cases = [(6, (16, 16, 16)), (5, (64, 8, 8)), (2048, (7, 8, 50)), (4, (8, 61, 9))]
    print("[case] newton split batch", flush=True)
    want, members = [], []
    for ne, nvel in cases:
        for alone in (True, False):
            s = bgk.Solver(_problem(ne, nvel))
            s.set_maxwellian(np.ascontiguousarray(_prim(ne + ne % 2)[: ne * 4]))
            if alone:
                s.rk3_step(1e-3, 3)
                want.append(s.get_state().cpu().numpy())
            else:
                members.append(s)
    b = bgk.Batch(stream, 8)
    for s in members:
        b.add(s, 1e-3, 3)
    b.step(3)
    done = b.poll()
    assert len(done) == len(members) and all(e is None for _, e in done)
    for s, w in zip(members, want):
        assert np.array_equal(s.get_state().cpu().numpy(), w)
    b.close()
