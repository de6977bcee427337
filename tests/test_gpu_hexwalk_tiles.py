"""Tiles that the hexahedral walk chooses by itself on small meshes: velocity
chunks of one octant (8^3) and of several (7 x 5 x 6, 13 x 4 x 4), fewer and more
elements than the device has work-groups for, rows that five elements do and do not
divide. The results must be those of tiles of one element, bit for bit."""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2308_06196_amd import workloads as wl
from tests.helpers import initial_state, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("nelem,nvel", [((1, 1, 1), (7, 5, 6)), ((2, 3, 1), (8, 8, 8)),
                                        ((7, 2, 3), (13, 4, 4)), ((11, 6, 4), (7, 5, 6)),
                                        ((10, 9, 8), (8, 8, 8))])
def test_chosen_tile(monkeypatch, nelem, nvel, precision):
    import torch

    from paper_2308_06196_amd import bgk
    print("[case] hex walk tile", nelem, nvel, ["fp64", "", "bf16"][precision], flush=True)
    sys.stdout.flush()
    pb = wl.problem(3, 3, list(nelem), [0.0] * 3, [2 * np.pi] * 3, list(nvel), [-5.0] * 3,
                    [5.0] * 3, 1e-2)
    f0 = torch.from_numpy(initial_state(pb, "tgv3d", seed=5, amp=0.2)).to("cuda:0")
    got = []
    for tile in (None, "1x1"):
        if tile is None:
            monkeypatch.delenv("BGK_WALK_TILE", raising=False)
        else:
            monkeypatch.setenv("BGK_WALK_TILE", tile)
        s = bgk.Solver(pb, precision=precision)
        s.set_state(f0)
        s.rk3_step(1e-3, 2)
        got.append((s.get_state(), s.moments(), s.diagnostics()))
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
    assert got[0][2] == got[1][2] and got[0][2]["newton_fail"] == 0
    if nelem == (2, 3, 1) and precision == 0:
        ref, _ = orc.rk3_step(oracle_problem(pb), f0.cpu().numpy(), 1e-3, 2)
        assert float(np.abs(got[0][0].cpu().numpy() - ref).max()) < 1e-12 * float(np.abs(ref).max())
