"""LDS of the hexahedral walk at the upper end of its range: an FP64 row of five
elements on 24^3 velocities (68,016 bytes, above 64 KiB), and forced rows of 16 on
a grid whose chunks read 44 columns (131,072 bytes of y traces and 36,032 beside
them, more than a compute unit has), which are cut to what fits. Bits of tiles of
one element."""
import sys

import pytest

from paper_2308_06196_amd import workloads as wl
from tests.helpers import initial_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 2])
@pytest.mark.parametrize("nelem,nvel,tile", [((5, 1, 1), (24, 24, 24), "5x1"),
                                             ((16, 2, 1), (80, 4, 4), "16x2")])
def test_wide_rows(monkeypatch, nelem, nvel, tile, precision):
    import torch

    from paper_2308_06196_amd import bgk
    print("[case] hex walk LDS", nelem, nvel, tile, ["fp64", "", "bf16"][precision], flush=True)
    sys.stdout.flush()
    pb = wl.problem(3, 3, list(nelem), [0.0] * 3, [6.3] * 3, list(nvel), [-5.0] * 3, [5.0] * 3,
                    1e-2)
    f0 = torch.from_numpy(initial_state(pb, "tgv3d", seed=5, amp=0.1)).to("cuda:0")
    got = []
    for t in (tile, "1x1"):
        monkeypatch.setenv("BGK_WALK_TILE", t)
        s = bgk.Solver(pb, precision=precision)
        s.set_state(f0)
        s.rk3_step(1e-3, 1)
        got.append((s.get_state(), s.moments()))
        assert s.diagnostics()["newton_fail"] == 0
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
