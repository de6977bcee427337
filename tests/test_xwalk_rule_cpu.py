"""Where the x walk is chosen, on the host: the lengths follow the measurements its
rule quotes (per element where runs were slower, by runs of that length where they
were faster). The check program includes the rule's own source and is built with
hipcc for the host only."""
import os
import subprocess
import tempfile

import pytest

from tests.test_slot_order_cpu import HERE, ROOT, _hipcc

# dim, p, elements, velocities, precision: run length
CASES = [
    # quadrilaterals: equal runs, enough pairs, carried waves
    ((2, 3, (32, 32, 1), (24, 24, 24), 1), 8), ((2, 3, (32, 64, 1), (16, 16, 16), 1), 8),
    ((2, 3, (32, 64, 1), (16, 16, 12), 1), 0), ((2, 3, (32, 64, 1), (16, 16, 12), 2), 8),
    ((2, 3, (32, 64, 1), (17, 17, 17), 2), 8), ((2, 3, (32, 64, 1), (13, 13, 13), 2), 0),
    ((2, 3, (32, 64, 1), (14, 14, 14), 2), 0), ((2, 3, (32, 64, 1), (12, 12, 12), 2), 0),
    # runs of unequal length
    ((2, 3, (45, 29, 1), (21, 22, 17), 1), 0), ((2, 3, (45, 29, 1), (24, 24, 24), 1), 8),
    ((2, 3, (45, 29, 1), (21, 22, 17), 2), 8), ((2, 3, (45, 29, 1), (18, 18, 18), 2), 0),
    ((2, 3, (13, 37, 1), (22, 22, 22), 2), 0), ((2, 3, (24, 24, 1), (8, 8, 8), 2), 0),
    # p = 2 hexahedra with increments
    ((3, 2, (20, 20, 20), (20, 20, 20), 2), 20), ((3, 2, (6, 6, 6), (16, 16, 16), 2), 2),
    ((3, 2, (3, 20, 20), (9, 9, 9), 2), 0), ((3, 2, (3, 20, 20), (12, 12, 12), 2), 3),
    ((3, 2, (5, 7, 9), (13, 11, 9), 2), 0), ((3, 2, (5, 7, 9), (12, 12, 12), 2), 2),
    ((3, 2, (1, 16, 16), (20, 20, 20), 2), 0),
    # p = 1 hexahedra
    ((3, 1, (16, 16, 16), (16, 16, 16), 0), 16), ((3, 1, (4, 9, 6), (16, 16, 16), 0), 0),
    ((3, 1, (14, 9, 12), (15, 15, 15), 1), 0),
    # not built
    ((2, 3, (32, 32, 1), (24, 24, 24), 0), 0), ((1, 3, (512, 1, 1), (24, 24, 24), 1), 0),
]


def test_run_lengths(monkeypatch):
    monkeypatch.delenv("BGK_XWALK", raising=False)
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not found")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "xwalk_rule_check")
        subprocess.run([hipcc, "-std=c++17", "-O1", "--offload-host-only",
                        "-Wno-unused-function", "-I", os.path.join(ROOT, "include"),
                        os.path.join(HERE, "xwalk_rule_check.cpp"), "-o", exe],
                       check=True, capture_output=True, timeout=300)
        text = "\n".join(" ".join(map(str, (c[0], c[1], *c[2], *c[3], c[4]))) for c, _ in CASES)
        r = subprocess.run([exe], input=text + "\n", capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    got = [int(x) for x in r.stdout.split()]
    bad = [(c, want, g) for (c, want), g in zip(CASES, got) if g != want]
    assert len(got) == len(CASES) and not bad, bad
