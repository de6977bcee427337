"""Where stages run several elements of a mesh row per work-group, on the host: the
choice follows the measurements its rule quotes. The check program includes the
rule's own source and is built with hipcc for the host only."""
import os
import subprocess
import tempfile

import pytest

from tests.test_slot_order_cpu import HERE, ROOT, _hipcc

FP64, FP32, BF16 = 0, 1, 2
# dim, p, elements, velocities, precision: several elements per work-group
CASES = [
    ((1, 2, (32, 1, 1), (16,) * 3, FP64), 0), ((1, 1, (512, 1, 1), (8,) * 3, FP64), 1),
    ((1, 3, (487, 1, 1), (22, 23, 21), BF16), 1), ((1, 1, (64, 1, 1), (16,) * 3, FP32), 1),
    # p = 1 quadrilaterals: runs of four
    ((2, 1, (1, 60, 1), (20,) * 3, FP64), 0), ((2, 1, (1, 60, 1), (20,) * 3, FP32), 0),
    ((2, 1, (3, 40, 1), (16,) * 3, FP32), 1), ((2, 1, (5, 31, 1), (16,) * 3, FP64), 1),
    # p = 2: runs of two
    ((2, 2, (1, 60, 1), (24,) * 3, FP64), 0), ((2, 2, (3, 40, 1), (20,) * 3, FP64), 0),
    ((2, 2, (3, 40, 1), (24,) * 3, FP64), 1), ((2, 2, (5, 31, 1), (12,) * 3, FP64), 0),
    ((2, 2, (5, 31, 1), (16,) * 3, FP64), 1), ((2, 2, (24, 40, 1), (16,) * 3, FP64), 1),
    ((2, 2, (3, 40, 1), (24,) * 3, FP32), 0), ((2, 2, (5, 31, 1), (24,) * 3, BF16), 0),
    ((2, 2, (33, 33, 1), (8,) * 3, FP32), 0), ((2, 2, (24, 24, 1), (8,) * 3, BF16), 0),
    ((2, 2, (8, 8, 1), (16,) * 3, FP32), 0), ((2, 2, (32, 32, 1), (24,) * 3, FP32), 1),
    # not built
    ((2, 3, (32, 32, 1), (24,) * 3, FP64), 0), ((3, 1, (8, 8, 8), (16,) * 3, FP64), 0),
]


def test_rows_rule(monkeypatch):
    monkeypatch.delenv("BGK_ROWS", raising=False)
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not found")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "rows_rule_check")
        subprocess.run([hipcc, "-std=c++17", "-O1", "--offload-host-only", "-Wno-unused-function",
                        "-I", os.path.join(ROOT, "include"),
                        os.path.join(HERE, "rows_rule_check.cpp"), "-o", exe],
                       check=True, capture_output=True, timeout=300)
        text = "\n".join(" ".join(map(str, (c[0], c[1], *c[2], *c[3], c[4]))) for c, _ in CASES)
        r = subprocess.run([exe], input=text + "\n", capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    got = [int(x) for x in r.stdout.split()]
    bad = [(c, want, g) for (c, want), g in zip(CASES, got) if g != want]
    assert len(got) == len(CASES) and not bad, bad
