"""Tuner entries of another version, and of the other side of preconditioning
(whose matvecs take another form), are not taken over."""
import json
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import json, sys
sys.path.insert(0, {root!r})
from paper_2410_22686_amd import Solver
s = Solver(2, 15, 16, [1e-4, 1e-6], side={side!r}, tune=True, device="cuda:0")
print("KERNELS " + json.dumps(s.kernels), flush=True)
"""


def child(cache, side):
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT, side=side)], env=dict(os.environ, PCOP_TUNE_CACHE=str(cache)),
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads([l for l in r.stdout.splitlines() if l.startswith("KERNELS ")][-1][len("KERNELS "):])


def rows(cache):
    return [l.split() for l in open(cache) if l.startswith("pcop-tune ")]


def test_other_versions_and_sides_are_tuned_afresh(tmp_path):
    cache = tmp_path / "tune.txt"
    child(cache, "right")
    row, = rows(cache)
    # choices timed on the kernels before version 3
    old = list(row)
    old[1], old[19] = "2", "3"
    cache.write_text(" ".join(old) + "\n")
    child(cache, "right")
    assert len(rows(cache)) == 2
    # right and flexible share an entry, left has its own
    cache.write_text(" ".join(row) + "\n")
    child(cache, "flexible")
    assert len(rows(cache)) == 1
    child(cache, "left")
    assert len(rows(cache)) == 2
