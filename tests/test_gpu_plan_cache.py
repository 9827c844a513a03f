"""The autotuner's cache file: times that other kernels left there are not believed."""
from __future__ import annotations

import os
import subprocess
import sys
from pathlib import Path

import pytest

pytestmark = pytest.mark.gpu

ROOT = Path(__file__).resolve().parent.parent

CHILD = """
import numpy as np, torch
import paper_2108_07004_amd as dm
import workloads as W
c = W.qam(64)
const = dm.Constellation(c.points, c.labels)
y = torch.zeros((70000, 2), device="cuda:0")
tx = torch.zeros(70000, dtype=torch.int16, device="cuda:0")
llr = torch.empty((70000, 6), device="cuda:0")
_, ns, _ = dm.Plan([(const, 0.01, y, tx, llr)], prec="fp16x3", autotune=True).info()
print("NS", float(ns[0]), flush=True)
"""


def _run(path):
    env = dict(os.environ, DM_AUTOTUNE_CACHE=str(path), PYTHONPATH=str(ROOT))
    out = subprocess.run([sys.executable, "-c", CHILD], env=env, cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr[-2000:]
    return float(out.stdout.split("NS ")[1])


def test_times_of_other_kernels_are_not_believed(tmp_path):
    path = tmp_path / "cache"
    stale = [f"shape2 gfx950 64 2 4 {kind} {sub} 1e-12\n" for kind in (0, 1) for sub in (1, 2, 4)]
    path.write_text("".join(stale))
    assert _run(path) > 1e-7  # the whole GPU does not reach 1e16 pairs/s
    mine = path.read_text()
    assert mine and not any(line in mine for line in stale)
    # its own times are: a second process takes them from the file
    forged = "".join(" ".join(line.split()[:-1] + ["2e-12"]) + "\n" for line in mine.splitlines())
    path.write_text(forged)
    assert _run(path) < 1e-11
