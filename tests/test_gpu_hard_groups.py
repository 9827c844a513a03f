"""Edges of the MFMA decision kernel: its two-level (group, then point) ranking against the oracle.

Shapes: one to many 32-point tiles (odd and even counts), tables of one and of several LDS chunks
and more than 4096 points, every operand depth (D = 1..8), symbol counts around the 64-symbol wave
and the 256..1024-symbol blocks, symbols halfway between points of different 16-label groups, and
values outside the operand range.  Decisions and counts are integers: equality.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2108_07004_amd as dm
import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("M,D,N", [
    (32, 2, 1), (32, 1, 63), (64, 2, 64), (128, 2, 65), (128, 3, 255), (256, 4, 257), (512, 5, 1023),
    (1024, 6, 1025), (2048, 7, 513), (2048, 8, 4095), (4096, 8, 777), (8192, 4, 321), (16384, 2, 300),
])
def test_group_ranking_matches_oracle(M, D, N):
    import torch
    c = W.gaussian_constellation(M, D, 63, M, D)
    g = W.rng(63, "misc", M, D, N)
    const = dm.Constellation(c.points, c.labels)
    tx = g.integers(0, M, size=N).astype(np.uint16)
    ys = [W.awgn(c.points, tx, g.standard_normal((N, D)), W.sigma2_from_snr_db(s)) for s in (2.0, 14.0)]
    # halfway between two points (ties up to rounding), and values far outside the operand range
    a, b = g.integers(0, M, size=(2, N))
    ys.append((0.5 * (c.points[a].astype(np.float64) + c.points[b])).astype(np.float32))
    wild = ys[0].copy()
    wild[::3] *= np.float32(3.0e4)
    wild[1::5, 0] = np.inf
    wild[2::7, D - 1] = np.nan
    ys.append(wild)
    outs = [torch.full((N,), -1, dtype=torch.int16, device=DEV) for _ in ys]
    se, be = dm.hard_decision(const, [_dev(y) for y in ys], _dev(tx.view(np.int16)), outs, method="mfma")
    for i, y in enumerate(ys):
        ref = oracle.hard_demap(c.points, c.labels, y, tx)
        got = outs[i].cpu().numpy().view(np.uint16)
        assert np.array_equal(got, ref["labels"]), (i, int(np.sum(got != ref["labels"])))
        assert (se[i], be[i]) == (ref["sym_err"], ref["bit_err"])
