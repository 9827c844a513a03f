"""Shapes of the shaping search's received blocks and shared tables: the GMI it reports against the
oracle's GMI of the constellation it returns, on the same block (tolerance of the GMI parity)."""
from __future__ import annotations

import math

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


@pytest.mark.parametrize("M,D,N,K", [(2, 1, 1, 1), (4, 1, 257, 3), (8, 3, 4097, 64), (64, 5, 1000, 7), (512, 8, 777, 5),
                                     (16, 2, 70001, 33)])
def test_reported_gmi_is_the_returned_constellations(M, D, N, K):
    c = W.gaussian_constellation(M, D, 72, M, D)
    g = W.rng(72, "misc", M, D, N)
    tx = g.integers(0, M, size=N).astype(np.uint16)
    z = g.standard_normal((N, D)).astype(np.float32)
    pts, lab, trace, _ = dm.gs_optimize(c.points, c.labels, 9.0, _dev(tx.view(np.int16)), _dev(z), iters=6,
                                        candidates=K, perturb_sd=0.05, swap_prob=0.5, seed=5)
    s2 = 1.0 / (2.0 * 10.0 ** 0.9)
    y = (pts.astype(np.float64)[tx] + math.sqrt(s2) * z.astype(np.float64)).astype(np.float32)
    ref = oracle.demap(pts, lab, s2, y, tx, llr=False)["gmi"]
    assert abs(trace[-1] - ref) <= 1e-4, (trace[-1], ref)
    assert np.all(np.diff(trace) >= 0.0)


def test_out_of_range_label_is_reported():
    c = W.qam(8)
    tx = np.zeros(300, dtype=np.uint16)
    tx[17] = 8
    with pytest.raises(dm.DemapError):
        dm.gs_optimize(c.points, c.labels, 9.0, _dev(tx.view(np.int16)), _dev(np.zeros((300, 2), np.float32)), iters=1,
                       candidates=2)
