"""Fix-up of the tables that take a wavefront per symbol (more than 8 dimensions from 512 points on, tables
of more than 16384 floats): few and many queued symbols against the oracle, parts bit for bit.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2108_07004_amd as dm
import workloads as W
from gpu_helpers import LLR_TOL_FP32, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [3, 130, 5001])
@pytest.mark.parametrize("M,D,snr_db", [(4096, 8, 24.0), (8192, 3, 45.0), (512, 16, 21.0), (1024, 9, 24.0), (512, 20, 18.0)])
def test_against_oracle(M, D, snr_db, N):
    import torch
    const = W.gaussian_constellation(M, D, 83, M, D)
    c = dm.Constellation(const.points, const.labels)
    g = W.rng(83, "misc", M, D)
    s2 = float(W.sigma2_from_snr_db(snr_db))
    y = W.awgn(const.points, g.integers(0, M, N), g.standard_normal((N, D)), s2)
    y_t = torch.from_numpy(y).to("cuda:0")
    whole = dm.demap_llr(c, s2, y_t)
    n = min(N, 200)
    ref = oracle.demap(const.points, const.labels, s2, y[-n:], np.zeros(n, dtype=np.uint16))["llr"]
    assert rel_err(whole[-n:].cpu().numpy(), ref) <= LLR_TOL_FP32
    assert np.mean(np.abs(ref) > 100.0) > 0.5  # most were recomputed
    assert torch.equal(dm.demap_llr(c, s2, y_t[-n:].contiguous()), whole[-n:])
