"""Recomputed LLRs whose far sums lie around 2^-980 and 2^-1880 (the kernels' shared scale, 2^K at a point),
where the range of a double ends and where the one-pass sums end and the recomputation under maxima begins.

Tolerance: every exponent K - c d^2 is one rounding of c, one of each difference (twice, squared), D of the
accumulated square and one of the result away from FP64, (D + 4) 2^-24 of the larger of c d^2 (the LLR, up to
the near side's exponent) and K <= 123; the same again for the logarithms and the near side.
"""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
import paper_2108_07004_amd as dm
import workloads as W

pytestmark = pytest.mark.gpu


def _check(const, s2, y):
    import torch
    c = dm.Constellation(const.points, const.labels)
    got = dm.demap_llr(c, s2, torch.from_numpy(y).to("cuda:0")).cpu().numpy().astype(np.float64)
    ref = oracle.demap(const.points, const.labels, s2, y, np.zeros(len(y), dtype=np.uint16))["llr"]
    tol = 2 * (const.D + 4) * 2.0 ** -24
    assert np.max(np.abs(got - ref) / np.maximum(123.0, np.abs(ref))) <= tol
    return ref


@pytest.mark.parametrize("N", [60, 7000])
@pytest.mark.parametrize("M", [64, 512, 16384])
@pytest.mark.parametrize("lo,hi", [(955.0, 1005.0), (1835.0, 1915.0)])
def test_uniform_table(M, N, lo, hi):
    """1D, natural labels: the top bit's far subset is the other half of the line, its nearest point
    d = |y| away, and half of the table's terms are the smallest that the sums hold."""
    m = M.bit_length() - 1
    x = (np.arange(M) - (M - 1) / 2.0) * (2.0 * math.sqrt(1.5) / M)
    const = W.Constellation(x[:, None].astype(np.float32), np.arange(M, dtype=np.uint16))
    c2 = 1.3 * hi  # log2(e) / (2 sigma2): far distances below 1
    near = x[M // 2]
    v = np.linspace(lo, hi, N)
    y = (near - np.sqrt((123 - m + v) / c2)).astype(np.float32)[:, None]
    ref = _check(const, 0.5 * math.log2(math.e) / c2, y)
    assert np.all(np.abs(ref[:, 0]) > 0.65 * lo)  # the top bit is the one in the range


@pytest.mark.parametrize("snr_db", [30.0, 30.5, 31.0, 31.5, 32.0, 33.0])
def test_8d(snr_db):
    const = W.gaussian_constellation(2048, 8, 81)
    g = W.rng(81, "misc")
    N = 7000
    tx = g.integers(0, 2048, N)
    s2 = float(W.sigma2_from_snr_db(snr_db))
    ref = _check(const, s2, W.awgn(const.points, tx, g.standard_normal((N, 8)), s2))
    band = np.abs(ref) * math.log2(math.e) - 112
    assert np.sum(((band > 955.0) & (band < 1000.0)) | ((band > 1835.0) & (band < 1905.0))) > 1000  # the inputs reach both
