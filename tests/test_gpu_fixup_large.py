"""Exact recomputation for 512 points and more against the oracle: every table depth, the smallest and
largest tables it holds, few queued symbols (a wavefront each) and many (a lane each, ragged last
batch), SNRs up to where sums leave the lane form's range, non-finite symbols among the queued.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2108_07004_amd as dm
import workloads as W
from gpu_helpers import GMI_TOL, LLR_TOL_FP32, DeviceBlock, rel_err

pytestmark = pytest.mark.gpu

SNRS = np.array([10.0, 18.0, 26.0, 40.0])


@pytest.mark.parametrize("N", [130, 9001])
@pytest.mark.parametrize("M,D", [(512, 1), (512, 8), (1024, 2), (1024, 4), (2048, 3), (2048, 5), (2048, 6), (2048, 7),
                                 (2048, 8), (8192, 2), (16384, 1)])
def test_large_tables(M, D, N):
    const = W.gaussian_constellation(M, D, 66, M, D)
    g = W.rng(66, "misc", M, D)
    c = dm.Constellation(const.points, const.labels)
    tx = g.integers(0, M, N).astype(np.uint16)
    blk = DeviceBlock(const, tx, g.standard_normal((N, D)), W.sigma2_from_snr_db(SNRS))
    llrs = blk.new_llrs()
    gmi, mi = dm.gmi_estimate(c, blk.sigma2, blk.ys, blk.tx_t, llrs)
    idx = np.unique(np.concatenate([np.arange(0, min(N, 300)), np.arange(max(0, N - 300), N)]))
    for s, s2 in enumerate(blk.sigma2):
        ref = oracle.demap(const.points, const.labels, s2, blk.y_host(s, idx), tx[idx])
        assert rel_err(llrs[s].cpu().numpy()[idx], ref["llr"]) <= LLR_TOL_FP32, s
        if N <= 600:
            assert abs(gmi[s] - ref["gmi"]) <= GMI_TOL and abs(mi[s] - ref["mi_mean"]) <= GMI_TOL, s
    # the same symbols in a launch of few: the form by lanes against the one by wavefronts
    part = [blk.new_llrs()[0][:100] for _ in SNRS]
    dm.gmi_estimate(c, blk.sigma2, [y[:100].contiguous() for y in blk.ys], blk.tx_t[:100].contiguous(), part)
    for s in range(len(SNRS)):
        assert rel_err(llrs[s][:100].cpu().numpy(), part[s].double().cpu().numpy()) <= 2 * LLR_TOL_FP32, s


def test_non_finite_symbols_as_by_wavefronts():
    """Symbols with infinities and NaN among many queued ones get what a small launch gives them."""
    import torch
    const = W.gaussian_constellation(1024, 4, 66, 1024, 4)
    c = dm.Constellation(const.points, const.labels)
    g = W.rng(66, "misc", 7)
    N = 8000
    tx = g.integers(0, 1024, N).astype(np.uint16)
    y = W.awgn(const.points, tx, g.standard_normal((N, 4)), W.sigma2_from_snr_db(25.0))
    y[3, 1] = np.inf
    y[64, 0] = -np.inf
    y[65, 3] = np.nan
    y[7990, 2] = 1.0e30
    y_t = torch.from_numpy(y).to("cuda:0")
    s2 = float(W.sigma2_from_snr_db(25.0))
    whole = dm.demap_llr(c, s2, y_t).cpu().numpy()
    for i in (3, 64, 65, 7990, 0, 66, 7999):
        one = dm.demap_llr(c, s2, y_t[i:i + 1].contiguous()).cpu().numpy()[0]
        assert np.array_equal(np.isnan(one), np.isnan(whole[i])), i
        fin = np.isfinite(one)
        assert np.array_equal(one[~fin & ~np.isnan(one)], whole[i][~fin & ~np.isnan(one)]), i
        assert rel_err(whole[i][fin], one[fin].astype(np.float64)) <= 2 * LLR_TOL_FP32, i


@pytest.mark.parametrize("M,D", [(16, 3), (16, 8), (32, 1), (32, 2), (64, 4), (64, 5), (64, 8)])
def test_small_tables_by_lane(M, D):
    """16 to 64 points, up to SNRs whose sums leave the one-pass form's range."""
    const = W.gaussian_constellation(M, D, 67, M, D)
    g = W.rng(67, "misc", M, D)
    c = dm.Constellation(const.points, const.labels)
    N = 700
    tx = g.integers(0, M, N).astype(np.uint16)
    blk = DeviceBlock(const, tx, g.standard_normal((N, D)), W.sigma2_from_snr_db(np.array([14.0, 22.0, 30.0, 45.0])))
    llrs = blk.new_llrs()
    gmi, mi = dm.gmi_estimate(c, blk.sigma2, blk.ys, blk.tx_t, llrs)
    for s, s2 in enumerate(blk.sigma2):
        ref = oracle.demap(const.points, const.labels, s2, blk.y_host(s), tx)
        assert rel_err(llrs[s].cpu().numpy(), ref["llr"]) <= LLR_TOL_FP32, s
        assert abs(gmi[s] - ref["gmi"]) <= GMI_TOL and abs(mi[s] - ref["mi_mean"]) <= GMI_TOL, s


@pytest.mark.parametrize("M,D", [(128, 2), (256, 4)])
@pytest.mark.parametrize("N", [1, 33, 600, 17000, 300000])
def test_row_chunks(M, D, N):
    """128 and 256 points: entry counts around the row form's chunk sizes, against the same symbols in
    other launches (their LLRs are bit-identical) and, for the first of them, the oracle."""
    import torch
    const = W.gaussian_constellation(M, D, 68, M, D)
    g = W.rng(68, "misc", M, D)
    c = dm.Constellation(const.points, const.labels)
    tx = g.integers(0, M, N).astype(np.uint16)
    s2 = float(W.sigma2_from_snr_db(24.0))
    y = W.awgn(const.points, tx, g.standard_normal((N, D)), s2)
    y_t = torch.from_numpy(y).to("cuda:0")
    whole = dm.demap_llr(c, s2, y_t)
    n = min(N, 500)
    ref = oracle.demap(const.points, const.labels, s2, y[:n], tx[:n])
    assert rel_err(whole[:n].cpu().numpy(), ref["llr"]) <= LLR_TOL_FP32
    for lo, hi in ((0, n), (N // 2, min(N, N // 2 + 3000))):
        assert torch.equal(dm.demap_llr(c, s2, y_t[lo:hi].contiguous()), whole[lo:hi])
