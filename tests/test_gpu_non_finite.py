"""GMI and MI of blocks that hold NaN, infinities and values whose distances overflow: such a symbol adds
nothing, and the others' terms are all there, whether flagged symbols are recomputed in the wave (a
burst of eight and more), from the queue (one alone) or in place (queue full), in a call and in a plan.

The sums over the block are held against the same block without those symbols.  A symbol's terms are
the same bits in both up to the FP32 rounding of m bit terms and the MI term, (m + 1) 2^-22.
"""
from __future__ import annotations

import numpy as np
import pytest

import paper_2108_07004_amd as dm
import workloads as W

pytestmark = pytest.mark.gpu

BAD = np.array([np.nan, np.inf, -np.inf, 1.0e30], dtype=np.float32)


def _inputs(M, D, N, snr_db, where):
    import torch
    const = W.gaussian_constellation(M, D, 80, M, D) if D != 2 else W.qam(M)
    g = W.rng(80, "misc", M, D, N)
    tx = g.integers(0, M, N).astype(np.uint16)
    s2 = float(W.sigma2_from_snr_db(snr_db))
    y = W.awgn(const.points, tx, g.standard_normal((N, D)), s2)
    y[where, g.integers(0, D, len(where))] = BAD[np.arange(len(where)) % 4]
    keep = np.ones(N, dtype=bool)
    keep[where] = False
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    return const, s2, (dev(y), dev(tx.view(np.int16)), N), (dev(y[keep]), dev(tx[keep].view(np.int16)), int(keep.sum()))


def _same_sums(m, whole, n_whole, finite, n_finite):
    for a, b in zip(whole, finite):
        assert np.isfinite(a) and abs(a * n_whole - b * n_finite) <= n_whole * (m + 1) * 2.0 ** -22, (a, b)


@pytest.mark.parametrize("snr_db", [6.0, 25.0])
@pytest.mark.parametrize("M,D", [(2, 1), (4, 2), (8, 2), (16, 2), (16, 8), (64, 2), (256, 4), (1024, 8)])
def test_call_and_plan(M, D, snr_db):
    where = np.concatenate([np.arange(640, 690), [3, 64, 2000, 4990]])
    const, s2, (y, tx, N), (yf, txf, nf) = _inputs(M, D, 5000, snr_db, where)
    c = dm.Constellation(const.points, const.labels)
    gw, mw = dm.gmi_estimate(c, [s2], [y], tx)
    gf, mf = dm.gmi_estimate(c, [s2], [yf], txf)
    _same_sums(const.m, (gw[0], mw[0]), N, (gf[0], mf[0]), nf)
    plan = dm.Plan([(c, s2, y, tx, None), (c, s2, yf, txf, None)], prec="fp32", autotune=False)
    plan.launch()
    g, mi, _ = plan.results()
    _same_sums(const.m, (g[0], mi[0]), N, (g[1], mi[1]), nf)


@pytest.mark.parametrize("M,D,prec", [(16, 3, "fp32"), (64, 3, "fp16x3")])
def test_queue_full(M, D, prec):
    """2^21 symbols, nearly all flagged: twice the allocation-free call's queue, the burst at the end."""
    N = 1 << 21
    const, s2, (y, tx, _), (yf, txf, nf) = _inputs(M, D, N, 40.0, np.arange(N - 5000, N - 4000))
    c = dm.Constellation(const.points, const.labels)
    gw, mw = dm.gmi_estimate_noalloc(c, [s2], [y], tx, [y.new_empty((N, const.m))], prec=prec)
    gf, mf = dm.gmi_estimate(c, [s2], [yf], txf, [y.new_empty((nf, const.m))], prec=prec)
    _same_sums(const.m, (gw[0], mw[0]), N, (gf[0], mf[0]), nf)
