"""The 64-symbols-per-wave MFMA kernel (M = 32..256, D = 2, 4, 8) at its edges: symbol counts around a wave
and each block size, SNRs up to where nearly every symbol takes the in-wave far pass (by both halves of
a wave or by one).  A symbol's LLRs may not depend on the wave, half or block that holds it.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2108_07004_amd as dm
import workloads as W
from gpu_helpers import GMI_TOL, DeviceBlock, rel_err

pytestmark = pytest.mark.gpu

# LLR and GMI / MI bounds of the split precisions over all shapes
BOUNDS = {"fp16x3": (1e-3, GMI_TOL), "bf16x3": (2e-2, 1e-3)}


@pytest.mark.parametrize("prec", ["fp16x3", "bf16x3"])
@pytest.mark.parametrize("M,D", [(32, 2), (64, 4), (128, 8), (256, 2), (256, 4), (256, 8)])
def test_partition_and_oracle(M, D, prec):
    import torch
    const = W.gaussian_constellation(M, D, 65, M, D)
    c = dm.Constellation(const.points, const.labels)
    g = W.rng(65, "misc", M, D)
    N = 70001
    tx = g.integers(0, M, N).astype(np.uint16)
    blk = DeviceBlock(const, tx, g.standard_normal((N, D)), W.sigma2_from_snr_db(np.array([3.0, 14.0, 21.0])))
    whole = blk.new_llrs()
    gmi, mi = dm.gmi_estimate(c, blk.sigma2, blk.ys, blk.tx_t, whole, prec=prec)
    ltol, gtol = BOUNDS[prec]
    for s, s2 in enumerate(blk.sigma2):  # (the GMI / MI bound is one of block means)
        ref = oracle.demap(const.points, const.labels, s2, blk.y_host(s), tx)
        assert rel_err(whole[s].cpu().numpy(), ref["llr"]) <= ltol, s
        assert abs(gmi[s] - ref["gmi"]) <= gtol and abs(mi[s] - ref["mi_mean"]) <= gtol, s
    for lo, n in ((0, 1), (5, 31), (0, 63), (64, 65), (7, 257), (1, 1025), (33, 17000), (0, 40001)):
        part = [torch.full((n, const.m), float("nan"), dtype=torch.float32, device="cuda:0") for _ in whole]
        dm.gmi_estimate(c, blk.sigma2, [y[lo:lo + n].contiguous() for y in blk.ys],
                        blk.tx_t[lo:lo + n].contiguous(), part, prec=prec)
        for s in range(len(part)):
            assert torch.equal(part[s], whole[s][lo:lo + n]), (lo, n, s)
