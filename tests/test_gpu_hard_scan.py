"""Hard decisions whose matrix ranking proves nothing: none, a few, most and all symbols of a wave (scanned by
the wave or by their own lanes), with NaN and infinities among them and ties between points.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2108_07004_amd as dm
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,D", [(32, 1), (32, 2), (64, 3), (128, 2), (512, 4), (2048, 8), (8192, 2)])
def test_any_number_of_unproven_symbols(M, D):
    import torch
    c = W.gaussian_constellation(M, D, 85, M, D)
    pts = c.points.copy()
    pts[M // 2 + 1] = pts[3]  # two labels at one point: the lower wins
    g = W.rng(85, "misc", M, D)
    N = 65 * 64 + 17
    tx = g.integers(0, M, size=N).astype(np.uint16)
    y = W.awgn(pts, tx, g.standard_normal((N, D)), W.sigma2_from_snr_db(12.0))
    for w in range(65):  # w symbols of wave w out of the operand range
        i = 64 * w + g.permutation(64)[:w]
        y[i] *= np.float32(2.0e4)
        if w > 3:
            y[i[0], 0], y[i[1], D - 1], y[i[2], 0] = np.nan, np.inf, -np.inf
            y[i[3]] = pts[3]
    tiny = (pts * np.float32(1e-3)).astype(np.float32)  # nothing is proven at this scale
    for table, yy in ((pts, y), (tiny, (y * np.float32(1e-3)).astype(np.float32))):
        const = dm.Constellation(table, c.labels)
        out = torch.full((N,), -1, dtype=torch.int16, device="cuda:0")
        se, be = dm.hard_decision(const, [torch.from_numpy(yy).to("cuda:0")],
                                  torch.from_numpy(tx.view(np.int16)).to("cuda:0"), [out], method="mfma")
        ref = oracle.hard_demap(table, c.labels, yy, tx)
        assert np.array_equal(out.cpu().numpy().view(np.uint16), ref["labels"])
        assert (se[0], be[0]) == (ref["sym_err"], ref["bit_err"])
