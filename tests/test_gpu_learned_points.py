"""The learned path runs the tiles of all its SNR points as one list: points, launches of up to 32 of
them, block sizes around the 32-symbol tile and points outside the trained range may not change any
point's LLRs (bit-identical to a call of its own) or GMI (the same sums, up to 2^-28 per wave).
"""
from __future__ import annotations

import numpy as np
import pytest

import paper_2108_07004_amd as dm
import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("n_snr,N", [(1, 1), (2, 31), (5, 33), (40, 257), (33, 5000), (3, 70001)])
def test_points_are_independent(n_snr, N):
    import torch
    c = W.product_pam(4, 2, "16qam")
    const = dm.Constellation(c.points, c.labels)
    net = dm.MLP(const, W.mlp_init_weights(2, 256, 4))
    y, s2, _, _ = W.mlp_samples(c, 1024, 0.0, 15.0, 4, "mlp_train", 70)
    net.train(const, _dev(y), _dev(s2), batch=1024, epochs=1, lr=1e-4, lr_final=1e-4)
    g = W.rng(70, "misc", n_snr, N)
    tx = g.integers(0, 16, N).astype(np.uint16)
    tx_t = _dev(tx.view(np.int16))
    snr = np.linspace(1.0, 14.0, n_snr)
    snr[n_snr // 2] = 20.0 if n_snr > 1 else 5.0  # outside the trained range: exact
    sig = W.sigma2_from_snr_db(snr)
    ys = [_dev(W.awgn(c.points, tx, g.standard_normal((N, 2)), v)) for v in sig]
    out = [torch.full((N, 4), float("nan"), device=DEV) for _ in sig]
    gmi, _, fb = dm.demap_learned(net, const, sig, ys, tx_t, out, max_gmi_loss=-1.0)
    assert fb.tolist() == [2 if s > 15.0 else 0 for s in snr]
    for s in sorted({0, 1 % n_snr, n_snr // 2, min(31, n_snr - 1), min(32, n_snr - 1), n_snr - 1}):
        one = [torch.full((N, 4), float("nan"), device=DEV)]
        g1, _, _ = dm.demap_learned(net, const, [sig[s]], [ys[s]], tx_t, one, max_gmi_loss=-1.0)
        assert torch.equal(out[s], one[0]), s
        assert abs(gmi[s] - g1[0]) <= 2.0 ** -28 * 2048 / N + 1e-12, s
