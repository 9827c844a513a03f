"""The fused training step over its batch range: gradients against the FP64 network.

Batches cover every split of the batch (16, 32 and 64 parts of dW1 / dW3), sample tiles that do and
do not divide over the XCD mapping, one and several passes of the bias sums, and the smallest and
largest input and output widths.  The reference stores activations and deltas as the kernels do
(BF16 pairs); the bounds are those of the single-batch gradient test.
"""
from __future__ import annotations

import numpy as np
import pytest

import paper_2108_07004_amd as dm
import workloads as W
from oracle import mlp

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("M,D,B", [
    (2048, 8, 256), (2048, 8, 512), (2048, 8, 768), (2, 1, 1024), (16, 2, 1280), (16, 13, 2048), (256, 4, 2304),
    (4096, 8, 4096), (64, 7, 4352), (2048, 8, 8192),
])
def test_gradients_over_batches(M, D, B):
    c = W.gaussian_constellation(M, D, 64, M, D)
    m = M.bit_length() - 1
    const = dm.Constellation(c.points, c.labels)
    w = W.mlp_init_weights(D, 256, m, 64)
    g = W.rng(64, "misc", M, D, B)
    for k in ("b1", "b2", "b3"):
        w[k] = g.normal(0.0, 0.1, w[k].shape).astype(np.float32)
    y, s2, _, _ = W.mlp_samples(c, B, 0.0, 15.0, 64, "mlp_eval", M, D)
    T = g.normal(0.0, 4.0, (B, m)).astype(np.float32)
    net = dm.MLP(const, w)
    grads, loss = net.gradients(_dev(y), _dev(s2), _dev(T))
    again, loss2 = net.gradients(_dev(y), _dev(s2), _dev(T))
    w64 = {k: np.asarray(v, dtype=np.float64) for k, v in w.items()}
    X = mlp.features(y, -10.0 * np.log10(2.0 * s2.astype(np.float64)))
    out, cache = mlp.forward_stored(w64, X, rnd_act=mlp.bf16x2_round)
    ref = mlp.backward_stored(w64, cache, out, T.astype(np.float64), rnd_act=mlp.bf16x2_round)
    ref_loss = mlp.loss(out, T.astype(np.float64))
    assert loss == loss2 and abs(loss - ref_loss) <= 1e-4 * abs(ref_loss), (loss, ref_loss)
    for k in ref:
        assert np.array_equal(grads[k], again[k])
        a, r = grads[k].astype(np.float64).ravel(), ref[k].ravel()
        cos = float(a @ r / (np.linalg.norm(a) * np.linalg.norm(r)))
        mx = float(np.max(np.abs(a - r)) / np.sqrt(np.mean(r * r)))
        assert cos >= 0.99999 and mx <= 2e-3, (k, cos, mx)
