"""Work lists of plans long enough that workgroups request claims ahead, and their ends, where they do not:
every symbol demapped once (LLRs of two claim sizes bit for bit, none left over), GMI as by the call.
"""
from __future__ import annotations

import pytest

import paper_2108_07004_amd as dm
import workloads as W
from gpu_helpers import GMI_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,D,prec,N", [(4, 2, "fp32", (1 << 22) + 5), (64, 2, "fp16x3", (1 << 21) + 77),
                                        (512, 4, "fp16x3", (1 << 21) + 513)])
def test_long_lists(M, D, prec, N):
    import torch
    const = W.gaussian_constellation(M, D, 84, M, D)
    c = dm.Constellation(const.points, const.labels)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(M)
    s2 = float(W.sigma2_from_snr_db(9.0))
    tx = torch.randint(0, M, (N,), generator=g, device="cuda:0")
    y = torch.from_numpy(const.points).to("cuda:0")[tx] + s2 ** 0.5 * torch.randn((N, D), generator=g, device="cuda:0")
    tx = tx.to(torch.int16)
    llrs, gmis = [], []
    for claim in (4, 1, 8):
        llr = torch.full((N, const.m), float("nan"), device="cuda:0")
        plan = dm.Plan([(c, s2, y, tx, llr), (c, s2, y[:700], tx[:700], None)], prec=prec, autotune=False, claim=claim)
        plan.launch()
        gmi, _, _ = plan.results()
        llrs.append(llr)
        gmis.append(gmi[0])
    assert not torch.isnan(llrs[0]).any()
    assert torch.equal(llrs[0], llrs[1]) and torch.equal(llrs[0], llrs[2])
    one, _ = dm.gmi_estimate(c, [s2], [y], tx, prec=prec)
    assert max(abs(v - one[0]) for v in gmis) <= GMI_TOL
