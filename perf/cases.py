"""Performance cases of the demapper: what its users run, each through a public entry point.

A case is a dict of plain values with a "kind":

  llr      demap_llr of one received block (an online receiver: LLRs for the decoder)
  gmi      gmi_estimate of one transmitted block at several noise levels (AIR curves), LLRs written
           or not, GMI and MI
  hard     hard_decision of several received blocks, decided labels and error counts (BER)
  plan     launch + results of a batched plan over uneven instances (scoring many constellations)
  gs       gs_optimize, the geometric-shaping search
  train    MLP.train of the learned demapper on a stream of samples (weights and loss come back)
  grad     MLP.gradients of one batch
  learned  demap_learned of one transmitted block at several noise levels, exact audit on

Constellations: "<M>-qam" (the 2D formats of the receiver, M <= 256), "dp-qpsk" and "dp-16qam"
(4D), "pam8d" (the 8D Gray product of 2048 points), "gauss<D>d-<M>" (random tables).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2108_07004_amd as dm
import workloads as W

DEV = "cuda:0"
PAM8D = [4, 4, 4, 2, 2, 2, 2, 2]
GELU_A, GELU_B = 0.7978845608028654, 0.044715  # tanh-form GELU


# ---------------------------------------------------------------------------------------- cases

def listed():
    return [
        # smallest call: one short frame of the paper's 16-QAM, LLRs only; launches and latency
        {"name": "llr-16qam-4k", "kind": "llr", "const": "16-qam", "N": 4096, "snr": 12.0, "prec": "fp32"},
        # the DP-QPSK workload: a 65,536-symbol block at 6 noise levels, launch-bound
        {"name": "gmi-dpqpsk", "kind": "gmi", "const": "dp-qpsk", "N": 65536, "n_snr": 6, "snr_lo": 0.0,
         "snr_hi": 10.0, "prec": "fp32", "llr": True},
        # the paper's 64-QAM receiver at its buffer size (2^20 symbols, here with a ragged tail),
        # default precision
        {"name": "llr-64qam-1m", "kind": "llr", "const": "64-qam", "N": (1 << 20) + 77, "snr": 18.0, "prec": "fp32"},
        # an AIR curve of DP-16QAM in the default precision
        {"name": "gmi-dp16qam-fp32", "kind": "gmi", "const": "dp-16qam", "N": 1 << 20, "n_snr": 11, "snr_lo": 0.0,
         "snr_hi": 20.0, "prec": "fp32", "llr": True},
        # the DP-16QAM workload at its full size on the matrix cores
        {"name": "gmi-dp16qam", "kind": "gmi", "const": "dp-16qam", "N": 1 << 22, "n_snr": 11, "snr_lo": 0.0,
         "snr_hi": 20.0, "prec": "fp16x3", "llr": True},
        # the 8D 2048-point workload (16 noise levels), a 2^21-symbol block
        {"name": "gmi-8d2048", "kind": "gmi", "const": "gauss8d-2048", "N": 1 << 21, "n_snr": 16, "snr_lo": 0.0,
         "snr_hi": 15.0, "prec": "fp16x3", "llr": True},
        # the paper's receiver: minimum-distance decisions and BER of 128-QAM, 8 blocks of 2^20
        {"name": "hard-128qam", "kind": "hard", "const": "128-qam", "N": 1 << 20, "n_snr": 8, "snr_lo": 14.0,
         "snr_hi": 28.0},
        # decisions of the 8D 2048-point workload
        {"name": "hard-8d2048", "kind": "hard", "const": "gauss8d-2048", "N": 1 << 20, "n_snr": 16, "snr_lo": 0.0,
         "snr_hi": 15.0},
        # 64 uneven candidates in one launch (fixed launch shape: the same arithmetic every time)
        {"name": "plan-64", "kind": "plan", "count": 64, "n_lo": 14, "n_hi": 22, "prec": "fp16x3", "llr": True},
        # 20 iterations of the shaping search from rectangular 8-QAM (GS-8 design point)
        {"name": "gs-8qam", "kind": "gs", "const": "8-qam", "N": 65536, "snr": 14.0, "iters": 20, "candidates": 32},
        # 64 Adam steps of the learned demapper
        {"name": "train-pam8d", "kind": "train", "const": "pam8d", "N": 1 << 18, "batch": 4096},
        # learned demapping with its exact audit
        {"name": "learned-pam8d", "kind": "learned", "const": "pam8d", "N": 1 << 20, "n_snr": 16, "snr_lo": 0.0,
         "snr_hi": 15.0},
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def size(M, n_snr, lo=1000, hi=1 << 22):
        # at most 2^36 (symbol, point) pairs in a pass: the 8D 2048-point listed case
        return logint(lo, max(lo + 1, min(hi, (1 << 36) // (M * n_snr))))

    kind = rng.choice(["llr", "llr", "gmi", "gmi", "gmi", "hard", "hard", "plan", "gs", "train", "grad", "learned"])
    const = rng.choice(["4-qam", "8-qam", "16-qam", "32-qam", "64-qam", "128-qam", "256-qam", "dp-qpsk", "dp-16qam",
                        "pam8d", "gauss8d-2048", "gauss4d-1024", "gauss2d-64", "gauss8d-16"])
    if kind in ("train", "grad", "learned"):
        const = rng.choice(["pam8d", "16-qam", "dp-16qam"])
    M = _points(const)[0].shape[0]
    precs = ["fp32", "fp32"] + (["fp16x3", "fp16x3", "bf16x3"] if M >= 32 else [])
    if kind == "llr":
        prec = rng.choice(precs)
        return {"kind": kind, "const": const, "N": size(M * (4 if prec == "fp32" else 1), 1, 500),
                "snr": round(rng.uniform(0.0, 22.0), 2), "prec": prec}
    if kind == "gmi":
        prec, ns = rng.choice(precs), rng.randint(1, 16)
        return {"kind": kind, "const": const, "N": size(M * (4 if prec == "fp32" else 1), ns), "n_snr": ns,
                "snr_lo": round(rng.uniform(-2.0, 8.0), 2), "snr_hi": round(rng.uniform(10.0, 22.0), 2),
                "prec": prec, "llr": rng.random() < 0.6}
    if kind == "hard":
        ns = rng.randint(1, 16)
        return {"kind": kind, "const": const, "N": size(M, ns), "n_snr": ns, "snr_lo": round(rng.uniform(0.0, 10.0), 2),
                "snr_hi": round(rng.uniform(12.0, 28.0), 2)}
    if kind == "plan":
        lo = rng.randint(10, 14)
        return {"kind": kind, "count": rng.randint(3, 64), "n_lo": lo, "n_hi": rng.randint(lo + 2, 21),
                "prec": rng.choice(["fp16x3", "fp32"]), "llr": rng.random() < 0.5}
    if kind == "gs":
        c = rng.choice(["8-qam", "16-qam", "32-qam", "64-qam", "128-qam"])
        return {"kind": kind, "const": c, "N": logint(4096, 65536), "snr": round(rng.uniform(10.0, 20.0), 2),
                "iters": rng.randint(5, 20), "candidates": rng.randint(4, 32)}
    if kind == "train":
        return {"kind": kind, "const": const, "N": logint(1 << 14, 1 << 18), "batch": 256 * rng.choice([4, 8, 16, 20])}
    if kind == "grad":
        return {"kind": kind, "const": const, "batch": 256 * rng.randint(1, 64)}
    ns = rng.randint(1, 16)
    return {"kind": "learned", "const": const, "N": size(2048, ns, 2000), "n_snr": ns, "snr_lo": 0.0, "snr_hi": 15.0}


# --------------------------------------------------------------------------------------- inputs

def _points(name):
    """(points M x D float32, labels M uint16)."""
    if name.endswith("-qam"):
        c = W.qam(int(name[:-4]))
    elif name == "dp-qpsk":
        c = W.dp_qpsk()
    elif name == "dp-16qam":
        c = W.dp_16qam()
    elif name == "pam8d":
        c = W.product_pam_mixed(PAM8D)
    else:  # gauss<D>d-<M>
        d, m = name[len("gauss"):].split("d-")
        c = W.gaussian_constellation(int(m), int(d), 2)
    return c.points, c.labels


def _snrs(case):
    if "n_snr" not in case:
        return [case["snr"]]
    return np.linspace(case["snr_lo"], case["snr_hi"], case["n_snr"]).tolist()


def _gen(seed, tag=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + tag)
    return g


def _block(points, N, snrs, g):
    """tx (N,) int16 rows and one received block per noise level, sharing one noise draw."""
    M, D = points.shape
    tx = torch.randint(0, M, (N,), generator=g, device=DEV)
    z = torch.randn((N, D), generator=g, device=DEV)
    x = torch.from_numpy(points).to(DEV)[tx]
    ys = [x + math.sqrt(float(W.sigma2_from_snr_db(s))) * z for s in snrs]
    return tx.to(torch.int16), ys


def _samples(points, N, g):
    """Training samples: uniform rows, SNR uniform on [0, 15] dB per sample."""
    M, D = points.shape
    tx = torch.randint(0, M, (N,), generator=g, device=DEV)
    s2 = 0.5 * torch.pow(10.0, -1.5 * torch.rand((N,), generator=g, device=DEV))
    z = torch.randn((N, D), generator=g, device=DEV)
    return torch.from_numpy(points).to(DEV)[tx] + s2.sqrt()[:, None] * z, s2


def _plan_instances(case):
    return W.batched_instances(case["count"], case["n_lo"], case["n_hi"])


def _weights(D, m):
    return W.mlp_init_weights(D, 256, m)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "plan":
        insts = _plan_instances(case)
        consts, items, flat, at = [], [], None, 0
        if case["llr"]:  # every instance's N x m LLRs, one after the other
            flat = torch.empty((sum(i.N * i.const.m for i in insts),), device=DEV)
        for inst in insts:
            c = dm.Constellation(inst.const.points, inst.const.labels)
            tx, ys = _block(inst.const.points, inst.N, [inst.snr_db], _gen(seed, inst.index))
            llr, n = None, inst.N * inst.const.m
            if flat is not None:
                llr, at = flat[at:at + n].view(inst.N, inst.const.m), at + n
            items.append((c, inst.sigma2, ys[0], tx, llr))
            consts.append(c)
        return {"kind": kind, "plan": dm.Plan(items, prec=case["prec"], autotune=False), "keep": (consts, items),
                "llr": flat}
    pts, lab = _points(case["const"])
    M, D = pts.shape
    m = M.bit_length() - 1
    g = _gen(seed)
    if kind == "gs":
        N = case["N"]
        return {"kind": kind, "case": case, "points": pts, "labels": lab, "seed": int(seed),
                "tx": torch.randint(0, M, (N,), generator=g, device=DEV).to(torch.int16),
                "z": torch.randn((N, D), generator=g, device=DEV)}
    c = dm.Constellation(pts, lab)
    if kind == "train":
        y, s2 = _samples(pts, case["N"], g)
        return {"kind": kind, "c": c, "net": dm.MLP(c, _weights(D, m)), "y": y, "s2": s2, "batch": case["batch"]}
    if kind == "grad":
        y, s2 = _samples(pts, case["batch"], g)
        return {"kind": kind, "c": c, "net": dm.MLP(c, _weights(D, m)), "y": y, "s2": s2,
                "target": dm.demap_llr_var(c, s2, y)}
    snrs = _snrs(case)
    tx, ys = _block(pts, case["N"], snrs, g)
    s = {"kind": kind, "c": c, "tx": tx, "ys": ys, "sigma2": W.sigma2_from_snr_db(snrs)}
    if kind == "hard":
        s["labels"] = [torch.empty((case["N"],), dtype=torch.int16, device=DEV) for _ in snrs]
        return s
    s["llr"] = [torch.empty((case["N"], m), device=DEV) for _ in snrs] if case.get("llr", True) else None
    if kind == "learned":
        s["net"] = dm.MLP(c, _weights(D, m))
    else:
        s["prec"] = case["prec"]
    return s


# ---------------------------------------------------------------------------------------- a pass

def run(s):
    kind = s["kind"]
    if kind == "llr":
        return {"llr": dm.demap_llr(s["c"], s["sigma2"][0], s["ys"][0], s["llr"][0], prec=s["prec"])}
    if kind == "gmi":
        gmi, mi = dm.gmi_estimate(s["c"], s["sigma2"], s["ys"], s["tx"], s["llr"], prec=s["prec"])
        return {"gmi": gmi, "mi": mi, "llr": s["llr"]}
    if kind == "hard":
        se, be = dm.hard_decision(s["c"], s["ys"], s["tx"], s["labels"])
        return {"sym_err": se, "bit_err": be, "labels": s["labels"]}
    if kind == "plan":
        s["plan"].launch()
        gmi, mi, _ = s["plan"].results()
        return {"gmi": gmi, "mi": mi, "llr": s["llr"]}
    if kind == "gs":
        c = s["case"]
        pts, labels, trace, accepted = dm.gs_optimize(s["points"], s["labels"], c["snr"], s["tx"], s["z"],
                                                      iters=c["iters"], candidates=c["candidates"], seed=s["seed"])
        return {"points": pts, "labels": labels, "trace": trace, "accepted": accepted}
    if kind == "train":
        loss = s["net"].train(s["c"], s["y"], s["s2"], batch=s["batch"])
        return {"loss": loss, "weights": s["net"].get_weights()}
    if kind == "grad":
        grads, loss = s["net"].gradients(s["y"], s["s2"], s["target"])
        return {"loss": loss, "grads": grads}
    # an untrained network would always fail its audit: the bound is set where it passes, so the
    # audit runs and the network's own results come back, as they do for a trained one
    gmi, loss, used = dm.demap_learned(s["net"], s["c"], s["sigma2"], s["ys"], s["tx"], s["llr"], max_gmi_loss=1e3)
    return {"gmi": gmi, "gmi_loss": loss, "used": used, "llr": s["llr"]}


# ------------------------------------------------------------------------------------------ work

def work(case):
    """Bytes: every input read once, every output written once.  Operations per (symbol, point):
    the cross term (2 D), the norm, scale and exponential (4) and two subset additions; for a
    decision the cross term, the norm and one comparison."""
    kind = case["kind"]
    if kind == "plan":
        by = fl = 0
        for i in _plan_instances(case):
            by += i.N * (4 * i.const.D + 2 + (4 * i.const.m if case["llr"] else 0))
            fl += i.N * i.const.M * (2 * i.const.D + 6)
        return {"bytes": by, "flops": fl}
    M, D = _points(case["const"])[0].shape
    m = M.bit_length() - 1
    net = 2 * ((D + 1) * 256 + 256 * 256 + 256 * m)
    if kind in ("train", "grad"):
        N = case["N"] // case["batch"] * case["batch"] if kind == "train" else case["batch"]
        params = (D + 1) * 256 + 256 + 256 * 256 + 256 + 256 * m + m
        return {"bytes": N * 4 * (D + 1) + 8 * params,
                "flops": N * (3 * net + (M * (2 * D + 6) if kind == "train" else 0))}
    if kind == "gs":
        evals = (case["iters"] + 1) * case["candidates"]
        return {"bytes": case["N"] * (4 * D + 2), "flops": evals * case["N"] * M * (2 * D + 6)}
    N, ns = case["N"], case.get("n_snr", 1)
    if kind == "hard":
        return {"bytes": N * ns * (4 * D + 2) + 2 * N, "flops": N * ns * M * (2 * D + 2)}
    llr = 4 * m if case.get("llr", True) else 0
    tx = 0 if kind == "llr" else 2 * N
    per = net if kind == "learned" else M * (2 * D + 6)
    return {"bytes": N * ns * (4 * D + llr) + tx, "flops": N * ns * per}


# ------------------------------------------------------------------------------------- in 64 bits

def _exact_block(points, labels, y, sigma2, tx, want_llr):
    """(llr or None, gmi, mi) of one block: two-term log-sum-exp in float64, chunk by chunk."""
    M, D = points.shape
    m = M.bit_length() - 1
    X = torch.from_numpy(points).to(DEV).double()
    lab = torch.from_numpy(labels.astype(np.int64)).to(DEV)
    bits = torch.stack([(lab >> (m - 1 - k)) & 1 for k in range(m)], 1).double()  # M x m
    sides = torch.cat([bits, 1.0 - bits], 1).contiguous()
    xn = (X * X).sum(1)
    N = y.shape[0]
    llr = torch.empty((N, m), dtype=torch.float64, device=DEV) if want_llr else None
    gs = ms = 0.0
    step = max(1, (1 << 27) // M)
    scale = 0.5 / float(sigma2)
    for a in range(0, N, step):
        yb = y[a:a + step].double()
        t = torch.mm(yb, X.t()).mul_(2.0).sub_(xn[None, :]).mul_(scale)  # -d^2 / (2 s2) + const(y)
        top = t.max(1, keepdim=True).values
        e = torch.exp_(t - top)
        S = torch.mm(e, sides)
        lo = torch.log(S[:, :m]) - torch.log(S[:, m:])
        bad = (S <= 1e-290).any(1).nonzero()[:, 0]  # a subset too far for one common maximum
        for b in bad.split(4096):
            tb = t[b]
            for k in range(m):
                one = bits[:, k] > 0
                lo[b, k] = torch.logsumexp(tb[:, one], 1) - torch.logsumexp(tb[:, ~one], 1)
        if want_llr:
            llr[a:a + step] = lo
        if tx is not None:
            row = tx[a:a + step].long()
            sent = bits[row]
            gs += float((m - torch.nn.functional.softplus((1.0 - 2.0 * sent) * lo).sum(1) / math.log(2.0)).sum())
            tt = t.gather(1, row[:, None])[:, 0] - top[:, 0]
            ms += float((m - (torch.log(e.sum(1)) - tt) / math.log(2.0)).sum())
    return llr, gs / N, ms / N


def _exact_net(w, y, sigma2):
    """The learned demapper's network in float64: y (N x D), one noise variance."""
    s = -10.0 * math.log10(2.0 * float(sigma2))
    t = {k: torch.from_numpy(v).to(DEV).double() for k, v in w.items()}

    def gelu(h):
        return 0.5 * h * (1.0 + torch.tanh(GELU_A * (h + GELU_B * h * h * h)))

    out = []
    for yb in y.split(1 << 18):
        f = torch.cat([yb.double(), torch.full((yb.shape[0], 1), (s - 7.5) / 7.5, dtype=torch.float64, device=DEV)], 1)
        a = gelu(torch.mm(f, t["W1"]) + t["b1"])
        a = gelu(torch.mm(a, t["W2"]) + t["b2"])
        out.append(torch.mm(a, t["W3"]) + t["b3"])
    return torch.cat(out)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("hard", "gs", "train"):
        # decisions and counts are whole numbers; the search and the optimiser's steps follow
        # comparisons and signs of rounded values, which have no 64-bit counterpart
        return None
    if kind == "plan":
        gmi, mi, llr = [], [], []
        for inst in _plan_instances(case):
            p, lab = inst.const.points, inst.const.labels
            tx, ys = _block(p, inst.N, [inst.snr_db], _gen(seed, inst.index))
            L, g, i = _exact_block(p, lab, ys[0], inst.sigma2, tx, case["llr"])
            gmi.append(g)
            mi.append(i)
            llr.append(L)
        return {"gmi": np.array(gmi), "mi": np.array(mi),
                "llr": torch.cat([L.reshape(-1) for L in llr]) if case["llr"] else None}
    pts, lab = _points(case["const"])
    M, D = pts.shape
    m = M.bit_length() - 1
    g = _gen(seed)
    if kind == "grad":
        return _exact_grad(case, pts, lab, m, g)
    snrs = _snrs(case)
    s2 = W.sigma2_from_snr_db(snrs)
    tx, ys = _block(pts, case["N"], snrs, g)
    if kind == "llr":
        return {"llr": _exact_block(pts, lab, ys[0], s2[0], None, True)[0]}
    if kind == "gmi":
        r = [_exact_block(pts, lab, y, v, tx, case["llr"]) for y, v in zip(ys, s2)]
        return {"gmi": np.array([x[1] for x in r]), "mi": np.array([x[2] for x in r]),
                "llr": [x[0] for x in r] if case["llr"] else None}
    w = _weights(D, m)
    llr = [_exact_net(w, y, v) for y, v in zip(ys, s2)]
    labels = torch.from_numpy(lab.astype(np.int64)).to(DEV)
    sent = labels[tx.long()]
    bits = torch.stack([(sent >> (m - 1 - k)) & 1 for k in range(m)], 1).double()
    gmi = [float((m - torch.nn.functional.softplus((1.0 - 2.0 * bits) * L).sum(1) / math.log(2.0)).mean()) for L in llr]
    return {"gmi": np.array(gmi), "gmi_loss": None, "used": None, "llr": llr}


def _exact_grad(case, pts, lab, m, g):
    """Soft-BCE gradients of the network in float64 (weights as given, targets in float64)."""
    y, s2 = _samples(pts, case["batch"], g)
    X = torch.from_numpy(pts).to(DEV).double()
    labels = torch.from_numpy(lab.astype(np.int64)).to(DEV)
    t = torch.mm(y.double(), X.t()) * 2.0 - (X * X).sum(1)[None, :]
    t = t * (0.5 / s2.double())[:, None]
    target = []
    for k in range(m):
        one = ((labels >> (m - 1 - k)) & 1) > 0
        target.append(torch.logsumexp(t[:, one], 1) - torch.logsumexp(t[:, ~one], 1))
    p = torch.sigmoid(torch.stack(target, 1))
    w = {k: torch.from_numpy(v).to(DEV).double().requires_grad_() for k, v in _weights(pts.shape[1], m).items()}
    snr = -10.0 * torch.log10(2.0 * s2.double())
    f = torch.cat([y.double(), ((snr - 7.5) / 7.5)[:, None]], 1)

    def gelu(h):
        return 0.5 * h * (1.0 + torch.tanh(GELU_A * (h + GELU_B * h * h * h)))

    o = gelu(gelu(f @ w["W1"] + w["b1"]) @ w["W2"] + w["b2"]) @ w["W3"] + w["b3"]
    sp = torch.nn.functional.softplus
    lt = torch.logit(p)
    loss = ((sp(o) - p * o) - (sp(lt) - p * lt)).mean()
    loss.backward()
    return {"loss": float(loss.detach()), "grads": {k: v.grad for k, v in w.items()}}
