"""The calls that a user of this library makes, at the sizes where they are made, for timing and comparison.

Three kinds of call, each through the package's public functions:
  search   `mine_negatives`: the shortlist search over a pool of queries (from scratch, or started from the
           thresholds of the search before), and the same search as an inference top-k over a few queries
  sample   `sample_negatives`, `sample_negatives_mixture`, `sample_negatives_pps`
  step     `xc_step`: one training step on a batch whose negatives have been sampled
Sizes are those of the workloads in `paper_2409_20156_amd.synth` and of the tests.
"""
import math

import torch

import paper_2409_20156_amd as xc

DEV = "cuda:0"


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _esize(case):
    return 2 if case["dtype"] == "bf16" else 4


# ---------------------------------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest training step (workload tiny): a handful of short launches, latency is everything
        {"name": "step_tiny_f32", "kind": "step", "dtype": "f32", "L": 4096, "d": 64, "B": 32, "k_p": 1, "k_h": 8,
         "k_r": 16, "loss": "bce", "lr": 0.05},
        # the hard + uniform mixture of a c4 batch, drawn on the device before every step
        {"name": "sample_c4", "kind": "sample", "form": "hard", "B": 2048, "k_h": 100, "k_r": 1024, "L": 1300000},
        # top 5 labels of a few online queries: inference with a trained classifier
        {"name": "topk_online", "kind": "search", "dtype": "bf16", "Zq": 32, "L": 131072, "d": 768, "k": 5,
         "warm": False},
        # single precision, nothing a multiple of anything: a small classifier trained in fp32
        {"name": "search_ragged_f32", "kind": "search", "dtype": "f32", "Zq": 1000, "L": 50021, "d": 300, "k": 32,
         "warm": False},
        # the shortlist search of workload c2, from scratch
        {"name": "search_c2", "kind": "search", "dtype": "bf16", "Zq": 10240, "L": 131072, "d": 768, "k": 64,
         "warm": False},
        # its refresh some training steps later, on a classifier that has moved a little
        {"name": "refresh_c2", "kind": "search", "dtype": "bf16", "Zq": 10240, "L": 131072, "d": 768, "k": 64,
         "warm": True},
        # the search of workload c4: the largest pool
        {"name": "search_c4", "kind": "search", "dtype": "bf16", "Zq": 65536, "L": 1300000, "d": 768, "k": 100,
         "warm": False},
        # the search of workload c5: the largest label set, short rows
        {"name": "search_c5", "kind": "search", "dtype": "bf16", "Zq": 16384, "L": 120000000, "d": 256, "k": 50,
         "warm": False},
        # training step, small batch on a classifier that the last-level cache holds
        {"name": "step_c2", "kind": "step", "dtype": "bf16", "L": 131072, "d": 768, "B": 512, "k_p": 4, "k_h": 64,
         "k_r": 256, "loss": "bce", "lr": 0.05},
        # the soft-max loss on workload c3
        {"name": "step_c3_softmax", "kind": "step", "dtype": "bf16", "L": 670000, "d": 768, "B": 1024, "k_p": 16,
         "k_h": 100, "k_r": 512, "loss": "softmax", "lr": 10.0},
        # large batch, most rows of the classifier touched
        {"name": "step_c4", "kind": "step", "dtype": "bf16", "L": 1300000, "d": 768, "B": 2048, "k_p": 8,
         "k_h": 100, "k_r": 1024, "loss": "bce", "lr": 0.05},
        # the batch of workload c5 on a quarter of its labels, so that the whole updated matrix can be compared:
        # short rows, most touched labels in one pair only
        {"name": "step_c5", "kind": "step", "dtype": "bf16", "L": 30000000, "d": 256, "B": 4096, "k_p": 3,
         "k_h": 50, "k_r": 2048, "loss": "bce", "lr": 0.01},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "step", "step", "sample"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    per = 8 if dtype == "bf16" else 4                     # elements of 16 bytes, the granularity of a row
    d = max(1, _log(rng, 64, 768) // per) * per
    if rng.random() < 0.3:
        d = rng.choice([64, 128, 192, 256, 384, 512, 768])
    if kind == "search":
        Zq = _log(rng, 1, 65536)
        L = _log(rng, 4096, 120000000)
        most = 1.2e14 if dtype == "bf16" else 4e12        # multiply-adds: an eighth of the largest listed search
        while Zq * L * d > most or L * d * (2 if dtype == "bf16" else 4) > 3e10:
            if Zq > 64 and rng.random() < 0.5:
                Zq = max(1, int(Zq * 0.7))
            else:
                L = max(4096, int(L * 0.7))
        return {"kind": kind, "dtype": dtype, "Zq": Zq, "L": L, "d": d, "k": _log(rng, 5, 100),
                "warm": rng.random() < 0.25}
    B = _log(rng, 32, 4096)
    L = _log(rng, 4096, 30000000)
    k_h = _log(rng, 8, 100)
    k_r = _log(rng, 16, 2048)
    if kind == "sample":
        return {"kind": kind, "form": rng.choice(["hard", "hard", "mixture", "pps"]), "B": B, "k_h": k_h, "k_r": k_r,
                "L": L}
    while L * d * (2 if dtype == "bf16" else 4) > 15e9:
        L = int(L * 0.7)
    loss = rng.choice(["bce", "bce", "softmax"])          # (the soft-max's coefficients are smaller: a larger rate)
    return {"kind": kind, "dtype": dtype, "L": L, "d": d, "B": B, "k_p": _log(rng, 1, 16), "k_h": k_h, "k_r": k_r,
            "loss": loss, "lr": 10.0 if loss == "softmax" else rng.choice([0.01, 0.05])}


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _matrix(g, n, d, dtype):
    """Rows of about unit length, entries N(0, 1/d)."""
    out = torch.empty((n, d), dtype=dtype, device=DEV)
    rows = max(1, (1 << 28) // d)
    for r in range(0, n, rows):
        out[r:r + rows].normal_(0.0, d ** -0.5, generator=g)
    return out


def _spread(rank, L):
    """Popularity rank -> label id: a bijection of [0, L) that scatters the frequent labels."""
    a = int(L * 0.6180339887) | 1
    while math.gcd(a, L) != 1:
        a += 2
    return (rank * a + L // 7) % L


def _positives(g, n, k_p, L):
    """int32 [n, k_p], -1 padded: 1..k_p labels per query, label frequencies following a Zipf law, none twice."""
    u = torch.rand((n, k_p), generator=g, device=DEV, dtype=torch.float64)
    rank = (torch.pow(float(L), u) - 1.0).to(torch.int64).clamp_(0, L - 1)
    lab = _spread(rank, L)
    count = torch.randint(1, k_p + 1, (n, 1), generator=g, device=DEV)
    keep = torch.arange(k_p, device=DEV)[None, :] < count
    for j in range(1, k_p):
        keep[:, j] &= ~(lab[:, :j] == lab[:, j:j + 1]).any(dim=1)
    return torch.where(keep, lab, torch.full_like(lab, -1)).to(torch.int32).contiguous()


def _shortlists(g, n, k, L):
    """int32 [n, k], distinct within a row: the popular labels turn up in many rows, the others in few."""
    j = torch.arange(k, device=DEV, dtype=torch.float64)[None, :]
    u = torch.rand((n, k), generator=g, device=DEV, dtype=torch.float64)
    rank = torch.arange(k, device=DEV)[None, :] + ((L - k) * torch.pow((j + u) / k, 4)).to(torch.int64)
    order = torch.rand((n, k), generator=g, device=DEV).argsort(dim=1)
    return _spread(rank.clamp_(max=L - 1), L).gather(1, order).to(torch.int32).contiguous()


def prepare(case, seed):
    g = _gen(seed)
    if case["kind"] == "sample":
        B, L, k_h, k_r = case["B"], case["L"], case["k_h"], case["k_r"]
        wide = k_h if case["form"] == "hard" else 2 * k_h              # the sampling forms choose from a wider list
        s = {"case": case, "seed": seed * 7919 + 1, "shortlist": _shortlists(g, B, min(wide, L), L),
             "neg": torch.zeros((B, k_h + k_r), dtype=torch.int32, device=DEV),
             "logq": torch.zeros((B, k_h + k_r), dtype=torch.float32, device=DEV)}
        s["scores"] = torch.randn(s["shortlist"].shape, generator=g, device=DEV).sort(dim=1, descending=True)[0].contiguous()
        return s
    dt, L, d = _dtype(case), case["L"], case["d"]
    W = _matrix(g, L, d, dt)
    n = case["Zq"] if case["kind"] == "search" else case["B"]
    code = xc.XC_BF16 if case["dtype"] == "bf16" else xc.XC_F32
    pos = _positives(g, n, case.get("k_p", 4), L)
    # a query lies near its first positive
    Z = (_matrix(g, n, d, torch.float32) + 0.5 * W[pos[:, 0].long()].float()).to(dt)
    if case["kind"] == "search":
        k = case["k"]
        s = {"case": case, "W": W, "Z": Z,
             "ws": torch.empty(xc.mine_workspace(n, L, d, k, code), dtype=torch.uint8, device=DEV),
             "out": torch.zeros((n, k), dtype=torch.int32, device=DEV)}
        if case["warm"]:
            # the search before, then some steps of training: a third of the rows have moved by a few per cent
            xc.mine_negatives(Z, W, k, workspace=s["ws"], out=s["out"])
            for r in range(0, L, 1 << 17):
                part = W[r:r + (1 << 17)]
                moved = torch.rand((part.shape[0], 1), generator=g, device=DEV) < 0.33
                step = torch.randn(part.shape, generator=g, device=DEV) * (0.02 * d ** -0.5)
                part.add_((step * moved).to(dt))
        return s
    B, k_p, k_h, k_r = case["B"], case["k_p"], case["k_h"], case["k_r"]
    n_neg = k_h + k_r
    neg = torch.cat([_shortlists(g, B, k_h, L),
                     torch.randint(0, L, (B, k_r), generator=g, device=DEV, dtype=torch.int32)], dim=1).contiguous()
    logq = torch.zeros((B, n_neg), dtype=torch.float32, device=DEV)
    logq[:, k_h:] = math.log(k_r / (L - k_h))
    P = B * (k_p + n_neg)
    return {"case": case, "W": W, "Z": Z, "pos": pos, "neg": neg, "logq": logq,
            "ws": torch.empty(xc.step_workspace(B, d, k_p, n_neg, code), dtype=torch.uint8, device=DEV),
            "out": {"loss": torch.zeros(1, dtype=torch.float32, device=DEV),
                    "dZ": torch.zeros((B, d), dtype=torch.float32, device=DEV),
                    "touched": torch.zeros(P, dtype=torch.int32, device=DEV),
                    "n_touched": torch.zeros(1, dtype=torch.int32, device=DEV)}}


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    if case["kind"] == "search":
        ids, scores = xc.mine_negatives(s["Z"], s["W"], case["k"], want_scores=True, workspace=s["ws"], out=s["out"],
                                        warm_margin=0.1 if case["warm"] else None)
        return {"ids": ids, "scores": scores}
    if case["kind"] == "sample":
        if case["form"] == "hard":
            neg, logq = xc.sample_negatives(s["shortlist"], case["k_h"], case["k_r"], case["L"], s["seed"],
                                            neg=s["neg"], logq=s["logq"])
        else:
            f = xc.sample_negatives_mixture if case["form"] == "mixture" else xc.sample_negatives_pps
            neg, logq = f(s["shortlist"], s["scores"], case["k_h"], case["k_r"], case["L"], s["seed"],
                          neg=s["neg"], logq=s["logq"])
        return {"neg": neg, "logq": logq}
    kind = xc.XC_LOSS_SOFTMAX if case["loss"] == "softmax" else xc.XC_LOSS_BCE
    r = xc.xc_step(s["Z"], s["W"], s["pos"], s["neg"], s["logq"], case["lr"], kind=kind, workspace=s["ws"],
                   out=s["out"])
    return {"loss": r["loss"], "dZ": r["dZ"], "touched": r["touched"], "n_touched": r["n_touched"], "W": s["W"]}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    if case["kind"] == "sample":
        n = case["k_h"] + case["k_r"]
        wide = case["k_h"] * (1 if case["form"] == "hard" else 4)      # ids, or ids and scores of a list twice as wide
        return {"bytes": case["B"] * (8.0 * n + 4.0 * wide), "flops": 0.0}
    row = case["d"] * _esize(case)
    if case["kind"] == "search":
        return {"bytes": float((case["L"] + case["Zq"]) * row + case["Zq"] * case["k"] * 8),
                "flops": 2.0 * case["Zq"] * case["L"] * case["d"]}
    B, L, k_h, k_r = case["B"], case["L"], case["k_h"], case["k_r"]
    k_pos = (case["k_p"] + 1) / 2
    pairs = B * (k_pos + k_h + k_r)
    # distinct rows: the uniform draws, and the hard ones by their law (density of u^4 over the ranks)
    t = (torch.arange(1000, dtype=torch.float64) + 0.5) / 1000
    dens = B * k_h * (t ** -0.75) / 4 / L + B * k_r / L
    rows = float(L * (1 - torch.exp(-dens)).mean())
    return {"bytes": 2.0 * rows * row + B * row + B * case["d"] * 4.0 + pairs * 8.0 + rows * 4.0,
            "flops": 6.0 * pairs * case["d"]}


def tolerance(case):
    # about four times what sums in another order (64 bits) were seen to differ by over these cases and drawn ones
    if case["kind"] == "search":
        # scores are sums of d products in fp32; ids may change places where two scores differ by less than that
        return {"rel": 1e-6, "max": 5e-6, "differ": 5e-4}
    if case["kind"] == "sample":
        return {"rel": 1e-6, "max": 1e-6}
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 5e-6}
    # an element of W whose sum lies at a rounding boundary moves by one bf16 unit (2^-7 of it at most)
    return {"rel": 2e-5, "max": 2e-2}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------
def _exact_search(s):
    case = s["case"]
    k, L = case["k"], case["L"]
    if case["Zq"] * L > 2e10 or case["Zq"] * L * case["d"] > 2e13:
        return None
    vals, ids = [], []
    zc = max(1, (1 << 28) // L)
    W = s["W"].double() if L * case["d"] < (1 << 31) else None
    for q in range(0, case["Zq"], zc):
        z = s["Z"][q:q + zc].double()
        if W is not None:
            sc = z @ W.T
        else:
            sc = torch.cat([z @ s["W"][r:r + (1 << 22)].double().T for r in range(0, L, 1 << 22)], dim=1)
        v, i = torch.topk(sc, k, dim=1)
        vals.append(v)
        ids.append(i.to(torch.int32))
    return {"ids": torch.cat(ids), "scores": torch.cat(vals)}


def _exact_step(s):
    case = s["case"]
    Z, W, pos, neg = s["Z"].double(), s["W"], s["pos"].long(), s["neg"].long()
    lq = s["logq"].double()
    B, d, L, k_p = case["B"], case["d"], case["L"], case["k_p"]
    ids = torch.cat([pos, neg], dim=1)
    ok = (ids >= 0) & (ids < L)
    for j in range(k_p):
        ok[:, k_p:] &= neg != pos[:, j:j + 1]
    labels = torch.unique(ids[ok])
    slot = torch.searchsorted(labels, ids.clamp(0, L - 1)).clamp_(max=labels.numel() - 1)
    dW = torch.zeros((labels.numel(), d), dtype=torch.float64, device=DEV)
    dZ = torch.empty((B, d), dtype=torch.float64, device=DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // (ids.shape[1] * d))
    for b in range(0, B, step):
        z, o = Z[b:b + step], ok[b:b + step]
        rows = W[ids[b:b + step].clamp(0, L - 1)].double()
        sc = torch.matmul(rows, z[:, :, None])[:, :, 0]
        y = torch.zeros_like(sc)
        y[:, :k_p] = 1.0
        q = torch.cat([torch.zeros_like(sc[:, :k_p]), lq[b:b + step]], dim=1)
        if case["loss"] == "bce":
            wt = torch.exp(-q) * o
            loss += (wt * (torch.nn.functional.softplus(sc) - y * sc)).sum()
            g = wt * (torch.sigmoid(sc) - y)
        else:
            t = torch.where(o, sc - q, torch.full_like(sc, -math.inf))
            npos = (o & (y > 0)).sum(dim=1, keepdim=True).double()
            lse = torch.logsumexp(t, dim=1, keepdim=True)
            yp = y * o / npos
            loss += (lse[:, 0] - torch.where(yp > 0, yp * t, torch.zeros_like(t)).sum(dim=1)).sum()
            g = torch.exp(t - lse) - yp
        g = g / B
        dZ[b:b + step] = torch.matmul(g[:, None, :], rows)[:, 0, :]
        for i in range(z.shape[0]):                       # a query's own slots: a fixed order of the sums
            dW.index_add_(0, slot[b + i], g[i][:, None] * z[i][None, :])
    touched = torch.zeros(ids.numel(), dtype=torch.int32, device=DEV)
    touched[:labels.numel()] = labels.to(torch.int32)
    out = torch.empty((L, d), dtype=torch.float64, device=DEV)
    for r in range(0, L, 1 << 20):
        out[r:r + (1 << 20)] = W[r:r + (1 << 20)]
    for r in range(0, labels.numel(), 1 << 20):
        out[labels[r:r + (1 << 20)]] -= case["lr"] * dW[r:r + (1 << 20)]
    return {"loss": loss / B, "dZ": dZ, "touched": touched,
            "n_touched": torch.tensor([labels.numel()], dtype=torch.int32, device=DEV), "W": out}


def exact(case, seed):
    if case["kind"] == "sample":
        if case["form"] != "hard":
            return None
        # the hard slots are copied with weight one; a uniform draw has log(k_r / (L - k_h))
        logq = torch.zeros((case["B"], case["k_h"] + case["k_r"]), dtype=torch.float64)
        logq[:, case["k_h"]:] = math.log(case["k_r"] / (case["L"] - case["k_h"]))
        return {"neg": None, "logq": logq}
    s = prepare(case, seed)
    return _exact_search(s) if case["kind"] == "search" else _exact_step(s)
