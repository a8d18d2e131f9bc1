"""The work this framework is used for, as cases that can be timed and compared.

Every case is one pass through the package's public entry points on seeded synthetic inputs: Jet
refinement of one level (small, ordinary, large; VLSI-like, row-net, SAT-like, graph), a multilevel
run over a hierarchy, a batch of small hypergraphs, rebalancing of an overloaded partition, a
clustering pass, a round of flow refinement, and training of the temperature network.  Inputs are
drawn on the GPU with torch, in the shapes of the benchmark's generators.

A case's "kind" says which of these it is; "family" the shape of its hypergraph:
  uniform  net sizes U[2, 8], pins uniform over all vertices
  vlsi     net sizes 2 + Geom(0.4) up to 64, pins within 2,000 IDs of an anchor, nets in anchor order
  rownet   net i around vertex i, sizes Zipf(2.1) on [2, 10^4], pins within max(4 |e|, 2048) of i
  sat      sizes Zipf(1.8) with a heavy tail, pins uniform over all vertices
  mesh     a triangulated grid: every net an edge
"wv" / "we" are the largest vertex / net weight (1: unit weights, no array is passed).
"sched" is the temperature schedule: "paper" (0.75 / 0.375 / 0, limit 8), "single" (0.75, limit 12)
or "net" (temperatures from the trained network, limit 8).
"""
import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_2504_12013_amd as jet
from paper_2504_12013_amd.jet import JetBatch, JetContext, TauNet

EPS = 0.03
SCHED = {"paper": dict(tau=(0.75, 0.375, 0.0), limit=8), "single": dict(tau=(0.75,), limit=12),
         "net": dict(tau=(0.75, 0.375, 0.0), limit=8)}
ROWNET_CAP, SAT_PINS_PER_VERTEX, SAT_WEIGHT = 10_000, 10, 8
TAU_BATCH = 256  # the training driver's minibatch


def listed():
    return [
        # the smallest call: a parity-sized hypergraph, latency and launches only
        dict(name="uniform-2k-k4", kind="refine", family="uniform", n=2000, m=4000, k=4, wv=1, we=1, sched="single"),
        # an ordinary odd-sized level with both weights, as a contracted level has
        dict(name="vlsi-50k-k11-weighted", kind="refine", family="vlsi", n=50_021, m=55_001, k=11, wv=4, we=3,
             sched="paper"),
        # the netlist benchmark's size
        dict(name="vlsi-1M-k8", kind="refine", family="vlsi", n=1_000_000, m=1_100_000, k=8, wv=4, we=1,
             sched="single"),
        # the finest level of a row-net run
        dict(name="rownet-1M-k64", kind="refine", family="rownet", n=1_000_003, m=1_000_003, k=64, wv=1, we=1,
             sched="paper"),
        # the headline's shape: a hierarchy refined coarsest to finest
        dict(name="vcycle-rownet-1M-k64", kind="vcycle", family="rownet", n=1_000_000, m=1_000_000, k=64, wv=1, we=1,
             levels=10, sched="paper"),
        # heavy-tailed nets, many blocks, weighted vertices
        dict(name="sat-300k-k128", kind="refine", family="sat", n=300_000, m=0, k=128, wv=8, we=1, sched="single"),
        # the graph benchmark's size
        dict(name="mesh-4M-k64", kind="refine", family="mesh", n=2048 * 2048, m=0, k=64, wv=1, we=1, sched="paper"),
        # many small instances in one call
        dict(name="batch-96", kind="batch", family="zipf", n=30_000, count=96, sched="single"),
        # a partition projected from elsewhere that misses the balance constraint
        dict(name="rebalance-sat-1M-k128", kind="rebalance", family="sat", n=1_000_000, m=0, k=128, wv=8, we=1),
        # one coarsening step of a netlist
        dict(name="coarsen-vlsi-1M", kind="coarsen", family="vlsi", n=1_000_000, m=1_100_000, k=8, wv=4, we=1),
        # one round of flow refinement after Jet
        dict(name="flows-vlsi-20k-k8", kind="flow", family="vlsi", n=20_000, m=22_000, k=8, wv=4, we=1),
        # an epoch of the temperature network's training, and its predictions
        dict(name="taunet-epoch-2k", kind="tau", samples=2048, epochs=1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; none costs more than the hierarchy or the flow round."""
    kind = rng.choice(["refine"] * 7 + ["vcycle", "batch", "rebalance", "coarsen", "flow", "tau"])
    if kind == "tau":
        return dict(kind=kind, samples=_logint(rng, 1, 4096), epochs=rng.choice([1, 2]))
    if kind == "batch":
        return dict(kind=kind, family="zipf", n=_logint(rng, 2000, 30_000), count=rng.randint(3, 96),
                    sched=rng.choice(["paper", "single"]))
    if kind == "flow":
        n = _logint(rng, 1000, 20_000)
        return dict(kind=kind, family="vlsi", n=n, m=int(1.1 * n), k=rng.randint(2, 8), wv=rng.choice([1, 4]), we=1)
    if kind == "coarsen":
        n = _logint(rng, 1000, 1_000_000)
        return dict(kind=kind, family="vlsi", n=n, m=int(1.1 * n), k=8, wv=rng.choice([1, 4]), we=rng.choice([1, 3]))
    if kind == "vcycle":
        n = _logint(rng, 50_000, 500_000)
        return dict(kind=kind, family="rownet", n=n, m=n, k=rng.choice([8, 16, 27, 64]), wv=1, we=1,
                    levels=rng.randint(4, 9), sched="paper")
    if kind == "rebalance":
        return dict(kind=kind, family="sat", n=_logint(rng, 3000, 1_000_000), m=0, k=rng.choice([2, 8, 27, 64, 128]),
                    wv=rng.choice([1, 8]), we=1)
    family = rng.choice(["uniform", "vlsi", "rownet", "sat", "mesh"])
    n = _logint(rng, 500, {"uniform": 300_000, "vlsi": 1_000_000, "rownet": 1_000_000, "sat": 150_000,
                           "mesh": 4_000_000}[family])
    m = {"uniform": int(2 * n), "vlsi": int(1.1 * n), "rownet": n, "sat": 0, "mesh": 0}[family]
    if family == "mesh":
        side = max(2, int(math.sqrt(n)))
        n = side * (side + rng.randint(0, 3))
    return dict(kind=kind, family=family, n=n, m=m, k=rng.choice([2, 4, 8, 11, 16, 27, 32, 64, 65, 128]),
                wv=rng.choice([1, 4, SAT_WEIGHT]), we=rng.choice([1, 1, 3]),
                sched=rng.choice(["paper", "paper", "single", "net"]))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rand(count, g):
    return torch.rand(count, generator=g, device="cuda", dtype=torch.float64)


def _randint(lo, hi, count, g):
    return torch.randint(lo, hi, (count,), generator=g, device="cuda")


def _zipf(count, a, cap, g):
    """Sizes in [2, cap] with P(s) proportional to s^-a."""
    w = torch.arange(2, cap + 1, device="cuda", dtype=torch.float64).pow_(-a)
    cdf = w.cumsum(0)
    return 2 + torch.searchsorted(cdf, _rand(count, g) * cdf[-1]).clamp_(max=cap - 2)


def _csr(net, pin, m, n):
    """CSR of the (net, pin) pairs: repeated pins and nets of fewer than two pins dropped."""
    key = torch.unique(net * n + pin)
    net, pin = key // n, key % n
    size = torch.bincount(net, minlength=m)
    keep = size >= 2
    pin = pin[keep[net]]
    size = size[keep]
    off = torch.zeros(size.numel() + 1, dtype=torch.int64, device="cuda")
    off[1:] = size.cumsum(0)
    return off, pin.to(torch.int32), keep


def _weights(count, top, g):
    return None if top <= 1 else _randint(1, top + 1, count, g).to(torch.int32)


def _hypergraph(case, g):
    family, n, m, k = case["family"], case["n"], case["m"], case["k"]
    if family == "mesh":
        cols = max(2, int(math.sqrt(n)))
        rows = n // cols
        n = rows * cols
        i = torch.arange(n, device="cuda").view(rows, cols)
        ends = [torch.stack([i[:, :-1].reshape(-1), i[:, 1:].reshape(-1)], 1),
                torch.stack([i[:-1].reshape(-1), i[1:].reshape(-1)], 1),
                torch.stack([i[:-1, :-1].reshape(-1), i[1:, 1:].reshape(-1)], 1)]
        e = torch.cat(ends)
        e = e[torch.sort(e[:, 0], stable=True)[1]]
        off = torch.arange(0, 2 * e.shape[0] + 1, 2, device="cuda")
        pins = e.reshape(-1).to(torch.int32)
    else:
        if family == "uniform":
            size = _randint(2, 9, m, g)
        elif family == "vlsi":
            size = 2 + (torch.log1p(-_rand(m, g)) / math.log(1 - 0.4)).long().clamp_(max=62)
        elif family == "rownet":
            size = _zipf(m, 2.1, min(ROWNET_CAP, n), g)
        else:
            total = SAT_PINS_PER_VERTEX * n
            size = _zipf(max(16, total // 8), 1.8, max(64, n // 20), g)
            m = min(size.numel(), int(torch.searchsorted(size.cumsum(0), total)) + 1)
            size = size[:m]
        p = int(size.sum())
        net = torch.repeat_interleave(torch.arange(m, device="cuda"), size)
        if family in ("uniform", "sat"):
            pin = _randint(0, n, p, g)
        else:
            if family == "vlsi":
                anchor, window = torch.sort(_randint(0, n, m, g))[0], torch.full((m,), 2000, device="cuda")
            else:
                anchor, window = torch.arange(m, device="cuda"), (4 * size).clamp_(min=2048)
            lo = (anchor - window).clamp_(min=0)
            hi = (anchor + window).clamp_(max=n - 1)
            pin = lo[net] + (_rand(p, g) * (hi - lo + 1)[net]).long()
            pin.clamp_(max=n - 1)
        off, pins, _ = _csr(net, pin, m, n)
    m = off.numel() - 1
    return SimpleNamespace(n=n, m=m, off=off, pins=pins, k=k, eps=EPS, net_w=_weights(m, case["we"], g),
                           vtx_w=_weights(n, case["wv"], g))


def _ranges_with_noise(n, k, share, g):
    part = (torch.arange(n, device="cuda") * k // n)
    at = torch.randperm(n, generator=g, device="cuda")[:max(1, int(share * n))]
    part[at] = _randint(0, k, at.numel(), g)
    return part.to(torch.int32)


def _round_robin(n, k, g):
    return (torch.randperm(n, generator=g, device="cuda") % k).to(torch.int32)


def _coarsened(hg, g):
    """The hypergraph after one random matching along nets: (coarse hypergraph, parent[n])."""
    n, m = hg.n, hg.m
    net = torch.repeat_interleave(torch.arange(m, device="cuda"), hg.off[1:] - hg.off[:-1])
    pin = hg.pins.long()
    mate = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    for _ in range(6):
        free = mate[pin] < 0
        e, v = net[free], pin[free]
        if v.numel() == 0:
            break
        choice = torch.full((n,), -1, dtype=torch.int64, device="cuda")
        choice.scatter_reduce_(0, v, (_randint(0, 1 << 31, v.numel(), g) << 32) | e, "amax")
        v = torch.nonzero(choice >= 0).view(-1)
        e = choice[v] & 0xffffffff
        order = torch.sort(e * (1 << 31) + _randint(0, 1 << 31, v.numel(), g))[1]
        v, e = v[order], e[order]
        start = torch.searchsorted(e, e)
        rank = torch.arange(v.numel(), device="cuda") - start
        first = torch.nonzero((rank[:-1] % 2 == 0) & (e[:-1] == e[1:])).view(-1)
        a, b = v[first], v[first + 1]
        mate[a], mate[b] = b, a
    ids = torch.arange(n, device="cuda")
    head = torch.where(mate >= 0, torch.minimum(ids, mate), ids)
    # coarse IDs in a random order of the pairs, as a random visiting order gives them
    heads = torch.nonzero(head == ids).view(-1)
    name = torch.empty(n, dtype=torch.int64, device="cuda")
    name[heads] = torch.randperm(heads.numel(), generator=g, device="cuda")
    parent = name[head]
    nc = heads.numel()
    vw = torch.ones(n, dtype=torch.int32, device="cuda") if hg.vtx_w is None else hg.vtx_w
    cw = torch.zeros(nc, dtype=torch.int32, device="cuda").index_add_(0, parent, vw)
    off, pins, keep = _csr(net, parent[pin], m, nc)
    return SimpleNamespace(n=nc, m=off.numel() - 1, off=off, pins=pins, k=hg.k, eps=hg.eps,
                           net_w=None if hg.net_w is None else hg.net_w[keep], vtx_w=cw), parent


def _tau_data(case, seed):
    g = _gen(seed)
    x = torch.randn(case["samples"], 16, generator=g, device="cuda") * 2.0 + 3.0
    t = torch.rand(case["samples"], generator=g, device="cuda")
    order = torch.randperm(case["samples"], generator=g, device="cuda")
    r = np.random.default_rng(seed)
    bound = lambda fan: math.sqrt(6.0 / fan)  # noqa: E731
    theta = np.concatenate([r.uniform(-bound(16), bound(16), 1024), np.zeros(64),
                            r.uniform(-bound(64), bound(64), 4096), np.zeros(64),
                            r.uniform(-bound(64), bound(64), 64), np.zeros(1)]).astype(np.float32)
    return x, t, order, theta


def prepare(case, seed):
    kind = case["kind"]
    if kind == "tau":
        x, t, order, theta = _tau_data(case, seed)
        return dict(kind=kind, x=x, t=t, order=order, theta=theta, net=TauNet(seed), epochs=case["epochs"],
                    mean=np.full(16, 3.0, np.float32), std=np.full(16, 2.0, np.float32))
    g = _gen(seed)
    if kind == "batch":
        hgs, starts = [], []
        for i in range(case["count"]):  # sizes spread evenly over the logarithm, k in turn
            n = int(round(1000 * (case["n"] / 1000) ** ((i + 0.5) / case["count"])))
            k = (2, 8, 32)[i % 3]
            m = int(round(1.2 * n))
            size = _zipf(m, 2.1, min(1000, n), g)
            net = torch.repeat_interleave(torch.arange(m, device="cuda"), size)
            off, pins, _ = _csr(net, _randint(0, n, net.numel(), g), m, n)
            hgs.append(SimpleNamespace(n=n, m=off.numel() - 1, off=off, pins=pins, k=k, eps=EPS, net_w=None,
                                       vtx_w=None))
            starts.append(_round_robin(n, k, g))
        return dict(kind=kind, batch=JetBatch(hgs), starts=starts, sched=SCHED[case["sched"]])
    hg = _hypergraph(case, g)
    if kind == "vcycle":
        hgs, parents = [hg], []
        for _ in range(case["levels"] - 1):
            coarse, parent = _coarsened(hgs[-1], g)
            hgs.append(coarse)
            parents.append(parent)
        # heaviest first into the blocks in turn: a weight-only balanced start
        c = hgs[-1]
        start = torch.empty(c.n, dtype=torch.int32, device="cuda")
        start[torch.sort(c.vtx_w, descending=True, stable=True)[1]] = (
            torch.arange(c.n, device="cuda") % c.k).to(torch.int32)
        return dict(kind=kind, ctxs=[JetContext(h) for h in hgs], parents=parents, start=start,
                    sched=SCHED[case["sched"]])
    ctx = JetContext(hg)
    state = dict(kind=kind, ctx=ctx, n=hg.n)
    if kind == "coarsen":
        total = hg.n if hg.vtx_w is None else int(hg.vtx_w.sum())
        state.update(order=torch.randperm(hg.n, generator=g, device="cuda").to(torch.int32),
                     wmax=-(-total // (160 * hg.k)))
    elif kind == "rebalance":
        # blocks of uneven popularity: some far over the limit, some far under it
        share = 0.3 + _rand(hg.k, g)
        part = torch.searchsorted(share.cumsum(0), _rand(hg.n, g) * share.sum()).clamp_(max=hg.k - 1)
        state.update(start=part.to(torch.int32))
    elif kind == "flow":
        part = _ranges_with_noise(hg.n, hg.k, 0.1, g)
        ctx.refine(part, **SCHED["paper"])
        state.update(start=part)
    else:
        start = {"uniform": lambda: _round_robin(hg.n, hg.k, g),
                 "sat": lambda: _round_robin(hg.n, hg.k, g)}.get(
            case["family"], lambda: _ranges_with_noise(hg.n, hg.k, 0.05 if case["family"] == "mesh" else 0.1, g))()
        state.update(start=start, sched=SCHED[case["sched"]], net=None)
        if case["sched"] == "net":
            state["net"] = TauNet(path=os.path.join(os.path.dirname(jet.__file__), "tau_net.bin"))
    return state


# ------------------------------------------------------------------ one pass

def _epochs(s):
    """The training driver's loop: minibatch Adam steps, then the network's predictions."""
    net, losses = s["net"], []
    net.set(s["theta"], s["mean"], s["std"])
    for _ in range(s["epochs"]):
        for idx in s["order"].split(TAU_BATCH):
            losses.append(net.train_step(s["x"][idx], s["t"][idx], lr=1e-3))
    return {"tau": net.forward(s["x"]), "losses": np.array(losses, np.float32), "params": net.get()[0]}


def run(s):
    kind = s["kind"]
    if kind == "tau":
        return _epochs(s)
    if kind == "coarsen":
        label, clusters = s["ctx"].coarsen(s["order"], s["wmax"])
        return {"label": label, "clusters": clusters}
    if kind == "batch":
        parts = [p.clone() for p in s["starts"]]
        _, stats, _ = s["batch"].refine(parts, **s["sched"])
        return {"parts": torch.cat(parts), "km1": np.array([x["km1_out"] for x in stats]),
                "iterations": np.array([x["iterations"] for x in stats])}
    part = s["start"].clone()
    if kind == "vcycle":
        ctxs, iterations = s["ctxs"], 0
        for lvl in range(len(ctxs) - 1, -1, -1):
            if lvl < len(ctxs) - 1:
                part = part[s["parents"][lvl]].contiguous()
            _, st, _ = ctxs[lvl].refine(part, **s["sched"])
            iterations += st["iterations"]
        return {"part": part, "km1": st["km1_out"], "iterations": iterations}
    if kind == "rebalance":
        _, st = s["ctx"].rebalance(part)
        return {"part": part, "km1": st["km1_out"], "rounds": st["rebalance_rounds"]}
    if kind == "flow":
        st = s["ctx"].flow_refine(part, max_rounds=1)
        return {"part": part, "km1": st["km1_out"], "flow_calls": st["flow_calls"], "moved": st["moved"]}
    if s["net"] is not None:
        _, st, tau = s["ctx"].refine_learned(part, s["net"], 0, 1, s["n"], **s["sched"])
        return {"part": part, "km1": st["km1_out"], "iterations": st["iterations"], "tau": np.array(tau, np.float32)}
    _, st, _ = s["ctx"].refine(part, **s["sched"])
    return {"part": part, "km1": st["km1_out"], "iterations": st["iterations"]}


# ------------------------------------------------------------------ what a pass cannot do without

def _zipf_mean(a, cap):
    s = np.arange(2, cap + 1, dtype=np.float64)
    w = s ** -a
    return float((s * w).sum() / w.sum())


def _nets_and_pins(case):
    n, m = case["n"], case["m"]
    if case["family"] == "uniform":
        return m, 5.0 * m
    if case["family"] == "vlsi":
        return m, 3.5 * m
    if case["family"] == "rownet":
        return m, _zipf_mean(2.1, min(ROWNET_CAP, n)) * m
    if case["family"] == "sat":
        p = SAT_PINS_PER_VERTEX * n
        return p / _zipf_mean(1.8, max(64, n // 20)), float(p)
    return 3.0 * n, 6.0 * n


def work(case):
    """The hypergraph read once, the partition (or labels) read and written once; for the network
    its products (forward, both backward products), the samples and the parameters."""
    if case["kind"] == "tau":
        rows = case["samples"] * case["epochs"]
        return {"bytes": 4.0 * (17 * rows + 18 * case["samples"] + 2 * 5313),
                "flops": 2.0 * 5184 * (3 * rows + case["samples"])}
    if case["kind"] == "batch":
        lo, hi = math.log(1000), math.log(max(1001, case["n"]))
        n = case["count"] * (math.exp(hi) - math.exp(lo)) / (hi - lo)
        return {"bytes": 1.2 * n * (8 + 4 * _zipf_mean(2.1, 1000)) + 8 * n, "flops": 0.0}
    m, p = _nets_and_pins(case)
    one = 8.0 * m + 4.0 * p + 8.0 * case["n"] + 4.0 * case["n"] * (case["wv"] > 1) + 4.0 * m * (case["we"] > 1)
    if case["kind"] == "vcycle":  # nets and pins shrink slowly, vertices halve
        one = sum((8.0 * m + 4.0 * p) * 0.95 ** lvl + 12.0 * case["n"] * 0.5 ** lvl for lvl in range(case["levels"]))
    return {"bytes": one, "flops": 0.0}


def exact(case, seed):
    """The network's training in 64 bits (Adam as published, mean squared error); the other cases
    return partitions, labels and counts, which are whole numbers."""
    if case["kind"] != "tau":
        return None
    x, t, order, theta = (v.cpu().numpy() if isinstance(v, torch.Tensor) else v for v in _tau_data(case, seed))
    x, t, th = (x.astype(np.float64) - 3.0) / 2.0, t.astype(np.float64), theta.astype(np.float64)

    def unpack(v):
        return (v[:1024].reshape(64, 16), v[1024:1088], v[1088:5184].reshape(64, 64), v[5184:5248], v[5248:5312],
                v[5312:])

    def forward(v, a):
        w1, b1, w2, b2, w3, b3 = unpack(v)
        h1 = np.maximum(a @ w1.T + b1, 0)
        h2 = np.maximum(h1 @ w2.T + b2, 0)
        return h1, h2, 1 / (1 + np.exp(-(h2 @ w3 + b3[0])))

    mo, ve, step, losses = np.zeros_like(th), np.zeros_like(th), 0, []
    for _ in range(case["epochs"]):
        for i in range(0, len(x), TAU_BATCH):
            idx = order[i:i + TAU_BATCH]
            a, y = x[idx], t[idx]
            h1, h2, out = forward(th, a)
            losses.append(float(np.mean((out - y) ** 2)))
            w1, _, w2, _, w3, _ = unpack(th)
            d3 = 2 * (out - y) / len(a) * out * (1 - out)
            d2 = np.outer(d3, w3) * (h2 > 0)
            d1 = (d2 @ w2) * (h1 > 0)
            gr = np.concatenate([(d1.T @ a).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), h2.T @ d3,
                                 [d3.sum()]])
            step += 1
            mo = 0.9 * mo + 0.1 * gr
            ve = 0.999 * ve + 0.001 * gr * gr
            th = th - 1e-3 * (mo / (1 - 0.9 ** step)) / (np.sqrt(ve / (1 - 0.999 ** step)) + 1e-8)
    return {"tau": forward(th, x)[2], "losses": np.array(losses), "params": th}
