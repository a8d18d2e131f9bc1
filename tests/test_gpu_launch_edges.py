"""Edges of the launch structure: contexts and batches at the sizes where a kernel's path, its grid
or its list of hypergraphs changes, against the oracle bit for bit.
"""
import sys

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def J():
    import paper_2504_12013_amd.jet as jet
    return jet


@pytest.mark.parametrize("ks", [(4,), (2, 8, 32), (8, 8, 3)])
def test_batch_with_lone_hypergraphs(ks):
    """A batch in which some k has a single hypergraph (sizes on and off a 256-vertex tile)."""
    items = [(W.random_hypergraph(n, 2 * n, k, 70 + i), W.part_roundrobin(n, k, 70 + i))
             for i, (k, n) in enumerate(zip(ks, (1000, 1024, 300)))]
    say(f"lone hypergraphs, k = {ks}")
    batch = J().JetBatch([h for h, _ in items])
    parts = [torch.from_numpy(p).to("cuda") for _, p in items]
    _, stats, rcs = batch.refine(parts, tau=(0.75, 0.0), limit=6)
    for i, (hg, part) in enumerate(items):
        out, orc, ost, _ = O.refine(hg, part, tau=(0.75, 0.0), limit=6)
        assert rcs[i] == orc, i
        assert np.array_equal(parts[i].cpu().numpy(), out), i
        for key in ("km1_in", "km1_out", "iterations", "rebalance_rounds", "moves_executed", "balanced"):
            assert stats[i][key] == ost[key], (i, key)


@pytest.mark.parametrize("k", [2, 63, 64, 65, 128])
@pytest.mark.parametrize("max_iters", [1, 1000])
def test_loop_trace_at_block_counts(k, max_iters):
    """Whole refinements and their iteration records where the control kernel's waves fill up, also
    with rounds that end on their best partition (nothing to roll back) after one iteration."""
    hg = W.random_hypergraph(1500, 2600, k, 90 + k, smin=2, smax=9, vw_max=3, eps=0.1)
    part = W.part_roundrobin(hg.n, k, 3)
    say(f"k = {k}, max_iters = {max_iters}")
    kw = dict(tau=(0.75, 0.375, 0.0), limit=4, max_iters=max_iters)
    ref, orc, ost, otr = O.refine(hg, part, **kw)
    ctx = J().JetContext(hg)
    d = torch.from_numpy(part).to("cuda")
    rc, st, tr = ctx.refine(d, trace_cap=4096, **kw)
    ctx.close()
    assert rc == orc
    assert np.array_equal(d.cpu().numpy(), ref)
    for key in ("km1_in", "km1_out", "iterations", "rebalance_rounds", "moves_executed", "balanced"):
        assert st[key] == ost[key], key
    assert len(tr) == ost["iterations"]


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("n,k", [(40, 2), (1030, 2), (4097, 2), (9000, 2), (13000, 3)])
def test_rebalance_selection_list_lengths(n, k, order):
    """Rebalancing with most vertices in one block: selections from lists of a few entries up to
    past the 4,096 a workgroup keeps in registers, in all three orders, weighted vertices."""
    rng = np.random.default_rng(n + k)
    hg = W.random_hypergraph(n, 2 * n, k, 11 + n, smin=2, smax=5, vw_max=7, nw_max=2)
    part = np.where(rng.random(n) < 0.93, 0, rng.integers(0, k, n)).astype(np.int32)
    say(f"n = {n}, k = {k}, order {order}")
    ref, orc, ost = O.rebalance(hg, part, rb_unweighted=order)[:3]
    ctx = J().JetContext(hg)
    d = torch.from_numpy(part).to("cuda")
    rc, st = ctx.rebalance(d, rb_unweighted=order)
    ctx.close()
    assert rc == orc
    assert np.array_equal(d.cpu().numpy(), ref)
    assert st["rebalance_rounds"] == ost["rebalance_rounds"]


@pytest.mark.parametrize("divisor", [0, 16, 1 << 20])
@pytest.mark.parametrize("k", [5, 64, 100])
def test_application_paths(divisor, k):
    """Both ways of applying a move list (per move, per net) and the switch between them, on nets of
    one pin (chunks full by nets, not pins), of a chunk's 64 pins, just above, and above 1,024."""
    rng = np.random.default_rng(k)
    n = 3000
    sizes = np.concatenate([np.ones(200, int), rng.integers(2, 9, 3000), [63, 64, 65, 66, 255, 256, 257, 1023, 1024,
                                                                        1025, 2500]])
    nets = [np.sort(rng.choice(n, s, replace=False)) for s in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    hg = W.Hypergraph(n=n, m=len(nets), off=off, pins=np.concatenate(nets).astype(np.int32), k=k, eps=0.05)
    part = W.part_uniform(n, k, 5)
    say(f"divisor {divisor}, k = {k}")
    kw = dict(tau=(0.75, 0.0), limit=5)
    ref, orc, ost, _ = O.refine(hg, part, **kw)
    ctx = J().JetContext(hg)
    ctx.set_option(J().JET_OPT_APPLY_DIVISOR, divisor)
    d = torch.from_numpy(part).to("cuda")
    rc, st, _ = ctx.refine(d, **kw)
    assert rc == orc
    assert np.array_equal(d.cpu().numpy(), ref)
    assert st["km1_out"] == ost["km1_out"] == ctx.km1(d)
    ctx.close()


@pytest.mark.parametrize("k,nw_max", [(2, 1), (7, 3), (16, 1), (33, 1), (64, 1), (64, 4), (128, 1)])
@pytest.mark.parametrize("hubs", [1, 9, 700])
def test_hub_vertices(hubs, k, nw_max):
    """Vertices with more than 256 incident nets, few and many of them, beside light ones: candidates,
    whole refinements and rebalancing from an overloaded start (waves share one hub, or take many)."""
    rng = np.random.default_rng(hubs * 131 + k)
    n, m = hubs + 500, 400 if hubs > 100 else 4000
    nets = []
    for e in range(m):
        heavy = rng.choice(hubs, max(1, int(0.9 * hubs)), replace=False)
        light = hubs + rng.choice(500, 3, replace=False)
        nets.append(np.sort(np.concatenate([heavy, light])))
    off = np.concatenate([[0], np.cumsum([len(e) for e in nets])]).astype(np.int64)
    nw = rng.integers(1, nw_max + 1, m).astype(np.int32) if nw_max > 1 else None
    vw = rng.integers(1, 4, n).astype(np.int32)
    hg = W.Hypergraph(n=n, m=m, off=off, pins=np.concatenate(nets).astype(np.int32), k=k, eps=0.1, net_w=nw, vtx_w=vw)
    part = W.part_uniform(n, k, 9)
    say(f"{hubs} hubs, k = {k}, net weights up to {nw_max}")
    ctx = J().JetContext(hg)
    d = torch.from_numpy(part).to("cuda")
    t, g, im = ctx.candidates(d, 24576)
    ot, og, oim = O.candidates(hg, part, 24576)
    assert np.array_equal(im.cpu().numpy(), oim)
    assert np.array_equal(t.cpu().numpy(), ot)
    sel = ot >= 0
    assert np.array_equal(g.cpu().numpy()[sel], og[sel])
    ref, orc, ost, _ = O.refine(hg, part, tau=(0.75, 0.0), limit=3)
    rc, st, _ = ctx.refine(d, tau=(0.75, 0.0), limit=3)
    assert rc == orc and np.array_equal(d.cpu().numpy(), ref)
    over = np.where(rng.random(n) < 0.7, 0, part).astype(np.int32)
    oref, orc, ost = O.rebalance(hg, over)[:3]
    d = torch.from_numpy(over).to("cuda")
    rc, st = ctx.rebalance(d)
    ctx.close()
    assert rc == orc and np.array_equal(d.cpu().numpy(), oref)
    assert st["rebalance_rounds"] == ost["rebalance_rounds"]


@pytest.mark.parametrize("B", [31, 32, 33, 2047, 2048, 2049, 5000])
def test_network_batch_edges(B):
    """Forward and gradient of the temperature network at the edges of the 32 samples a batch sum holds
    in flight and of the 2,048 waves of a forward launch.  The batch sums run in sample order in FP32:
    rounding grows at most with B half-ulps of terms of at most a few units."""
    from oracle import mlp as M
    rng = np.random.default_rng(B)
    net = J().TauNet(seed=B)
    th, mean, std = net.get()
    X = (rng.normal(size=(B, 16)) * std + mean).astype(np.float32)
    t = rng.uniform(0, 1, B).astype(np.float32)
    say(f"network, batch of {B}")
    y = net.forward(torch.from_numpy(X)).cpu().numpy()
    assert np.max(np.abs(y - M.forward(th, M.standardise(X, mean, std))[0])) <= 1e-5
    loss, g = net.grad(torch.from_numpy(X), torch.from_numpy(t))
    ref_loss, ref_g = M.grad(th, M.standardise(X, mean, std), t)
    tol = 4.0 * (B + 256) * 2.0 ** -24
    assert abs(loss - ref_loss) <= tol
    assert np.all(np.abs(g.cpu().numpy() - ref_g) <= tol * np.maximum(1.0, np.abs(ref_g)))


@pytest.mark.parametrize("members", [63, 64, 65, 300])
@pytest.mark.parametrize("size", [32, 33, 34, 256, 257, 258])
def test_coarsening_table_and_group_edges(size, members):
    """Vertices whose rating table is the last of one size or the first of the next (a net of `size`
    pins alone around them), beside a centre that `members` leaves propose to in one sub-round."""
    star = [[0, i] for i in range(1, members + 1)]
    n0 = members + 1
    nets = star + [list(range(n0 + j * size, n0 + (j + 1) * size)) for j in range(6)]
    n = n0 + 6 * size
    off = np.concatenate([[0], np.cumsum([len(e) for e in nets])]).astype(np.int64)
    vw = (np.arange(n) % 4 + 1).astype(np.int32)
    hg = W.Hypergraph(n=n, m=len(nets), off=off, pins=np.concatenate(nets).astype(np.int32), k=2, eps=0.05, vtx_w=vw)
    order = np.concatenate([[0], np.random.default_rng(size).permutation(np.arange(1, n))]).astype(np.int32)
    say(f"net of {size} pins, group of {members}")
    for wmax, first in ((20, 100), (members, 0)):
        olab, ocnt = O.coarsen(hg, order, wmax, first, 1)
        ctx = J().JetContext(hg)
        lab, cnt = ctx.coarsen(torch.from_numpy(order).to("cuda"), wmax, first, 1)
        ctx.close()
        assert cnt == ocnt
        assert np.array_equal(lab.cpu().numpy(), olab)


@pytest.mark.parametrize("replays", [1, 2])
@pytest.mark.parametrize("overloaded", [False, True])
def test_loop_launches_what_the_loop_asks_for(replays, overloaded):
    """One piece in flight: exactly a piece per Jet phase, rebalancing round and rollback; two: at most
    one more per piece, and the same refinement."""
    hg = W.random_hypergraph(3000, 5000, 6, 21, smin=2, smax=7, vw_max=3, eps=0.05)
    part = W.part_roundrobin(hg.n, 6, 2)
    if overloaded:
        part[: hg.n // 3] = 0
    kw = dict(tau=(0.75, 0.375, 0.0), limit=5)
    say(f"pieces in flight {replays}, overloaded start {overloaded}")
    ref, orc, ost, otr = O.refine(hg, part, **kw)
    ctx = J().JetContext(hg)
    ctx.set_option(J().JET_OPT_REPLAYS, replays)
    d = torch.from_numpy(part).to("cuda")
    rc, st, tr = ctx.refine(d, trace_cap=4096, **kw)
    need = ost["iterations"] + ost["rebalance_rounds"] + 3
    pieces = ctx.loop_counts()[1]
    ctx.close()
    assert rc == orc and tr == otr
    assert np.array_equal(d.cpu().numpy(), ref)
    assert pieces == need if replays == 1 else need <= pieces <= 2 * need


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("nw_max,vw_max", [(1, 1), (1, 1 << 17), (1 << 15, 1), (300, 300)])
def test_split_selection_digits(nw_max, vw_max, order, monkeypatch):
    """The grid-wide first pass on priorities inside and far outside the range its digit resolves, with
    lists of a tile and of several per workgroup."""
    monkeypatch.setenv("JET_SEL_SPLIT_MIN", "0")
    rng = np.random.default_rng(nw_max + vw_max)
    n, k = 12000, 3
    hg = W.random_hypergraph(n, 2 * n, k, 5, smin=2, smax=5, vw_max=vw_max, nw_max=nw_max)
    part = np.where(rng.random(n) < 0.9, 1, rng.integers(0, k, n)).astype(np.int32)
    say(f"net weights to {nw_max}, vertex weights to {vw_max}, order {order}")
    ref, orc, ost = O.rebalance(hg, part, rb_unweighted=order)[:3]
    ctx = J().JetContext(hg)
    d = torch.from_numpy(part).to("cuda")
    rc, st = ctx.rebalance(d, rb_unweighted=order)
    ctx.close()
    assert rc == orc
    assert np.array_equal(d.cpu().numpy(), ref)
    assert st["rebalance_rounds"] == ost["rebalance_rounds"]


@pytest.mark.parametrize("graph", [0, 1])
def test_afterburner_branches(graph):
    """Nets of every size class at the pin count from which their kernels run beside each other, from a
    captured graph and launched one by one, twice on one context."""
    rng = np.random.default_rng(17)
    n, k = 20000, 9
    sizes = np.concatenate([rng.integers(2, 9, 60000), np.full(300, 200), np.full(120, 900), np.full(20, 6000)])
    nets = [np.sort(rng.choice(n, s, replace=False)) for s in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    hg = W.Hypergraph(n=n, m=len(nets), off=off, pins=np.concatenate(nets).astype(np.int32), k=k, eps=0.05)
    assert hg.p >= 1 << 19
    part = W.part_uniform(n, k, 4)
    say(f"{hg.p} pins, graph {graph}")
    kw = dict(tau=(0.75,), limit=3, max_iters=6)
    ref, orc, ost, _ = O.refine(hg, part, **kw)
    ctx = J().JetContext(hg)
    ctx.set_option(J().JET_OPT_GRAPH, graph)
    for _ in range(2):
        d = torch.from_numpy(part).to("cuda")
        rc, st, _ = ctx.refine(d, **kw)
        assert rc == orc and st["km1_out"] == ost["km1_out"]
        assert np.array_equal(d.cpu().numpy(), ref)
    ctx.close()


@pytest.mark.parametrize("k", [2, 3, 4, 63, 64, 65, 124, 128])
def test_counts_where_rows_and_chunks_end(k):
    """Pin counts (rows of every alignment, also in a caller's table at an odd offset) and the metric on
    nets of one pin, of a chunk's 64 pins and above, and a partition out of range."""
    rng = np.random.default_rng(k)
    n = 3000
    sizes = np.concatenate([np.ones(70, int), np.full(40, 2), rng.integers(2, 20, 900), [63, 64, 65, 1023, 1024, 1025]])
    nets = [np.sort(rng.choice(n, s, replace=False)) for s in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    hg = W.Hypergraph(n=n, m=len(nets), off=off, pins=np.concatenate(nets).astype(np.int32), k=k, eps=0.05)
    part = W.part_uniform(n, k, 8)
    say(f"k = {k}")
    ref = np.zeros((hg.m, k), np.int64)
    np.add.at(ref, (np.repeat(np.arange(hg.m), sizes), part[hg.pins]), 1)
    ctx = J().JetContext(hg)
    d = torch.from_numpy(part).to("cuda")
    assert np.array_equal(ctx.phi(d).cpu().numpy().reshape(hg.m, k), ref)
    odd = torch.full((hg.m * k + 2,), -7, dtype=torch.int32, device="cuda")
    J().jet_phi(ctx.h, d, odd[1:-1])
    assert np.array_equal(odd[1:-1].cpu().numpy().reshape(hg.m, k), ref)
    assert int(odd[0]) == int(odd[-1]) == -7
    assert ctx.km1(d) == int(((ref > 0).sum(axis=1) - 1).clip(min=0).sum())
    bad = part.copy()
    bad[17] = k
    with pytest.raises(J().JetError, match="part"):
        ctx.km1(torch.from_numpy(bad).to("cuda"))
    assert ctx.km1(d) == O.km1(hg, part)
    ctx.close()
