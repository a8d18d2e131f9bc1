"""The hub pass in each of its forms -- bit-sliced counts of one, two and four words (unit net weights), lane
groups of 1, 2, 4, 8 and 16 (with net weights) -- on hubs whose nets fill one workgroup's share, just
exceed it, or take several, alone and among many: candidates, rebalancing rounds and refinements against
the oracle."""
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


def dev(a, dtype=torch.int32):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


def hypergraph(k, degrees, nw_max, seed):
    """Hubs of the given degrees among 400 light vertices; 6,000 nets."""
    rng = np.random.default_rng(seed)
    m, light, hubs = 6000, 400, len(degrees)
    net = [np.repeat(np.arange(m), 2)]
    pin = [hubs + np.concatenate([rng.choice(light, 2, replace=False) for _ in range(m)])]
    for v, d in enumerate(degrees):
        net.append(rng.choice(m, d, replace=False))
        pin.append(np.full(d, v))
    net, pin = np.concatenate(net), np.concatenate(pin)
    order = np.lexsort((pin, net))
    off = np.concatenate([[0], np.cumsum(np.bincount(net, minlength=m))]).astype(np.int64)
    nw = rng.integers(1, nw_max + 1, m).astype(np.int32) if nw_max > 1 else None
    return W.Hypergraph(n=hubs + light, m=m, off=off, pins=pin[order].astype(np.int32), k=k, eps=0.1, net_w=nw,
                        vtx_w=rng.integers(1, 4, hubs + light).astype(np.int32))


DEGREES = {"one": [5000], "edges": [257, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 6000],
           "many": [300 + 37 * i % 3000 for i in range(150)]}


@pytest.mark.parametrize("hubs", list(DEGREES))
@pytest.mark.parametrize("k,nw_max", [(7, 3), (16, 3), (32, 3), (64, 3), (65, 3), (128, 3), (32, 1), (64, 1), (128, 1)])
def test_hub_forms_match_oracle(k, nw_max, hubs):
    import paper_2504_12013_amd.jet as J
    hg = hypergraph(k, DEGREES[hubs], nw_max, k + nw_max)
    part = W.part_uniform(hg.n, k, 5)
    print(f"hubs {hubs}, k = {k}, net weights up to {nw_max}", flush=True)
    rng = np.random.default_rng(k)
    ctx = J.JetContext(hg)
    t, g, im = ctx.candidates(dev(part), 24576)
    ot, og, oim = O.candidates(hg, part, 24576)
    assert np.array_equal(im.cpu().numpy(), oim)
    assert np.array_equal(t.cpu().numpy(), ot)
    assert np.array_equal(g.cpu().numpy()[ot >= 0], og[ot >= 0])
    over = np.where(rng.random(hg.n) < 0.5, rng.integers(0, 2, hg.n), part).astype(np.int32)
    for dz in (100_000, 0):
        d = dev(over)
        sel, moved = ctx.rebalance_round(d, dz)
        new, osel, omoved = O.rebalance_round(hg, over, dz)
        assert moved == omoved and np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(d.cpu().numpy(), new)
    d = dev(over)
    rc, st, _ = ctx.refine(d, tau=(0.75, 0.0), limit=3)
    ref, orc, ost, _ = O.refine(hg, over, tau=(0.75, 0.0), limit=3)
    ctx.close()
    assert rc == orc and np.array_equal(d.cpu().numpy(), ref)
    assert st["iterations"] == ost["iterations"] and st["rebalance_rounds"] == ost["rebalance_rounds"]
