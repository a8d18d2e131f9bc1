"""Unit net weights have two candidate and two gain kernels, eight lanes or one lane per vertex.  The lane
degree option chooses between them at every size (the default keeps eight on few vertices), and the
one-lane kernels are compared with the oracle where they can go wrong: words of 32 blocks, degrees
around the five and nine planes, tails of a wave, hubs beside them, and several hypergraphs in one context.

With hubs in the input the device marks tell the kernels apart: hubs are a family of their own beside the
one-lane candidates and share the launch of the eight-lane ones."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FORCE_ONE, FORCE_EIGHT = 1 << 20, 0


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def J():
    import paper_2504_12013_amd.jet as jet
    return jet


def dev(a, dtype=torch.int32):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


def hypergraph(k, hubs, light, degree, seed):
    """`light` vertices in exactly `degree` nets each, `hubs` vertices in 600 each."""
    rng = np.random.default_rng(seed)
    n = hubs + light
    nets = [list(hubs + p) for _ in range(degree) for p in np.array_split(rng.permutation(light), (light + 2) // 3)]
    m = len(nets)
    for v in range(hubs):
        for e in rng.choice(m, 600, replace=False):
            nets[e].append(v)
    sizes = np.array([len(e) for e in nets])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pins = np.concatenate([np.sort(np.array(e)) for e in nets]).astype(np.int32)
    return W.Hypergraph(n=n, m=m, off=off, pins=pins, k=k, eps=0.1, vtx_w=rng.integers(1, 4, n).astype(np.int32))


def families(ctx, part):
    J().jet_prof_enable(ctx.h, True)
    ctx.candidates(dev(part), 24576)
    fam = J().jet_prof_read(ctx.h)
    J().jet_prof_enable(ctx.h, False)
    return fam


@pytest.mark.parametrize("lane_degree,one_lane", [(None, False), (24, False), (0, False), (5, False), (25, True),
                                                  (FORCE_ONE, True)])
def test_lane_degree_decides_on_few_vertices(lane_degree, one_lane):
    hg = hypergraph(8, 3, 1003, 20, 1)
    ctx = J().JetContext(hg)
    if lane_degree is not None:
        ctx.set_option(J().JET_OPT_CAND_LANE_DEGREE, lane_degree)
    fam = families(ctx, W.part_uniform(hg.n, 8, 2))
    ctx.close()
    print(lane_degree, sorted(fam), flush=True)
    assert ("candidates_hub" in fam) == one_lane


@pytest.mark.parametrize("lane_degree", [FORCE_ONE, FORCE_EIGHT])
@pytest.mark.parametrize("light,degree,hubs", [(63, 31, 0), (1003, 31, 3), (1003, 32, 3), (1025, 256, 0), (1025, 200, 2)])
@pytest.mark.parametrize("k", [8, 32, 33, 64, 65, 100, 128])
def test_lane_kernels_match_oracle(k, light, degree, hubs, lane_degree):
    hg = hypergraph(k, hubs, light, degree, 100 + k + degree)
    part = W.part_uniform(hg.n, k, 9)
    print(f"k = {k}, {light} light vertices of degree {degree}, {hubs} hubs, lane degree {lane_degree}", flush=True)
    rng = np.random.default_rng(k)
    lock = (rng.random(hg.n) < 0.2).astype(np.uint8)
    ctx = J().JetContext(hg)
    ctx.set_option(J().JET_OPT_CAND_LANE_DEGREE, lane_degree)
    if hubs:
        assert ("candidates_hub" in families(ctx, part)) == (lane_degree == FORCE_ONE)
    for lk in (None, lock):
        t, g, im = ctx.candidates(dev(part), 24576, None if lk is None else dev(lk, torch.uint8))
        ot, og, oim = O.candidates(hg, part, 24576, lk)
        assert np.array_equal(im.cpu().numpy(), oim)
        assert np.array_equal(t.cpu().numpy(), ot)
        assert np.array_equal(g.cpu().numpy()[ot >= 0], og[ot >= 0])
    over = np.where(rng.random(hg.n) < 0.6, 0, part).astype(np.int32)
    d = dev(over)
    sel, moved = ctx.rebalance_round(d, 100_000)
    new, osel, omoved = O.rebalance_round(hg, over, 100_000)
    assert moved == omoved and np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(d.cpu().numpy(), new)
    d = dev(part)
    rc, st, _ = ctx.refine(d, tau=(0.75, 0.0), limit=3)
    ref, orc, ost, _ = O.refine(hg, part, tau=(0.75, 0.0), limit=3)
    ctx.close()
    assert rc == orc and np.array_equal(d.cpu().numpy(), ref)
    assert st["iterations"] == ost["iterations"] and st["rebalance_rounds"] == ost["rebalance_rounds"]


@pytest.mark.parametrize("lane_degree", [FORCE_ONE, FORCE_EIGHT])
@pytest.mark.parametrize("k", [8, 64, 128])
def test_lane_kernels_in_a_batch(k, lane_degree):
    """Several hypergraphs of one k in one context (their tiles listed per phase), with hubs in some."""
    items = []
    for i, (light, degree, hubs) in enumerate([(255, 20, 0), (256, 31, 2), (700, 40, 0), (1003, 12, 1), (64, 31, 0)]):
        hg = hypergraph(k, hubs, light, degree, 300 + i)
        items.append((hg, W.part_uniform(hg.n, k, i)))
    batch = J().JetBatch([h for h, _ in items])
    batch.set_option(J().JET_OPT_CAND_LANE_DEGREE, lane_degree)
    parts = [dev(p) for _, p in items]
    print(f"batch, k = {k}, lane degree {lane_degree}", flush=True)
    _, stats, rcs = batch.refine(parts, tau=(0.75, 0.0), limit=4)
    for i, (hg, part) in enumerate(items):
        ref, orc, ost, _ = O.refine(hg, part, tau=(0.75, 0.0), limit=4)
        assert rcs[i] == orc and np.array_equal(parts[i].cpu().numpy(), ref), i
        assert stats[i]["iterations"] == ost["iterations"], i
