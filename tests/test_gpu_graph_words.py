"""The graph form of the one-lane candidate kernel (every net of two pins, blocks of the neighbours) in its
one, two and four words of blocks and with five and nine planes, small: candidates, rebalancing and refinements
against the oracle.  The device marks tell the form: it reads 8 bytes per incidence, the general one 8 and
the connectivity mask."""
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


def graph(n, degree, k, hub, seed):
    """A ring lattice of even degree with shuffled labels; hub: vertex 0 joined to 300 more."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    e = np.concatenate([np.stack([i, (i + d) % n], 1) for d in range(1, degree // 2 + 1)])
    e = rng.permutation(n)[e]
    if hub:
        e = np.concatenate([e, np.stack([np.zeros(300, int), 1 + rng.choice(n - 1, 300, replace=False)], 1)])
    e = np.unique(np.sort(e, axis=1), axis=0)
    off = np.arange(0, 2 * len(e) + 1, 2, dtype=np.int64)
    return W.Hypergraph(n=n, m=len(e), off=off, pins=e.astype(np.int32).ravel(), k=k, eps=0.05)


@pytest.mark.parametrize("n,degree,hub", [(2011, 6, False), (2048, 30, False), (2049, 32, False), (3001, 8, True)])
@pytest.mark.parametrize("k", [2, 32, 33, 64, 65, 96, 97, 128])
def test_graph_words_match_oracle(k, n, degree, hub):
    import paper_2504_12013_amd.jet as J
    hg = graph(n, degree, k, hub, k)
    part = W.part_uniform(n, k, 3)
    part[: n // 2] = np.sort(part[: n // 2])[(np.arange(n // 2))]
    print(f"n = {n}, degree {degree}, k = {k}, hub {hub}", flush=True)
    rng = np.random.default_rng(k)
    lock = (rng.random(n) < 0.2).astype(np.uint8)
    ctx = J.JetContext(hg)
    ctx.set_option(J.JET_OPT_CAND_LANE_DEGREE, 1 << 20)
    for tau in (0.0, 0.75):
        for lk in (None, lock):
            tq = O.quantize_tau(tau)
            J.jet_prof_enable(ctx.h, True)
            t, g, im = ctx.candidates(dev(part), tq, None if lk is None else dev(lk, torch.uint8))
            fam = J.jet_prof_read(ctx.h)
            J.jet_prof_enable(ctx.h, False)
            ot, og, oim = O.candidates(hg, part, tq, lk)
            assert np.array_equal(im.cpu().numpy(), oim)
            assert np.array_equal(t.cpu().numpy(), ot)
            assert np.array_equal(g.cpu().numpy()[ot >= 0], og[ot >= 0])
            if lk is None and not hub:
                assert fam["candidates"]["alg_bytes"] == 18.0 * n + 8.0 * hg.p
    d = dev(part)
    rc, st, _ = ctx.refine(d, tau=(0.75, 0.0), limit=3)
    ref, orc, ost, _ = O.refine(hg, part, tau=(0.75, 0.0), limit=3)
    ctx.close()
    assert rc == orc and np.array_equal(d.cpu().numpy(), ref)
    assert st["iterations"] == ost["iterations"]
