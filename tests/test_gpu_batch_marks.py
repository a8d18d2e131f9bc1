"""Device marks of a batch: the families' times of its unions add up to time that passed on the device, so
their sum stays below the time of the call (unions that ran beside each other counted it several times)."""
import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_family_times_add_up():
    import paper_2504_12013_amd.jet as J
    items = [W.vlsi_like(seed=i, n=60_000, m=66_000) for i in range(8)]
    hgs, ks = [], (2, 4, 8, 11, 16, 32, 48, 64)
    for (hg, _), k in zip(items, ks):
        hgs.append(W.Hypergraph(n=hg.n, m=hg.m, off=hg.off, pins=hg.pins, k=k, eps=hg.eps))
    starts = [torch.from_numpy(W.part_uniform(h.n, h.k, 1)).to("cuda") for h in hgs]
    kw = dict(tau=(0.75,), limit=6)
    batch = J.JetBatch(hgs)
    plain = [p.clone() for p in starts]
    batch.refine(plain, **kw)
    batch.prof_enable(True)
    batch.refine([p.clone() for p in starts], **kw)  # graphs with the marks
    batch.prof_enable(True)
    parts = [p.clone() for p in starts]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    batch.refine(parts, **kw)
    torch.cuda.synchronize()
    wall = 1000.0 * (time.perf_counter() - t0)
    fam = batch.prof_read()
    batch.prof_enable(False)
    total = sum(f["total_ms"] for f in fam.values())
    print(f"families {total:.2f} ms of {wall:.2f} ms", flush=True)
    for a, b in zip(plain, parts):
        assert torch.equal(a, b)
    assert 0.1 * wall < total < wall
