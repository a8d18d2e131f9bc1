"""Flow refinement where nets have up to thousands of pins (row-net shapes): the net nodes have long arc
lists and many neighbours push into them at once.  Partition and counts against the oracle."""
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


@pytest.mark.parametrize("workers", [1, 4])
@pytest.mark.parametrize("n,k", [(3000, 4), (10_000, 3)])
def test_flow_round_on_long_nets(n, k, workers):
    import paper_2504_12013_amd.jet as J
    hg = W.rownet_matrix(seed=n, n=n, k=k)
    part = W.part_uniform(n, k, 3)
    part, _, _, _ = O.refine(hg, part, tau=(0.75, 0.0), limit=4)
    print(f"rows {n}, longest net {int(np.diff(hg.off).max())}, k = {k}, {workers} workers", flush=True)
    out, ost = O.flow_refine(hg, part, max_rounds=1)
    ctx = J.JetContext(hg)
    ctx.set_option(J.JET_OPT_FLOW_WORKERS, workers)
    d = torch.from_numpy(part).to("cuda")
    st = ctx.flow_refine(d, max_rounds=1)
    ctx.close()
    for key in ("km1_in", "km1_out", "rounds", "matchings", "pairs", "accepted", "flow_calls", "moved"):
        assert st[key] == ost[key], key
    assert np.array_equal(d.cpu().numpy(), out)
