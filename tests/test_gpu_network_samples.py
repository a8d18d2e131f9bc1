"""Every sample of a batch counts once in the temperature network's gradient and loss.  The targets are the
network's own predictions except at a few marked samples (first, last, around the 32 samples that a batch
sum holds in flight and the 2,048 waves of a forward launch), so the gradient is the marked samples' alone
and each of them is far above the tolerance in every group of parameters."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U = 2.0 ** -24
GROUPS = np.cumsum([0, 1024, 64, 4096, 64, 64, 1])


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def samples_grad(th, X, d3, absolute=False):
    """Per-sample gradients [S, 5313] of the rows of X for given dL/dz3; absolute: every product's size."""
    W1, _, W2, _, w3, _ = M.unpack(th)
    _, (X, z1, h1, z2, h2, _) = M.forward(th, X)
    if absolute:
        W2, w3, X, d3 = np.abs(W2), np.abs(w3), np.abs(X), np.abs(d3)
    d2 = np.outer(d3, w3) * (z2 > 0)
    d1 = (d2 @ W2) * (z1 > 0)
    S = len(X)
    return np.concatenate([(d1[:, :, None] * X[:, None, :]).reshape(S, -1), d1,
                           (d2[:, :, None] * h1[:, None, :]).reshape(S, -1), d2, d3[:, None] * h2, d3[:, None]], 1)


@pytest.mark.parametrize("B", [1, 31, 32, 33, 64, 65, 2047, 2048, 2049, 4097, 5000])
def test_every_sample_counts_once(B):
    import paper_2504_12013_amd.jet as J
    rng = np.random.default_rng(B)
    net = J.TauNet(seed=B)
    th32, mean, std = net.get()
    th = th32.astype(np.float64)
    marked = sorted({s for s in (0, 30, 31, 32, 2046, 2047, 2048, 2049, B - 2, B - 1) if 0 <= s < B})
    X = rng.normal(size=(B, 16)).astype(np.float32)
    for s in marked:  # no unit of a marked sample near its kink
        while min(np.abs(c).min() for c in M.forward(th, X[s:s + 1].astype(np.float64))[1][1:4:2]) < 1e-4:
            X[s] = rng.normal(size=16)
    raw = X * std + mean  # standardised to X again on the device
    y = net.forward(torch.from_numpy(raw)).cpu().numpy()
    t = y.copy()
    t[marked] += np.where(y[marked] < 0.5, np.float32(0.5), np.float32(-0.5))
    print(f"batch {B}, marked {marked}", flush=True)
    loss, g = net.grad(torch.from_numpy(raw), torch.from_numpy(t))
    Xs = M.standardise(raw.astype(np.float64), mean.astype(np.float64), std.astype(np.float64))
    y64 = M.forward(th, Xs)[0]
    err = y64[marked] - t[marked]
    d3 = 2 * err / B * y64[marked] * (1 - y64[marked])
    each = samples_grad(th, Xs[marked], d3)
    # rounding: some hundred operations on the way of a term, a thousand allowed; the unmarked samples'
    # predictions are within four ulps of their targets
    tol = 2048 * U * samples_grad(th, Xs[marked], d3, True).sum(0)
    rest = np.setdiff1d(np.arange(B), marked)
    for part in np.array_split(rest, max(1, len(rest) // 256)):
        if len(part):
            tol = tol + samples_grad(th, Xs[part], np.full(len(part), 2 * 4 * U / B * 0.25), True).sum(0)
    for a, b in zip(GROUPS[:-1], GROUPS[1:]):  # one marked sample more or less would show
        assert np.all(np.max(np.abs(each[:, a:b]) / (tol[a:b] + 1e-300), axis=1) > 20)
    assert np.all(np.abs(g.cpu().numpy() - each.sum(0)) <= tol)
    ref = np.sum(err ** 2) / B
    assert abs(loss - ref) <= 1e-4 * ref  # predictions are within 1e-5 of the exact ones, the differences are 0.5
    net.close()
