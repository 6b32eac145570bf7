"""The hidden layers' inputs are FP32 sums in the order of the inputs, four to
a matrix instruction: activations and accumulation are FP32, and the sign of a
sum decides whether its unit passes a gradient.

The weights are powers of two whose FP32 sums depend on the order and the
precision alone: an eighth added to 2^24 is lost (also four at once: half a
unit in the last place is 1), after 2^24 has been taken off again it is kept.
So a wider sum, or one split into parts, gives other outputs and other units
that are on.  Every value is exact in FP32 and bfloat16, so the comparison is."""
import numpy as np
import pytest
import torch

from oracle import mlp_ref as R

pytestmark = pytest.mark.gpu

BIG, SMALL = np.float32(2.0 ** 24), np.float32(0.125)


def _rows(K):
    """Weight rows of K inputs: BIG first, -BIG at `off`, SMALL elsewhere
    (but not in the two instructions that hold the large values)."""
    rows = []
    for off in (4, 8, 16, 20, 32, 36, K // 2, K // 2 + 4, K - 8, K - 1):
        w = np.full(K, SMALL, dtype=np.float32)
        w[:4] = 0
        w[off // 4 * 4:off // 4 * 4 + 4] = 0
        w[0], w[off] = BIG, -BIG
        rows.append(w)
    return np.stack(rows)


def _sum_in_order(w, x):
    acc = np.float32(0)
    for k in range(0, w.size, 4):
        acc = np.float32(np.float64(acc) + np.sum(w[k:k + 4].astype(np.float64) * x[k:k + 4].astype(np.float64)))
    return acc


@pytest.mark.parametrize("B", [1, 16, 35])
@pytest.mark.parametrize("layer", [1, 2])
def test_hidden_sums(layer, B):
    import paper_2606_06255_amd as rf
    dev = torch.device("cuda:0")
    P = {name: np.zeros(shape, dtype=np.float32) for name, shape in R.SHAPES}
    scale = np.float32(2.0) ** (np.arange(B) % 5 - 2).astype(np.float32)  # one power of two per input row
    if layer == 1:
        rows = _rows(516)
        P["W1"][:len(rows)] = rows
        P["W2"][:] = np.eye(64)
    else:
        rows = _rows(64)
        P["W1"][:, 0] = 1.0
        P["W2"][:len(rows)] = rows
    P["W3"][:64] = np.eye(64)
    X = np.ones((B, 516), dtype=np.float32) * scale[:, None]
    z = np.stack([[_sum_in_order(w, np.full(w.size, s)) for w in rows] for s in scale])
    wide = rows.astype(np.float64).sum(1)
    assert np.any((z[0] > 0) != (wide > 0)) and np.any(z[0] > 0)  # the order decides which units are on
    want = np.zeros((B, 72), dtype=np.float32)
    want[:, :len(rows)] = np.maximum(z, 0)
    net = rf.MLP(dev, rows=B)
    net.load(np.concatenate([P[name].ravel() for name, _ in R.SHAPES]))
    Xd = torch.from_numpy(X).to(dev)
    assert np.array_equal(net.forward(Xd).cpu().numpy(), want)
    # targets 1 below every output: dY = 2 / B, so a unit's bias gradient is 0 exactly when it is off
    g, _ = net.gradient(Xd, torch.from_numpy(want - 1).to(dev))
    at = sum(int(np.prod(s)) for n, s in R.SHAPES[:2 * layer - 1])
    db = g.cpu().numpy()[at:at + len(rows)]
    assert np.allclose(db, np.where(z[0] > 0, 2.0, 0.0), rtol=1e-6, atol=0)
