"""The network's gradient at the edges of its kernels: batches of one row to a
few row blocks (16 rows), row counts on both sides of a wavefront's group of
loads (256 rows), and misaligned inputs.

Tolerance: the hidden layers' inputs are summed in FP64, so the ReLU masks are
the reference's, and what is left is FP32 rounding: of dY, of sums of 72 and 64
products, and over the rows, each 2^-24 relative to its terms, 150 roundings or
1e-5 in the worst case and less than 1e-6 as they add up.  1e-4 leaves room for
the cancellation in sums over up to 600 rows."""
import numpy as np
import pytest
import torch

from oracle import mlp_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 15, 16, 17, 31, 33, 255, 256, 257, 600])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_gradient_edges(B, offset):
    import paper_2606_06255_amd as rf
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(100 * B + offset)
    theta = np.concatenate([(rng.uniform(-1, 1, int(np.prod(s))) * np.sqrt(6.0 / s[-1])).astype(np.float32)
                            for _, s in R.SHAPES])
    X = rng.normal(size=(B, R.SHAPES[0][1][1])).astype(np.float32)
    T = rng.normal(size=(B, R.SHAPES[-1][1][0])).astype(np.float32)
    W = rng.random(T.shape).astype(np.float32)
    net = rf.MLP(dev, rows=B)
    net.load(theta)

    def shifted(a):   # a contiguous view `offset` floats into its storage
        buf = torch.zeros(a.size + offset, device=dev)
        v = buf[offset:].view(a.shape)
        v.copy_(torch.from_numpy(a))
        return v

    for w in (W, None):
        g, loss = net.gradient(shifted(X), shifted(T), None if w is None else shifted(w))
        again, _ = net.gradient(shifted(X), shifted(T), None if w is None else shifted(w))
        assert torch.equal(g, again)
        gr, Lr = R.gradient(theta, X, T, np.ones_like(W) if w is None else w)
        assert abs(float(loss.item()) - Lr) <= 1e-5 * abs(Lr)
        g = g.cpu().numpy().astype(np.float64)
        o = 0
        for name, shape in R.SHAPES:
            size = int(np.prod(shape))
            a, b = g[o:o + size], gr[o:o + size]
            assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b), name
            o += size
