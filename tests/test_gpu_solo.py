"""Small clouds by one workgroup, against the oracle, bit for bit: point counts
on both sides of every number of points a thread holds and of the limits that
hand a cloud to a team, sample counts around the ring of 64 selections, equal
distances, exhausted clouds, and coordinates whose squares overflow or vanish."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    import paper_2606_06255_amd as rf
    if not torch.cuda.is_available():
        raise RuntimeError("GPU tests need a GPU")
    return rf


def cloud(n, kind):
    rng = np.random.default_rng(n)
    if kind == "lattice":
        return rng.integers(0, 7, (n, 3)).astype(np.float32)
    if kind == "huge":
        return (rng.normal(size=(n, 3)) * 5e18).astype(np.float32)
    if kind == "tiny":
        return (rng.normal(size=(n, 3)) * 1e-22).astype(np.float32)
    return rng.random((n, 3)).astype(np.float32)


def same(got, ref, what):
    gi, gd = got[0].cpu().numpy(), got[1].cpu().numpy()
    bad = np.flatnonzero(gi != ref[0])
    assert bad.size == 0, "%s: first index mismatch at %d" % (what, bad[0])
    bad = np.flatnonzero(gd.view(np.uint32) != ref[1].view(np.uint32))
    assert bad.size == 0, "%s: first distance mismatch at %d" % (what, bad[0])


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 512, 513, 1024, 1025, 2048, 2049, 3072, 3073, 3584, 3585])
@pytest.mark.parametrize("kind", ["uniform", "lattice", "huge", "tiny"])
def test_point_counts(rf, n, kind):
    P = cloud(n, kind)
    x = torch.from_numpy(P).cuda()
    for euclid in (False, True):
        m = n if n <= 600 or kind == "lattice" else 400
        ref = oracle.fps(P, m, n // 2, threads=0, euclid=euclid)
        same(rf.fps(x, m, n // 2, flags=rf.F_SQRT if euclid else 0), ref, "n=%d %s euclid=%d" % (n, kind, euclid))


@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 66, 127, 128, 129, 192, 193, 600])
def test_sample_counts(rf, m):
    P = cloud(600, "uniform")
    x = torch.from_numpy(P).cuda()
    idx = rf.build_index(x)
    oi = torch.full((m + 8,), 77, dtype=torch.int32, device="cuda")
    od = torch.full((m + 8,), 77.0, device="cuda")
    ref = oracle.fps(P, m, 5, threads=0)
    for _ in range(2):
        rf.sample(idx, m, 5, out_idx=oi, out_d2=od)
        same((oi[:m], od[:m]), ref, "m=%d" % m)
        assert (oi[m:] == 77).all() and (od[m:] == 77.0).all()
        assert rf.read_status(idx) == 0


def test_batch_limits(rf):
    sizes = [4095, 4096, 4097, 8191, 8192, 8193, 1, 2, 513, 3000] * 30   # more than the device holds at once
    rng = np.random.default_rng(0)
    base = {n: rng.random((n, 3)).astype(np.float32) for n in set(sizes)}
    ms = [max(1, n // 16) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    x = torch.from_numpy(np.concatenate([base[n] for n in sizes])).cuda()
    refs = {n: oracle.fps(base[n], max(1, n // 16), n // 3, threads=0) for n in base}
    for starts in ([n // 3 for n in sizes],):
        gi, gd = rf.sample_batched(x, off, ms, starts, n_vox=8)
        o = 0
        for n, m in zip(sizes, ms):
            same((gi[o:o + m], gd[o:o + m]), refs[n], "batch cloud of %d" % n)
            o += m


def test_replayed_graph(rf):
    P = [cloud(n, "uniform") for n in (700, 1500)]
    xs = [torch.from_numpy(p).cuda() for p in P]
    x = xs[0].clone()
    idx = rf.build_index(x)
    oi = torch.empty(200, dtype=torch.int32, device="cuda")
    od = torch.empty(200, device="cuda")
    rf.sample(idx, 200, 1, out_idx=oi, out_d2=od)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rf.build_index(x, reuse=idx)
        rf.sample(idx, 200, 1, out_idx=oi, out_d2=od)
    for r in range(4):
        Q = cloud(700, "uniform") + np.float32(r)
        Q = Q[np.random.default_rng(r).permutation(700)]
        x.copy_(torch.from_numpy(Q))
        g.replay()
        same((oi, od), oracle.fps(Q, 200, 1, threads=0), "replay %d" % r)
        rf.fps(xs[1], 300, 0)      # the program's own work between the replays
