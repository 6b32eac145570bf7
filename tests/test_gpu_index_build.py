"""The index build at the edges of its kernels: one workgroup against several
(4,096 points), radix tiles (2,048), blocks of sorted positions (256), the
scatter's row sums against the prefix sum (524,288 points), tile lengths from
1 to 64 and voxels longer than many tiles.  Voxel and tile counts are compared
with the voxel rule evaluated in FP64 here, and the tiles' points, order and
spheres through the sampler against the oracle."""
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


def counts(P, n_vox, tile):
    """Active voxels and tiles: V_id on cubes of edge (1 + 1e-4) max(E) / n_vox."""
    D = P.astype(np.float64)
    lo, E = D.min(0), (D.max(0) - D.min(0)).max()
    L = (1.0 + 1e-4) * E / n_vox if E > 0 else 1.0
    v = np.clip(np.floor((D - lo) / L), 0, n_vox - 1).astype(np.int64)
    _, c = np.unique(v[:, 2] * n_vox ** 2 + v[:, 1] * n_vox + v[:, 0], return_counts=True)
    return len(c), int(((c + tile - 1) // tile).sum())


def cloud(n, kind):
    rng = np.random.default_rng(n)
    if kind == "heaps":   # a few voxels of thousands of points among many of one
        P = np.where(rng.random((n, 1)) < 0.7, 0.001 * rng.random((n, 3)), rng.random((n, 3)))
    else:
        P = rng.random((n, 3))
    return P.astype(np.float32)


@pytest.mark.parametrize("kind", ["uniform", "heaps"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1023, 1025, 2047, 2049, 4095, 4096, 4097, 6145, 20000])
def test_counts_and_samples(rf, n, kind):
    P = cloud(n, kind)
    x = torch.from_numpy(P).cuda()
    m = min(n, 300)
    ri, rd = oracle.fps(P, m, n // 2, threads=0)
    for n_vox, tile in ((1, 64), (5, 1), (12, 7), (12, 64), (40, 33), (150, 64)):
        idx = rf.build_index(x, n_vox=n_vox, tile=tile)
        assert rf.read_status(idx) == 0
        info = rf.read_index_info(idx)
        assert (info["n_voxels"], info["n_tiles"]) == counts(P, n_vox, tile), (n_vox, tile)
        gi, gd = rf.sample(idx, m, n // 2)
        st = rf.read_status(idx)
        if st == 6:      # this many tiles exceed the on-chip budget
            gi, gd = rf.sample(idx, m, n // 2, flags=rf.F_UNFUSED)
            st = rf.read_status(idx)
        assert st == 0
        assert np.array_equal(gi.cpu().numpy(), ri), (n_vox, tile)
        assert np.array_equal(gd.cpu().numpy().view(np.uint32), rd.view(np.uint32)), (n_vox, tile)


@pytest.mark.parametrize("n", [524288, 524289, 1300000])
def test_large_counts(rf, n):
    P = cloud(n, "uniform")
    x = torch.from_numpy(P).cuda()
    ri, _ = oracle.fps(P, 40, 3, threads=0)
    for n_vox, tile in ((30, 64), (60, 5)):
        idx = rf.build_index(x, n_vox=n_vox, tile=tile)
        info = rf.read_index_info(idx)
        assert (info["n_voxels"], info["n_tiles"]) == counts(P, n_vox, tile)
        gi, _ = rf.sample(idx, 40, 3, flags=rf.F_UNFUSED)
        assert rf.read_status(idx) == 0
        assert np.array_equal(gi.cpu().numpy(), ri)


@pytest.mark.parametrize("n", [3, 4096, 4097])
def test_non_finite(rf, n):
    for bad in (np.nan, np.inf, -np.inf):
        P = cloud(n, "uniform")
        P[n - 1, 1] = bad
        idx = rf.build_index(torch.from_numpy(P).cuda())
        assert rf.read_status(idx) == 2
        gi, _ = rf.sample(idx, 2, 0)
        assert rf.read_status(idx) == 2 and (gi.cpu().numpy() == -1).all()
