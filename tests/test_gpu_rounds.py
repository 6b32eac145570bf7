"""The multi-pick sampler at the edges of its merge, against the oracle, bit
for bit: lists on both sides of 64, 128, 192 and 256 candidates (where the
conflict and certification layouts change, and where a list is cut), one
workgroup (no exchange), slots wider than two units per thread, more than 64
tiles per wavefront, clouds of equal distances, exhausted clouds, and
coordinates whose squares overflow, vanish or lose bits to the origin."""
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


def check(rf, P, m, start, what, n_vox=0, tile=0, groups=0, lookahead=0, euclid=False):
    ri, rd = oracle.fps(P, m, start, threads=0, euclid=euclid)
    x = torch.from_numpy(np.ascontiguousarray(P)).cuda()
    gi, gd = rf.fps(x, m, start, n_vox=n_vox, tile=tile, groups=groups, lookahead=lookahead,
                    flags=rf.F_SQRT if euclid else 0)
    gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    bad = np.flatnonzero(gi != ri)
    assert bad.size == 0, "%s: first index mismatch at %d" % (what, bad[0])
    bad = np.flatnonzero(gd.view(np.uint32) != rd.view(np.uint32))
    assert bad.size == 0, "%s: first distance mismatch at %d" % (what, bad[0])


def clouds(kind, n):
    rng = np.random.default_rng(n + len(kind))
    if kind == "uniform":
        return rng.random((n, 3)).astype(np.float32)
    if kind == "lattice":      # every distance shared by many points
        s = int(round(n ** (1 / 3))) + 1
        g = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
        return np.ascontiguousarray(rng.permutation(g).astype(np.float32))
    if kind == "repeated":     # exhausted: every distance 0 before the last sample
        b = rng.random((max(1, n // 3), 3)).astype(np.float32)
        return np.ascontiguousarray(b[rng.integers(0, len(b), n)])
    if kind == "one point":
        return np.full((n, 3), 0.7, np.float32)
    scale, off = {"far": (1.0, 4e5), "tiny": (1e-21, 0.0), "huge": (4e18, 0.0), "wide": (1.0, 0.0)}[kind]
    P = rng.normal(size=(n, 3)) * scale + off
    if kind == "wide":
        P *= 10.0 ** rng.uniform(-12, 12, (n, 1))
    return P.astype(np.float32)


@pytest.mark.parametrize("kind", ["uniform", "lattice"])
@pytest.mark.parametrize("groups,lookahead", [(1, 0), (7, 8), (8, 8), (9, 8), (16, 8), (24, 8), (32, 8), (33, 8),
                                              (21, 3), (64, 4), (128, 3), (255, 4), (256, 8), (256, 3)])
def test_list_lengths(rf, kind, groups, lookahead):
    P = clouds(kind, 4500)
    check(rf, P, 1500, 17, "%s groups=%d lookahead=%d" % (kind, groups, lookahead), n_vox=8, groups=groups,
          lookahead=lookahead)


@pytest.mark.parametrize("kind", ["uniform", "lattice", "repeated", "one point", "far", "tiny", "huge", "wide"])
@pytest.mark.parametrize("groups", [0, 1, 5])
def test_cloud_kinds(rf, kind, groups):
    for n in (2, 63, 65, 1000, 2500):
        P = clouds(kind, n)
        for euclid in (False, True):
            check(rf, P, n, n // 2, "%s n=%d groups=%d euclid=%d" % (kind, n, groups, euclid), groups=groups,
                  euclid=euclid)


@pytest.mark.parametrize("tile", [1, 3])
def test_many_tiles_per_wavefront(rf, tile):
    P = clouds("uniform", 1500)
    check(rf, P, 700, 0, "tile=%d" % tile, n_vox=8, tile=tile, groups=1)
    P = clouds("lattice", 1500)
    check(rf, P, 700, 0, "lattice tile=%d" % tile, n_vox=8, tile=tile, groups=2, lookahead=8)
