"""Batches whose clouds get teams of different sizes, against the oracle, bit
for bit: every size from a whole XCD to one workgroup in one call, clouds that
need no exchange, more clouds than workgroups, and the same workspace used
again by another batch and another team size."""
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


def make(rng, sizes):
    return [(rng.random((n, 3)) * rng.uniform(0.5, 20) + rng.normal(size=3) * 5).astype(np.float32) for n in sizes]


def check(rf, clouds, ms, starts, ws=None, euclid=False, **kw):
    off = np.concatenate([[0], np.cumsum([len(c) for c in clouds])]).astype(np.int32)
    x = torch.from_numpy(np.concatenate(clouds)).cuda()
    idx, d2 = rf.sample_batched(x, off, ms, starts, ws=ws, flags=rf.F_SQRT if euclid else 0, **kw)
    idx, d2 = idx.cpu().numpy(), d2.cpu().numpy()
    o = 0
    for c, (P, m, s) in enumerate(zip(clouds, ms, starts)):
        ri, rd = oracle.fps(P, m, s, threads=0, euclid=euclid)
        what = "cloud %d of %d: N=%d m=%d" % (c, len(clouds), len(P), m)
        assert np.array_equal(idx[o:o + m], ri), what
        assert np.array_equal(d2[o:o + m].view(np.uint32), rd.view(np.uint32)), what
        o += m


# sizes whose smallest teams are 32, 16, 8, 4, 2 and 1 workgroups, several of
# each, so that the device cannot hold all at once
EVERY = [100000, 90000] * 5 + [50000, 60000] * 4 + [25000] * 6 + [13000] * 5 + [7000] * 5 + [3000, 900, 2, 1] * 3


@pytest.mark.parametrize("lookahead", [0, 2, 8])
def test_every_level(rf, lookahead):
    rng = np.random.default_rng(11 + lookahead)
    order = rng.permutation(len(EVERY))
    sizes = [EVERY[i] for i in order]
    clouds = make(rng, sizes)
    ms = [max(1, min(n // 8, 700)) if i % 5 else 1 for i, n in enumerate(sizes)]
    starts = [int(rng.integers(0, n)) for n in sizes]
    check(rf, clouds, ms, starts, lookahead=lookahead, n_vox=12)


@pytest.mark.parametrize("count", [1, 7, 8, 9, 255, 256, 257, 700])
def test_counts_around_the_device(rf, count):
    rng = np.random.default_rng(count)
    sizes = [int(v) for v in rng.integers(20, 300, count)]
    if count < 10:
        sizes = [s * 37 for s in sizes]
    clouds = make(rng, sizes)
    check(rf, clouds, [max(1, n // 4) for n in sizes], [n // 3 for n in sizes], euclid=count % 2 == 0, n_vox=6)


def test_workspace_shared_by_batches(rf):
    rng = np.random.default_rng(5)
    ws = rf.BatchWorkspace(60000, 64, torch.device("cuda:0"), n_vox=8)
    for sizes, groups in (([30000, 9000, 500, 12000], 0), ([700] * 40, 0), ([9000] * 6, 16), ([5000] * 10, 0),
                          ([20000, 200, 3000], 32), ([700] * 64, 2)):
        clouds = make(rng, sizes)
        check(rf, clouds, [n // 5 for n in sizes], [0] * len(sizes), ws=ws, groups=groups, n_vox=8)
