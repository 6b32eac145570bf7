"""Which calls one workgroup takes (round_layout.h): on both sides of the rule's
edges the outputs are the oracle's, and sampling a whole cloud of the largest
such size takes no longer than the team that it would otherwise get."""
import statistics
import time

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


@pytest.mark.parametrize("euclid", [False, True])
@pytest.mark.parametrize("n,m", [(3072, 3072), (3073, 1536), (3073, 1537), (3073, 3073), (3584, 1792), (3584, 1793),
                                 (3584, 3584), (3585, 10)])
def test_edges(rf, n, m, euclid):
    P = np.random.default_rng(n + m).random((n, 3)).astype(np.float32)
    ri, rd = oracle.fps(P, m, 7, threads=0, euclid=euclid)
    gi, gd = rf.fps(torch.from_numpy(P).cuda(), m, 7, flags=rf.F_SQRT if euclid else 0)
    assert np.array_equal(gi.cpu().numpy(), ri)
    assert np.array_equal(gd.cpu().numpy().view(np.uint32), rd.view(np.uint32))


def test_whole_cloud_is_not_slower_than_a_team(rf):
    """One workgroup took 1.4 times a team's time here; a fifth leaves room
    for the noise of medians over 25 calls, timed in turn."""
    n = 3584
    idx = rf.build_index(torch.from_numpy(np.random.default_rng(0).random((n, 3)).astype(np.float32)).cuda())
    times = {0: [], 3: []}   # the default, and a team with the lookahead it would use
    for _ in range(28):
        for lookahead, t in times.items():
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            rf.sample(idx, n, 0, lookahead=lookahead)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
    default, team = (statistics.median(t[3:]) for t in times.values())
    assert default <= 1.2 * team, (default, team)
