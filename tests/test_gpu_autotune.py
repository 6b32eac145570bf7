"""The batch autotuner against the call it tunes: it never leaves a caller with
a shape that takes clearly longer than not tuning."""
import statistics
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    import paper_2606_06255_amd as rf
    if not torch.cuda.is_available():
        raise RuntimeError("GPU tests need a GPU")
    return rf


@pytest.mark.parametrize("sizes", [[512 + 56 * i for i in range(64)], [8000, 12000] * 16], ids=["small", "middle"])
def test_not_slower_than_untuned(rf, sizes):
    """Uniform shapes take 1.4 times the untuned call's time and more on these
    batches.  A tenth is the autotuner's own margin; another fifth is left for
    noise."""
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    m = np.array([s // 4 for s in sizes], dtype=np.int32)
    x = torch.from_numpy(np.random.default_rng(1).random((off[-1], 3)).astype(np.float32)).cuda()
    chosen, ms, (idx, d2) = rf.autotune_batched(x, off, m, reps=5)
    kw = dict(groups=chosen["groups"], lookahead=chosen["lookahead"], tile=chosen["tile"])
    times = ([], [])
    for _ in range(8):
        for t, k in zip(times, ({}, kw)):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            gi, gd = rf.sample_batched(x, off, m, **k)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
            assert torch.equal(gi, idx) and torch.equal(gd, d2)
    untuned, tuned = (statistics.median(t[1:]) for t in times)
    assert tuned <= 1.1 * 1.2 * untuned, (chosen, untuned, tuned)


def test_fields_of_base_are_kept(rf):
    off, m = np.array([0, 700, 1500], dtype=np.int32), np.array([100, 200], dtype=np.int32)
    x = torch.from_numpy(np.random.default_rng(2).random((1500, 3)).astype(np.float32)).cuda()
    for base in (dict(groups=8), dict(lookahead=3), dict(groups=16, lookahead=2, tile=32)):
        chosen, _, _ = rf.autotune_batched(x, off, m, reps=1, **base)
        assert all(chosen[k] == v for k, v in base.items())
        assert chosen["groups"] and chosen["lookahead"]   # no call without a shape where part of one was asked for
