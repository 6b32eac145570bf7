"""The counters and clocks of an instrumented call on clouds where they can go
wrong: tiles that are never skipped (distances beyond the pruning bound's
range), rounds of a few picks, and tiles that do not fill a filter block."""
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


def _telemetry(rf, P, m, flags=None, **kw):
    idx = rf.build_index(torch.from_numpy(P).cuda(), tile=kw.pop("tile", 0))
    plain = rf.sample(idx, m, 0, **kw)
    out = rf.sample(idx, m, 0, flags=rf.F_TELEMETRY if flags is None else flags, **kw)
    assert torch.equal(plain[0], out[0]) and torch.equal(plain[1], out[1])
    return rf.read_telemetry(idx)


@pytest.mark.parametrize("groups", [0, 1, 5])
@pytest.mark.parametrize("scale,n", [(1e-21, 40), (1e-21, 700), (4e18, 40), (4e18, 700), (1.0, 33), (1.0, 700)])
def test_pruned_tests_are_counted_without_padding(rf, scale, n, groups):
    """Every tile is tested against every pick of a round but the last one's;
    a test that is not pruned visits the tile's points."""
    P = (np.random.default_rng(n).normal(size=(n, 3)) * scale).astype(np.float32)
    t = _telemetry(rf, P, n // 2, groups=groups)
    assert 0 <= t["tiles_pruned"] <= t["tile_tests"]
    assert t["tile_tests"] <= t["tiles"] * t["iters"]
    kept = t["tile_tests"] - t["tiles_pruned"]
    assert kept <= t["points_visited"] <= 64 * kept
    if scale != 1.0:
        assert t["tiles_pruned"] < t["tile_tests"]   # some tile lies beyond the bound's range
    # one point a tile: a kept test visits exactly one point
    t = _telemetry(rf, P, n // 2, groups=groups, tile=1)
    assert t["points_visited"] == t["tile_tests"] - t["tiles_pruned"]


@pytest.mark.parametrize("m,groups", [(6000, 0), (6000, 256), (1500, 64)])
def test_clocks_cover_the_phases(rf, m, groups):
    """The parts of a phase are clocked, and inside it.  The first workgroup
    waits for another one in some rounds at least, a tick (10 ns) a round on
    average (its own clocks make it a late one)."""
    P = np.random.default_rng(3).random((24000, 3)).astype(np.float32)
    t = _telemetry(rf, P, m, flags=rf.F_CLOCKS, groups=groups)
    rounds = t["exchanges"]
    assert rounds > 10
    assert rounds <= t["ticks_wait"] <= t["ticks_exchange_poll"] <= t["ticks_exchange"]
    assert 0 < t["ticks_lookahead_steps"] < t["ticks_lookahead"]
    parts = [t["ticks_merge_" + k] for k in ("list", "rank", "walk", "picks")]
    assert all(0 < v < t["ticks_merge"] for v in parts) and sum(parts) <= t["ticks_merge"]
    assert 0 < t["ticks_apply_update"] < t["ticks_apply"] == t["ticks_apply_loop"]
    assert t["apply_pairs"] >= t["apply_rekeys"] > 0
    assert t["merge_above"] >= t["merge_listed"] > t["merge_failures"] >= 0


def test_team_is_reported(rf):
    P = np.random.default_rng(5).random((9000, 3)).astype(np.float32)
    for flags in (rf.F_CLOCKS, rf.F_TELEMETRY):
        for groups, lookahead in ((7, 8), (4, 2), (64, 3)):
            t = _telemetry(rf, P, 900, flags=flags, groups=groups, lookahead=lookahead)
            assert t["team"] == groups + 65536 * lookahead
        t = _telemetry(rf, P, 900, flags=flags)
        assert 1 <= t["team"] % 65536 <= 256 and 2 <= t["team"] // 65536 <= 8
