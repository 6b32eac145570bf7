"""How the teams of a batch take clouds and split (batch_teams.h, the kernel's
own definition), run on the CPU with a thread per workgroup: every cloud is
sampled once by a whole team of its level, and no slot is written again before
all members have read it, also when one workgroup is held back before it reads
the last exchange of a team."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("teams") / "libteams_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-pthread", "-Wall", "-o", out,
                    os.path.join(HERE, "native", "teams_shim.cpp")], check=True)
    return ctypes.CDLL(out)


def run(shim, per_xcd, clouds, slow=-1, at=0, wait=1):
    """clouds: one list of exchange counts per level."""
    levels = shim.shim_levels()
    clouds = clouds + [[]] * (levels - len(clouds))
    first = np.concatenate([[0], np.cumsum([len(c) for c in clouds])]).astype(np.uint32)
    ex = np.array([e for c in clouds for e in c], dtype=np.int32)
    members = np.zeros(len(ex), dtype=np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    bad = shim.shim_teams(per_xcd, len(ex), p(first), p(ex), slow, at, wait, p(members))
    want = np.array([(per_xcd >> lev) * (e > 0) for lev, c in enumerate(clouds) for e in c])
    return bad, members, want


@pytest.mark.parametrize("per_xcd", [2, 4, 8, 16])
def test_every_cloud_by_a_whole_team(shim, per_xcd):
    rng = np.random.default_rng(per_xcd)
    for it in range(20):
        clouds = [rng.integers(0, 6, rng.integers(0, 7)).tolist() for _ in range(int(np.log2(per_xcd)) + 1)]
        bad, members, want = run(shim, per_xcd, clouds)
        assert bad == 0 and np.array_equal(members, want), clouds


@pytest.mark.parametrize("slow", [0, 1, 2, 3])
@pytest.mark.parametrize("levels", [[[3], [4, 4]], [[3, 1], [], [5, 5, 5, 5]], [[2], [2, 2], [3, 3, 3, 3]]])
def test_split_waits_for_a_slow_workgroup(shim, levels, slow):
    """Held back before it reads the last exchange of the whole team."""
    X = 8
    clouds = levels + [[]] * (4 - len(levels))
    for s in (slow, slow + 4):
        bad, members, want = run(shim, X, clouds, slow=s, at=sum(levels[0]))
        assert bad == 0 and np.array_equal(members, want), (clouds, s)


def test_without_the_wait_a_read_is_lost(shim):
    """The model does see the fault: a team that splits at once loses reads."""
    lost = [run(shim, 8, [[3], [4, 4], [4, 4, 4, 4]], slow=s, at=3, wait=0)[0] for s in range(8)]
    assert any(lost)
