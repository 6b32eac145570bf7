"""The multi-pick sampler's distance filter and capacity rule, on the CPU.

The filter (prune_bound.h) may keep any pair but must never drop one whose
FP32 formula distance is below the limit: checked at limits one ulp above the
formula distance, over the exponent range, with clouds near and far from the
origin the filter shifts to, and for several ways of rounding its product.
The capacity rule (round_layout.h) must never grant a share that the
sampler's own layout cannot hold."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("round") / "libround_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fno-fast-math", "-frounding-math", "-fPIC",
                    "-shared", "-Wall", "-o", out, os.path.join(HERE, "native", "round_shim.cpp")], check=True)
    return ctypes.CDLL(out)


def run(shim, s, p, o, limit, way):
    n = len(s)
    keep, d = np.zeros(n, np.uint8), np.zeros(n, np.float32)
    c = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    shim.shim_filter(n, c(s), c(p), c(o), c(limit), way, c(keep), c(d))
    return keep.astype(bool), d


@pytest.mark.parametrize("way", [0, 1, 2, 3])
@pytest.mark.parametrize("scale", [1e-30, 1e-18, 1e-6, 1.0, 1e6, 1e17, 1e19, 3e37])
def test_filter_keeps_every_near_pair(shim, scale, way):
    rng = np.random.default_rng(int(way * 100 + np.log10(scale) + 50))
    n = 20000
    for off in (0.0, 1.0, 1e3, 1e6):
        with np.errstate(over="ignore", invalid="ignore"):
            o = (rng.normal(size=3) * off * scale).astype(np.float32)
            p = (o + rng.normal(size=(n, 3)) * scale * 10.0 ** rng.uniform(-6, 0, (n, 1))).astype(np.float32)
            s = (p + rng.normal(size=(n, 3)) * scale * 10.0 ** rng.uniform(-6, 0, (n, 1))).astype(np.float32)
        ok = np.isfinite(p).all(1) & np.isfinite(s).all(1) & np.isfinite(o).all()
        p, s = np.ascontiguousarray(p[ok]), np.ascontiguousarray(s[ok])
        if not len(p):
            continue
        _, d = run(shim, s, p, o, np.zeros(len(p), np.float32), way)
        limit = np.nextafter(d, np.float32(np.inf)).astype(np.float32)
        keep, _ = run(shim, s, p, o, limit, way)
        assert keep.all(), "dropped %d pairs below the limit" % (~keep).sum()
        # a limit that is not a number never drops a pair
        keep, _ = run(shim, s, p, o, np.full(len(p), np.nan, np.float32), way)
        assert keep.all()


def test_filter_drops_far_pairs(shim):
    rng = np.random.default_rng(3)
    o = np.zeros(3, np.float32)
    p = rng.random((10000, 3)).astype(np.float32)
    s = rng.random((10000, 3)).astype(np.float32)
    _, d = run(shim, s, p, o, np.zeros(len(p), np.float32), 0)
    keep, _ = run(shim, s, p, o, (0.9 * d - np.float32(1e-3)).clip(0).astype(np.float32), 0)
    assert keep.mean() < 0.01


def test_granted_shares_fit_the_layout(shim):
    lds = 160 * 1024     # what a gfx950 workgroup may use
    budget, dyn = shim.shim_budget(lds), shim.shim_dynamic(lds)
    for G in (1, 2, 3, 16, 32, 64, 100, 128, 255, 256):
        for R in (2, 3, 4, 8):
            for tiles in list(range(0, 140)) + list(range(140, 4000, 37)):
                # the largest share of so many tiles the rule grants
                lo, hi = -1, 64 * tiles
                while lo < hi:
                    mid = (lo + hi + 1) // 2
                    if shim.shim_granted(tiles, mid, G, R, budget):
                        lo = mid
                    else:
                        hi = mid - 1
                if lo >= 0:
                    need = shim.shim_need(tiles, lo)
                    assert need <= dyn, (G, R, tiles, lo, need, dyn)
