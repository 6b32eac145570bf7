"""The work that users of this framework have it do, as timed cases.

Every case goes through the package's public entry points on the GPU:
sampling one cloud (build_index + sample, or fps in one call), sampling a
cloud in stages, sampling a batch of uneven clouds (eagerly or from a
captured graph), sampling with the trained parameter network's grid, and one
gradient of that network's training.  Sizes are those of bench.py and the
tests (4,096 to 1,048,576 points, batches of 32) and of ordinary object-sized
clouds below them.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2606_06255_amd as rf
from paper_2606_06255_amd.param_model import ParamModel, fps_auto

DEV = "cuda:0"
# the parameter network: 516 features, two hidden layers of 64, 72 outputs (36 relative log times, 36 rates)
INPUTS, HIDDEN, OUTPUTS = 516, 64, 72
PARAMS = HIDDEN * (INPUTS + 1 + HIDDEN + 1) + OUTPUTS * (HIDDEN + 1)


def listed():
    return [
        # An object-sized cloud, one call: the smallest work, where launches
        # and the host path count.
        {"name": "object_1k", "op": "single", "cloud": "object", "n": 1024, "m": 256, "start": 0, "euclid": False,
         "reuse": False},
        # The unit cube of the smoke test and the bench.
        {"name": "cube_4k", "op": "single", "cloud": "cube", "n": 4096, "m": 1024, "start": 0, "euclid": False,
         "reuse": False},
        # An indoor room, as the scene-segmentation backbones sample it, with
        # workspace and outputs kept between clouds.
        {"name": "room_80k", "op": "single", "cloud": "room", "n": 80000, "m": 20000, "start": 0, "euclid": False,
         "reuse": True},
        # One ragged spinning-sensor sweep over rounded Euclidean distances
        # (the paper's update rule), from a start inside the cloud.
        {"name": "sweep_euclid_114k", "op": "single", "cloud": "sweep", "n": 114623, "m": 28655, "start": 57311,
         "euclid": True, "reuse": True},
        # The headline workload: 1,048,576 points of a dense sweep.
        {"name": "dense_1m", "op": "single", "cloud": "sweep", "n": 1048576, "m": 65536, "start": 0, "euclid": False,
         "reuse": True},
        # A sweep down-sampled in three stages, as a point backbone runs it:
        # small and medium clouds whose order is that of the picks.
        {"name": "sweep_stages", "op": "stages", "cloud": "sweep", "n": 114624, "stages": 3},
        # A training batch of small uneven clouds, eager.
        {"name": "batch_small_64", "op": "batch", "clouds": 64, "lo": 512, "hi": 4096, "sizes": 0,
         "cloud": "object", "graph": False},
        # The bench's batch: 32 uneven rooms and sweeps, replayed from a
        # captured graph as a serving loop does.
        {"name": "batch_32_graph", "op": "batch", "clouds": 32, "lo": 8000, "hi": 120000, "sizes": 0,
         "cloud": "mixed", "graph": True},
        # A large room with the grid picked by the trained network.
        {"name": "auto_room_250k", "op": "auto", "cloud": "room", "n": 250007, "m": 31250},
        # One full-batch gradient of the parameter network's training.
        {"name": "network_gradient_2000", "op": "gradient", "rows": 2000},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    op = rng.choices(["single", "stages", "batch", "auto", "gradient"], [10, 2, 5, 2, 2])[0]
    if op == "single":
        cloud = rng.choice(["object", "cube", "room", "sweep"])
        hi = {"object": 16384, "cube": 65536, "room": 200000, "sweep": 1048576}[cloud]
        n = _log_int(rng, 1000, hi)
        # a quarter kept up to 200,000 points (28,655 of a sweep of 114,623),
        # a sixteenth of larger sweeps (65,536 of 1,048,576)
        m = n // 4 if n <= 200000 else n // 16
        return {"op": op, "cloud": cloud, "n": n, "m": rng.randint(m // 2, m), "start": rng.randrange(n),
                "euclid": rng.random() < 0.25, "reuse": rng.random() < 0.5}
    if op == "stages":
        return {"op": op, "cloud": rng.choice(["room", "sweep"]), "n": _log_int(rng, 8000, 114624),
                "stages": rng.randint(2, 4)}
    if op == "batch":
        small = rng.random() < 0.5
        lo = rng.randint(200, 1000) if small else rng.randint(4000, 8000)
        return {"op": op, "clouds": _log_int(rng, 8, 128) if small else rng.randint(4, 32), "lo": lo,
                "hi": rng.randint(2 * lo, 6000) if small else rng.randint(2 * lo, 100000), "sizes": rng.randrange(1 << 20),
                "cloud": "object" if small else "mixed", "graph": rng.random() < 0.3}
    if op == "auto":
        n = _log_int(rng, 8000, 200000)
        return {"op": op, "cloud": rng.choice(["room", "sweep"]), "n": n, "m": n // 8}
    return {"op": op, "rows": _log_int(rng, 32, 2000)}


# ---------------------------------------------------------------------------
# Inputs, made on the GPU from the seed
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _surfaces(g, n, size, boxes, spheres, noise):
    """n points on the walls, floor and ceiling of a box-shaped room, on the
    upright faces and tops of boxes in it and on spheres, in random order
    with Gaussian jitter; a point's surface is drawn by area."""
    size = torch.tensor(size, device=DEV, dtype=torch.float64)
    zero = torch.zeros(3, device=DEV, dtype=torch.float64)
    org, uu, vv = [], [], []
    ex, ey, ez = torch.diag(size)

    def rect(o, u, v):
        org.append(o)
        uu.append(u)
        vv.append(v)

    for o, u, v in ((zero, ex, ey), (ez, ex, ey), (zero, ey, ez), (ex, ey, ez), (zero, ex, ez), (ey, ex, ez)):
        rect(o, u, v)
    short = float(size.min())
    for _ in range(boxes):
        s = (0.1 + 0.5 * _rand(g, 3)) * short
        o = _rand(g, 3) * (size - s).clamp_min(0.0)
        o = torch.stack([o[0], o[1], zero[2]])
        sx, sy, sz = torch.diag(s)
        for q in ((o + sz, sx, sy), (o, sy, sz), (o + sx, sy, sz), (o, sx, sz), (o + sy, sx, sz)):
            rect(*q)
    org, uu, vv = torch.stack(org), torch.stack(uu), torch.stack(vv)
    area = torch.linalg.norm(torch.linalg.cross(uu, vv), dim=1)
    if spheres:
        rad = (0.07 + 0.2 * _rand(g, spheres)) * short
        cen = rad[:, None] + _rand(g, spheres, 3) * (size[None, :] - 2 * rad[:, None])
        area = torch.cat([area, 4.0 * math.pi * rad * rad])
    cum = torch.cumsum(area, 0)
    which = torch.searchsorted(cum, _rand(g, n) * cum[-1]).clamp_max(area.numel() - 1)
    flat = which.clamp_max(org.shape[0] - 1)
    ab = _rand(g, n, 2)
    p = org[flat] + ab[:, :1] * uu[flat] + ab[:, 1:] * vv[flat]
    if spheres:
        ball = (which - org.shape[0]).clamp_min(0)
        d = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
        d = d / torch.linalg.norm(d, dim=1, keepdim=True)
        p = torch.where((which >= org.shape[0])[:, None], cen[ball] + rad[ball][:, None] * d, p)
    p = p + noise * torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    return p.float().contiguous()


def _sweep(g, n):
    """n returns of a spinning sensor at the origin in azimuth-major order:
    64 beams (128 above 300,000 points) against the ground, 40 boxes and a
    far wall, with range noise, thinned to n."""
    beams = 64 if n < 300000 else 128
    steps = -(-n // beams) if n % beams == 0 else int(math.ceil(n / (beams * 0.995)))
    el = torch.deg2rad(torch.linspace(-25.0, 3.0, beams, device=DEV, dtype=torch.float64))
    az = torch.arange(steps, device=DEV, dtype=torch.float64) * (2.0 * math.pi / steps)
    dx = (torch.cos(az)[:, None] * torch.cos(el)[None, :]).reshape(-1)
    dy = (torch.sin(az)[:, None] * torch.cos(el)[None, :]).reshape(-1)
    dz = torch.sin(el).repeat(steps)
    ground = -1.7
    t = 80.0 / torch.sqrt(dx * dx + dy * dy)
    t = torch.minimum(t, torch.where(dz < 0, ground / dz, torch.full_like(t, math.inf)))
    side = 1.0 + 4.0 * _rand(g, 40, 3)
    rr, th = 5.0 + 75.0 * _rand(g, 40), 2.0 * math.pi * _rand(g, 40)
    inv = [1.0 / dx, 1.0 / dy, 1.0 / dz]
    for b in range(40):
        mid = torch.stack([rr[b] * torch.cos(th[b]), rr[b] * torch.sin(th[b]), ground + side[b, 2] / 2])
        tn, tf = torch.full_like(t, -math.inf), torch.full_like(t, math.inf)
        for a in range(3):
            t1 = (mid[a] - side[b, a] / 2) * inv[a]
            t2 = (mid[a] + side[b, a] / 2) * inv[a]
            tn = torch.maximum(tn, torch.minimum(t1, t2))
            tf = torch.minimum(tf, torch.maximum(t1, t2))
        t = torch.where((tn <= tf) & (tn > 0) & (tn < t), tn, t)
    t = t + 0.02 * torch.randn(t.numel(), generator=g, device=DEV, dtype=torch.float64)
    p = torch.stack([t * dx, t * dy, t * dz], dim=1)
    if p.shape[0] > n:
        keep = torch.randperm(p.shape[0], generator=g, device=DEV)[:n].sort().values
        p = p[keep]
    return p.float().contiguous()


def _cloud(kind, g, n):
    if kind == "cube":
        return torch.rand(n, 3, generator=g, device=DEV)
    if kind == "room":
        return _surfaces(g, n, (10.0, 8.0, 3.0), 20, 10, 0.005)
    if kind == "object":
        return _surfaces(g, n, (1.0, 0.6, 0.8), 2, 2, 0.002)
    return _sweep(g, n)


def _batch_sizes(case):
    r = random.Random(case["sizes"])
    return [_log_int(r, case["lo"], case["hi"]) for _ in range(case["clouds"])]


def _batch_inputs(case, seed):
    g = _gen(seed)
    sizes = _batch_sizes(case)
    kinds = [case["cloud"] if case["cloud"] != "mixed" else ("room", "sweep")[i % 2] for i in range(case["clouds"])]
    x = torch.cat([_cloud(k, g, s) for k, s in zip(kinds, sizes)]).contiguous()
    offsets = [0]
    for s in sizes:
        offsets.append(offsets[-1] + s)
    return x, offsets, [s // 4 for s in sizes]


def _gradient_inputs(case, seed):
    """Rows as the parameter sweep gives them: log size, extents, the mostly
    empty log-occupancy histogram; targets are zero-mean log times and rates
    in [0, 1]; the second head counts a quarter."""
    g, rows = _gen(seed), case["rows"]
    x = torch.zeros(rows, INPUTS, device=DEV)
    x[:, 0] = torch.rand(rows, generator=g, device=DEV) * 2.4 - 1.0
    x[:, 1:4] = 0.6 + 2.0 * torch.rand(rows, 3, generator=g, device=DEV)
    occ = torch.rand(rows, 512, generator=g, device=DEV)
    x[:, 4:] = torch.where(occ > 0.75, torch.log1p(2.0 * torch.rand(rows, 512, generator=g, device=DEV)), 0.0 * occ)
    t = torch.empty(rows, OUTPUTS, device=DEV)
    half = OUTPUTS // 2
    lm = 0.4 * torch.randn(rows, half, generator=g, device=DEV)
    t[:, :half] = lm - lm.mean(1, keepdim=True)
    t[:, half:] = torch.rand(rows, half, generator=g, device=DEV)
    w = torch.ones(rows, OUTPUTS, device=DEV)
    w[:, half:] = 0.25
    params = torch.zeros(PARAMS, device=DEV)  # weight matrices uniform as at the start of training, biases 0
    at = 0
    for outs, ins in ((HIDDEN, INPUTS), (HIDDEN, HIDDEN), (OUTPUTS, HIDDEN)):
        u = 2.0 * torch.rand(outs * ins, generator=g, device=DEV) - 1.0
        params[at : at + outs * ins] = u * math.sqrt(6.0 / ins)
        at += outs * ins + outs
    return x, t, w, params


# ---------------------------------------------------------------------------
# The calls
# ---------------------------------------------------------------------------
def _outputs(m):
    return torch.empty(m, dtype=torch.int32, device=DEV), torch.empty(m, dtype=torch.float32, device=DEV)


def _stage_sizes(case):
    return [case["n"] // 4 ** (k + 1) for k in range(case["stages"])]


def prepare(case, seed):
    op = case["op"]
    if op == "single":
        st = {"case": case, "x": _cloud(case["cloud"], _gen(seed), case["n"])}
        if case["reuse"]:
            # a program that samples many clouds keeps workspace and outputs
            st["index"] = rf.build_index(st["x"])
            st["out"] = _outputs(case["m"])
        return st
    if op == "stages":
        st = {"case": case, "x": _cloud(case["cloud"], _gen(seed), case["n"])}
        st["index"] = rf.build_index(st["x"])
        return st
    if op == "batch":
        x, offsets, m = _batch_inputs(case, seed)
        st = {"case": case, "x": x, "m_total": sum(m)}
        st["offsets"] = torch.tensor(offsets, dtype=torch.int32, device=DEV)
        st["m"] = torch.tensor(m, dtype=torch.int32, device=DEV)
        st["ws"] = rf.BatchWorkspace(x.shape[0], len(m), x.device)
        st["out"] = _outputs(st["m_total"])
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _batched(st)
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            st["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(st["graph"]):
                _batched(st)
        return st
    if op == "auto":
        return {"case": case, "x": _cloud(case["cloud"], _gen(seed), case["n"]), "model": ParamModel(torch.device(DEV))}
    x, t, w, params = _gradient_inputs(case, seed)
    net = rf.MLP(torch.device(DEV), rows=case["rows"])
    net.load(params.cpu().numpy())
    return {"case": case, "x": x, "t": t, "w": w, "net": net}


def _batched(st):
    rf.sample_batched(st["x"], st["offsets"], st["m"], m_total=st["m_total"], ws=st["ws"], out_idx=st["out"][0],
                      out_d2=st["out"][1], check=False)


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "single":
        flags = rf.F_SQRT if case["euclid"] else 0
        if not case["reuse"]:
            idx, d2 = rf.fps(st["x"], case["m"], case["start"], flags=flags)
        else:
            st["index"] = rf.build_index(st["x"], reuse=st["index"])
            idx, d2 = rf.sample(st["index"], case["m"], case["start"], flags=flags, out_idx=st["out"][0],
                                out_d2=st["out"][1])
        return {"idx": idx, "d2": d2}
    if op == "stages":
        x, out = st["x"], []
        for m in _stage_sizes(case):
            st["index"] = rf.build_index(x, reuse=st["index"])
            idx, d2 = rf.sample(st["index"], m)
            x = rf.gather_xyz(x, idx)
            out.append({"idx": idx, "d2": d2})
        return {"stages": out, "xyz": x}
    if op == "batch":
        if case["graph"]:
            st["graph"].replay()
        else:
            _batched(st)
        return {"idx": st["out"][0], "d2": st["out"][1]}
    if op == "auto":
        idx, d2, _ = fps_auto(st["model"], st["x"], case["m"])
        return {"idx": idx, "d2": d2}
    g, loss = st["net"].gradient(st["x"], st["t"], st["w"])
    return {"grad": g, "loss": loss}


def work(case):
    """Points read once, indices and distances written once (and, between
    stages, the picks' coordinates); nine operations give a distance, and
    every point and every pick needs at least one."""
    op = case["op"]
    if op == "gradient":
        r, p = case["rows"], PARAMS
        return {"bytes": 4 * r * (INPUTS + 2 * OUTPUTS) + 8 * p, "flops": 4 * r * p + 2 * r * HIDDEN * (HIDDEN + OUTPUTS)}
    if op == "batch":
        n = sum(_batch_sizes(case))
        m = sum(v // 4 for v in _batch_sizes(case))
    elif op == "stages":
        ms = _stage_sizes(case)
        n, m = case["n"] + sum(ms[:-1]), sum(ms)
        return {"bytes": 12 * n + 20 * m, "flops": 9 * (n + m)}
    else:
        n, m = case["n"], case["m"]
    return {"bytes": 12 * n + 8 * m, "flops": 9 * (n + m)}


# ---------------------------------------------------------------------------
# References in plain torch.  Which point is picked is defined on FP32
# distances (ties to the lower index), so the order is followed in FP32; the
# distance of every pick to its nearest earlier pick is then taken in 64 bits.
# ---------------------------------------------------------------------------
def _fps(clouds, ms, starts, euclid):
    """FPS of several clouds at once: padded rows, one step per pick."""
    b, n = len(clouds), max(c.shape[0] for c in clouds)
    p = torch.zeros(3, b, n, device=DEV)
    d = torch.full((b, n), -1.0, device=DEV)  # padding is never the largest
    for i, c in enumerate(clouds):
        p[:, i, : c.shape[0]] = c.T
        d[i, : c.shape[0]] = math.inf
    rows, steps = torch.arange(b, device=DEV), max(ms)
    near = torch.zeros(b, n, dtype=torch.int64, device=DEV)
    idx = torch.empty(steps, b, dtype=torch.int64, device=DEV)
    src = torch.empty(steps, b, dtype=torch.int64, device=DEV)
    cur = torch.tensor(starts, dtype=torch.int64, device=DEV)
    for j in range(steps):
        idx[j] = cur
        src[j] = near[rows, cur]
        s = p[:, rows, cur]
        q = p - s[:, :, None]
        q = q * q
        q = q[0] + q[1] + q[2]
        if euclid:
            q = torch.sqrt(q.double()).float()
        less = q < d
        d = torch.where(less, q, d)
        near.masked_fill_(less, j)
        cur = torch.argmax(d, dim=1)
    out = []
    for i, c in enumerate(clouds):
        k = idx[: ms[i], i]
        c64 = c.double()
        v = ((c64[k] - c64[k[src[: ms[i], i]]]) ** 2).sum(1)
        v = torch.sqrt(v) if euclid else v
        v[0] = math.inf
        out.append((k, v))
    return out


def exact(case, seed):
    op = case["op"]
    if op in ("single", "auto"):
        x = _cloud(case["cloud"], _gen(seed), case["n"])
        k, v = _fps([x], [case["m"]], [case.get("start", 0)], case.get("euclid", False))[0]
        return {"idx": k.int(), "d2": v}
    if op == "stages":
        x, out = _cloud(case["cloud"], _gen(seed), case["n"]), []
        for m in _stage_sizes(case):
            k, v = _fps([x], [m], [0], False)[0]
            x = x[k].contiguous()
            out.append({"idx": k.int(), "d2": v})
        return {"stages": out, "xyz": x.double()}
    if op == "batch":
        x, offsets, m = _batch_inputs(case, seed)
        got = _fps([x[a:b] for a, b in zip(offsets, offsets[1:])], m, [0] * len(m), False)
        return {"idx": torch.cat([k for k, _ in got]).int(), "d2": torch.cat([v for _, v in got])}
    x, t, w, params = _gradient_inputs(case, seed)
    x, t, w = x.double(), t.double(), w.double()
    cut = [HIDDEN * INPUTS, HIDDEN, HIDDEN * HIDDEN, HIDDEN, OUTPUTS * HIDDEN, OUTPUTS]
    w1, b1, w2, b2, w3, b3 = torch.split(params, cut)
    # weight matrices are used in bfloat16, the gradient passes straight
    # through that rounding
    w1, w2, w3 = (v.bfloat16().double().reshape(s) for v, s in ((w1, (HIDDEN, -1)), (w2, (HIDDEN, HIDDEN)), (w3, (-1, HIDDEN))))
    z1 = x @ w1.T + b1.double()
    a1 = z1.clamp_min(0)
    z2 = a1 @ w2.T + b2.double()
    a2 = z2.clamp_min(0)
    e = a2 @ w3.T + b3.double() - t
    dy = 2.0 * w * e / case["rows"]
    dz2 = (dy @ w3) * (z2 > 0)
    dz1 = (dz2 @ w2) * (z1 > 0)
    grad = torch.cat([v.reshape(-1) for v in (dz1.T @ x, dz1.sum(0), dz2.T @ a1, dz2.sum(0), dy.T @ a2, dy.sum(0))])
    return {"grad": grad, "loss": ((w * e * e).sum() / case["rows"]).reshape(1)}
