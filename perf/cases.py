"""The work a user of sd3 has it do, as timed cases.

A case is a dict of plain values.  `kind` names the entry point: "mesh" (distance /
intersects of two batches of meshes), "segments" (segments against one mesh), "volume"
and "ranker" (a training step of the tile-pair ranker); `data` the inputs, which have
the shapes of `paper_1808_09571_amd/synth.py` (its own generators place vertices row by
row on the host; a batch of thousands of rows is made here on the GPU instead).
"""
import math

import numpy as np
import torch

from paper_1808_09571_amd import ranker, sd3, synth

DEV = "cuda:0"
F64 = torch.float64
_kept = {}


def listed():
    return [
        # one geometry pair, a few thousand triangles: an interactive query, all latency
        {"name": "ico_pair_distance", "kind": "mesh", "data": "ico", "rows": 1, "op": "distance",
         "precision": "fp32", "order": "bound", "launch": "eager", "tile": 0, "semantics": "surface"},
        # two terrain surfaces of 524,288 triangles each (the TIN pair of the benchmark),
        # asked again and again as the survey is edited: a replayed graph
        {"name": "tin512_distance_graph", "kind": "mesh", "data": "tin", "cells": 512, "gap": 0.01,
         "op": "distance", "precision": "fp32", "order": "learned", "launch": "graph", "tile": 0,
         "semantics": "surface"},
        # the largest single pair: 4,000,000-triangle terrain under a 1,003,520-triangle ore body
        {"name": "terrain4m_distance", "kind": "mesh", "data": "terrain_blob", "nx": 2000, "ny": 1000,
         "freq": 224, "gap": 0.001, "op": "distance", "precision": "fp32", "order": "bound",
         "launch": "eager", "tile": 0, "semantics": "surface"},
        # the headline: a whole column of drill-hole tubes against ore bodies (1.7e8 triangles)
        {"name": "holes4096_distance_graph", "kind": "mesh", "data": "tubes", "rows": 4096,
         "op": "distance", "precision": "fp32", "order": "learned", "launch": "graph", "tile": 64,
         "semantics": "surface"},
        # the join predicate over an ordinary column, called without a graph
        {"name": "holes1000_intersects", "kind": "mesh", "data": "tubes", "rows": 1000,
         "op": "intersects", "precision": "fp32", "order": "bound", "launch": "eager", "tile": 0,
         "semantics": "surface"},
        # the plain FP64 option over a column
        {"name": "holes250_distance_fp64", "kind": "mesh", "data": "tubes", "rows": 250,
         "op": "distance", "precision": "fp64", "order": "bound", "launch": "eager", "tile": 0,
         "semantics": "surface"},
        # closed bodies as solids (one inside another counts as touching), a short column
        {"name": "solids150_distance", "kind": "mesh", "data": "bodies", "rows": 150,
         "op": "distance", "precision": "fp32", "order": "bound", "launch": "eager", "tile": 0,
         "semantics": "solid"},
        # the paper's own query: 5,000,000 drill-hole segments against a 500-face ore body
        {"name": "segments5m_distance", "kind": "segments", "holes": 100000, "segs": 50, "freq": 5,
         "op": "distance", "r": 0.0, "mem": "device"},
        # the distance filter against a finely modelled ore body
        {"name": "segments300k_within_mesh20k", "kind": "segments", "holes": 6001, "segs": 50,
         "freq": 32, "op": "within", "r": 2.0, "mem": "device"},
        # a small table held in host memory
        {"name": "segments10k_intersects_host", "kind": "segments", "holes": 333, "segs": 30,
         "freq": 5, "op": "intersects", "r": 0.0, "mem": "host"},
        # volume of a column of ore bodies
        {"name": "volume1000", "kind": "volume", "rows": 1000},
        # a minibatch of the ranker's training: loss, gradients and the Adam update
        {"name": "ranker_step4096", "kind": "ranker", "n": 4096},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ico", "tin", "terrain_blob", "tubes", "tubes", "bodies", "segments", "segments",
                       "volume", "ranker"])
    if kind == "segments":
        freq = _logint(rng, 2, 40)
        segs = rng.randint(1, 70)
        most = min(5e6, 5e6 * 500 / (20 * freq * freq))
        op = rng.choice(["distance", "intersects", "within"])
        return {"kind": "segments", "holes": max(1, _logint(rng, 64, most) // segs), "segs": segs, "freq": freq,
                "op": op, "r": round(math.exp(rng.uniform(-2, 3)), 3) if op == "within" else 0.0,
                "mem": rng.choice(["device", "device", "host"])}
    if kind == "volume":
        return {"kind": "volume", "rows": _logint(rng, 1, 3000)}
    if kind == "ranker":
        return {"kind": "ranker", "n": _logint(rng, 100, 65536)}
    op = rng.choice(["distance", "distance", "intersects"])
    c = {"kind": "mesh", "data": kind, "op": op, "precision": rng.choice(["fp32", "fp32", "fp64"]),
         "order": rng.choice(["bound", "learned"]) if op == "distance" else "bound",
         "launch": rng.choice(["eager", "graph"]), "tile": rng.choice([0, 0, 32, 64, 128]),
         "semantics": "surface"}
    if kind == "ico":
        c["rows"] = _logint(rng, 1, 200)
    elif kind == "tin":
        c.update(cells=_logint(rng, 40, 700), gap=round(math.exp(rng.uniform(-7, 0)), 5))
    elif kind == "terrain_blob":
        c.update(nx=_logint(rng, 150, 2000), ny=_logint(rng, 100, 1000), freq=_logint(rng, 10, 224),
                 gap=round(math.exp(rng.uniform(-8, 0)), 6))
    elif kind == "tubes":
        c["rows"] = _logint(rng, 2, 2000)
    else:
        c.update(rows=_logint(rng, 1, 400), launch="eager", semantics="solid")
    return c


# ---------------------------------------------------------------------------
# inputs, made on the GPU
# ---------------------------------------------------------------------------
def _gpu(x, dtype=F64):
    return torch.as_tensor(x, dtype=dtype).to(DEV)


def _sphere(freq):
    """Geodesic sphere of a frequency: (unit vertices, triangles) on the GPU."""
    key = ("sphere", freq)
    if key not in _kept:
        u, t = synth.geodesic_sphere(freq)
        _kept[key] = (_gpu(u), _gpu(t, torch.int32))
    return _kept[key]


def _ico3():
    if "ico3" not in _kept:
        u, t = synth.icosphere(3)
        _kept["ico3"] = (_gpu(u), _gpu(t, torch.int32))
    return _kept["ico3"]


def _fade(t):
    return t * t * t * (t * (t * 6.0 - 15.0) + 10.0)


def _noise3(u, g, rows, freq=2.0, octaves=2, gain=0.5):
    """Value noise in [-1, 1] of `rows` random lattices at the points u [n, 3]: [rows, n]."""
    total, wsum = 0.0, 0.0
    for o in range(octaves):
        fq = freq * 2.0 ** o
        n = int(math.ceil(2.0 * fq)) + 2
        table = _gpu(g.uniform(-1.0, 1.0, size=(rows, n * n * n)))
        q = (u + 1.0) * fq
        i = q.floor().long().clamp(0, n - 2)
        f = _fade(q - i)
        acc = 0.0
        for dx in (0, 1):
            for dy in (0, 1):
                for dz in (0, 1):
                    w = ((f[:, 0] if dx else 1 - f[:, 0]) * (f[:, 1] if dy else 1 - f[:, 1])
                         * (f[:, 2] if dz else 1 - f[:, 2]))
                    acc = acc + w * table[:, ((i[:, 0] + dx) * n + i[:, 1] + dy) * n + i[:, 2] + dz]
        total = total + gain ** o * acc
        wsum += gain ** o
    return total / wsum


def _offsets(counts):
    off = np.zeros(len(counts) + 1, dtype=np.int64)
    np.cumsum(counts, out=off[1:])
    return off


def _blobs(g, freqs, radius, center, noise=0.3):
    """A batch of ore bodies, one per row: geodesic spheres with radial noise."""
    freqs = np.asarray(freqs, dtype=np.int64)
    v_off, t_off = _offsets(10 * freqs ** 2 + 2), _offsets(20 * freqs ** 2)
    xyz = torch.empty((int(v_off[-1]), 3), dtype=F64, device=DEV)
    tri = torch.empty((int(t_off[-1]), 3), dtype=torch.int32, device=DEV)
    radius = np.broadcast_to(np.asarray(radius, dtype=np.float64), freqs.shape)
    for f in np.unique(freqs):
        rows = np.nonzero(freqs == f)[0]
        u, t = _sphere(int(f))
        r = _gpu(radius[rows])[:, None] * (1.0 + noise * _noise3(u, g, len(rows)))
        at = _gpu(v_off[rows], torch.int64)[:, None] + torch.arange(u.shape[0], device=DEV)
        xyz[at.reshape(-1)] = (u[None] * r[:, :, None] + _gpu(center[rows])[:, None]).reshape(-1, 3)
        at = _gpu(t_off[rows], torch.int64)[:, None] + torch.arange(t.shape[0], device=DEV)
        tri[at.reshape(-1)] = t.repeat(len(rows), 1)
    return sd3.Batch(xyz.reshape(-1), tri.reshape(-1), v_off, t_off)


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _perp(d):
    x = torch.zeros_like(d)
    x[..., 0] = (d[..., 0].abs() < 0.9).to(F64)
    x[..., 1] = 1.0 - x[..., 0]
    return _unit(torch.linalg.cross(d, x))


def _tubes(g, nseg, aim, dirn, radius=0.05, sides=16):
    """A batch of drill holes, one per row: gently curving polylines of nseg steps through
    `aim`, swept with a 16-gon on parallel-transport frames, closed by two fan caps."""
    R, nseg = len(nseg), np.asarray(nseg, dtype=np.int64)
    half = nseg // 2
    S = int((nseg - half).max())
    ang = _gpu(np.radians(g.uniform(0.0, 5.0, size=(S, 2 * R))))
    phi = _gpu(g.uniform(0.0, 2 * math.pi, size=(S, 2 * R)))
    step = _gpu(g.uniform(0.2, 0.4, size=(S, 2 * R)))
    d, p = _gpu(np.concatenate([dirn, -dirn])), _gpu(np.concatenate([aim, aim]))
    pts = torch.empty((S + 1, 2 * R, 3), dtype=F64, device=DEV)
    pts[0] = p
    ca, sa, cp, sp = (x[:, :, None] for x in (ang.cos(), ang.sin(), phi.cos(), phi.sin()))
    for s in range(S):  # each step turns by at most 5 degrees about a random axis
        ax = _perp(d)
        d = _unit(ca[s] * d + sa[s] * (cp[s] * ax + sp[s] * torch.linalg.cross(d, ax)))
        p = p + step[s][:, None] * d
        pts[s + 1] = p
    M = int(nseg.max()) + 1
    n, h = _gpu(nseg, torch.int64)[:, None], _gpu(half, torch.int64)[:, None]
    j = torch.arange(M, device=DEV)[None].expand(R, M)
    jc = torch.minimum(j, n)
    k = jc - h
    row = torch.arange(R, device=DEV)[:, None]
    path = pts[k.abs(), torch.where(k < 0, row + R, row)]
    del pts
    lo, hi = (jc - 1).clamp(min=0), torch.minimum(jc + 1, n)
    tang = _unit(path[row, hi] - path[row, lo]).transpose(0, 1).contiguous()
    nrm = torch.empty_like(tang)
    nrm[0] = _perp(tang[0])
    for i in range(1, M):
        v = nrm[i - 1] - (nrm[i - 1] * tang[i]).sum(-1, keepdim=True) * tang[i]
        nrm[i] = _unit(v)
    nrm, tang = nrm.transpose(0, 1), tang.transpose(0, 1)
    live = j <= n
    path, nrm, bi = path[live], nrm[live], torch.linalg.cross(tang, nrm)[live]
    th = 2 * math.pi * torch.arange(sides, dtype=F64, device=DEV) / sides
    xyz = path[:, None] + radius * (th.cos()[None, :, None] * nrm[:, None] + th.sin()[None, :, None] * bi[:, None])
    counts = 2 * sides * nseg + 2 * (sides - 2)
    t_off, v_off = _offsets(counts), _offsets(sides * (nseg + 1))
    total = int(t_off[-1])
    rows = torch.repeat_interleave(torch.arange(R, device=DEV), _gpu(counts, torch.int64), output_size=total)
    t = torch.arange(total, device=DEV) - _gpu(t_off[:-1], torch.int64)[rows]
    wall = 2 * sides * _gpu(nseg, torch.int64)[rows]
    i, s = t // (2 * sides), (t % (2 * sides)) // 2
    a, b = i * sides + s, i * sides + (s + 1) % sides
    odd = t % 2 == 1
    tri = torch.stack([a, torch.where(odd, b + sides, b), torch.where(odd, a + sides, b + sides)], dim=1)
    c = t - wall
    last = (wall // (2 * sides)) * sides
    kk = c // 2 + 1
    c = c % 2 == 1
    cap = torch.stack([torch.where(c, last, 0), torch.where(c, last + kk, kk + 1), torch.where(c, last + kk + 1, kk)], dim=1)
    tri = torch.where((t < wall)[:, None], tri, cap).to(torch.int32)
    return sd3.Batch(xyz.reshape(-1).contiguous(), tri.reshape(-1).contiguous(), v_off, t_off)


def _loguniform(g, lo, hi, n):
    return np.exp(g.uniform(math.log(lo), math.log(hi), size=n))


def _ore_freqs(g, rows):
    return np.maximum(1, np.round(np.sqrt(_loguniform(g, 1000, 200000, rows) / 20.0))).astype(np.int64)


def _tube_rows(g, rows):
    """Drill-hole tubes (200-20,000 triangles) against ore bodies (1,000-200,000), about a
    third of the rows touching."""
    nseg = np.maximum(1, np.round((_loguniform(g, 200, 20000, rows) - 28) / 32)).astype(np.int64)
    freqs = _ore_freqs(g, rows)
    center = g.uniform(-100.0, 100.0, size=(rows, 3))
    d = g.normal(size=(rows, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    off = np.cross(d, g.normal(size=(rows, 3)))
    off /= np.linalg.norm(off, axis=1, keepdims=True)
    aim = center + g.uniform(0.0, 3.3 * 5.0, size=(rows, 1)) * off
    return _tubes(g, nseg, aim, d), _blobs(g, freqs, 5.0, center)


def _terrain(g, nx, ny, sx, sy, amplitude=50.0, octaves=6):
    """Heights [nx + 1, ny + 1] of fractal value noise over [0, sx] x [0, sy]."""
    x, y = torch.linspace(0, sx, nx + 1, dtype=F64, device=DEV), torch.linspace(0, sy, ny + 1, dtype=F64, device=DEV)
    L, total, wsum = max(sx, sy), 0.0, 0.0
    for o in range(octaves):
        fq, w = 4.0 * 2.0 ** o, 0.5 ** o
        m, n = int(math.ceil(fq * sx / L)) + 2, int(math.ceil(fq * sy / L)) + 2
        table = _gpu(g.uniform(-1.0, 1.0, size=(m, n)))
        u, v = x / L * fq, y / L * fq
        i, j = u.floor().long().clamp(0, m - 2), v.floor().long().clamp(0, n - 2)
        fu, fv = _fade(u - i)[:, None], _fade(v - j)[None]
        a = table[i][:, j] * (1 - fu) + table[i + 1][:, j] * fu
        b = table[i][:, j + 1] * (1 - fu) + table[i + 1][:, j + 1] * fu
        total = total + w * (a * (1 - fv) + b * fv)
        wsum += w
    return x, y, amplitude * total / wsum


def _grid(x, y, z):
    nx, ny = len(x) - 1, len(y) - 1
    xyz = torch.stack([x[:, None].expand_as(z), y[None].expand_as(z), z], dim=2)
    v00 = (torch.arange(nx, device=DEV)[:, None] * (ny + 1) + torch.arange(ny, device=DEV)[None]).reshape(-1)
    v10, v01, v11 = v00 + ny + 1, v00 + 1, v00 + ny + 2
    tri = torch.stack([v00, v10, v11, v00, v11, v01], dim=1).to(torch.int32)
    return sd3.Batch(xyz.reshape(-1).contiguous(), tri.reshape(-1).contiguous(),
                     np.array([0, (nx + 1) * (ny + 1)], np.int64), np.array([0, 2 * nx * ny], np.int64))


def _meshes(case, g):
    """The two batches of a mesh case."""
    d = case["data"]
    if d == "ico":
        R, (u, t) = case["rows"], _ico3()
        off = np.array([2.5, 0.0, 0.0]) + g.uniform(-0.6, 0.6, size=(R, 3))
        v_off, t_off = _offsets([u.shape[0]] * R), _offsets([t.shape[0]] * R)
        tri = t.repeat(R, 1).reshape(-1)
        return (sd3.Batch(u.repeat(R, 1).reshape(-1), tri, v_off, t_off),
                sd3.Batch((u[None] + _gpu(off)[:, None]).reshape(-1), tri.clone(), v_off, t_off))
    if d == "tin":
        n = case["cells"]
        ext = 1000.0 * n / 512
        x, y, za = _terrain(g, n, n, ext, ext)
        _, _, zb = _terrain(g, n, n, ext, ext)
        return _grid(x, y, za), _grid(x, y, zb + (case["gap"] - (zb - za).min()))
    if d == "terrain_blob":
        # the body's lowest vertex straight above the terrain's highest
        nx, ny = case["nx"], case["ny"]
        x, y, z = _terrain(g, nx, ny, float(nx), float(ny))
        a = _grid(x, y, z)
        b = _blobs(g, [case["freq"]], 50.0, np.zeros((1, 3)))
        va, vb = a.xyz.view(-1, 3), b.xyz.view(-1, 3)
        shift = va[va[:, 2].argmax()] - vb[vb[:, 2].argmin()]
        shift[2] += case["gap"]
        vb += shift
        return a, b
    if d == "tubes":
        return _tube_rows(g, case["rows"])
    # bodies: small closed bodies inside, across or beside a larger one
    R = case["rows"]
    a = _blobs(g, g.integers(2, 9, size=R), g.uniform(0.1, 0.4, size=R), g.uniform(-1.2, 1.2, size=(R, 3)), 0.15)
    return a, _blobs(g, g.integers(4, 11, size=R), 1.0, np.zeros((R, 3)), 0.15)


def _context():
    if "ctx" not in _kept:
        _kept["ctx"] = sd3.Context(0)
        _kept["weights"] = ranker.load(device=DEV)
    return _kept["ctx"]


def prepare(case, seed):
    g = np.random.Generator(np.random.PCG64(int(seed)))
    ctx = _context()
    s = {"case": case, "ctx": ctx}
    if case["kind"] == "mesh":
        a, b = _meshes(case, g)
        w = _kept["weights"] if case["order"] == "learned" else None
        s.update(a=a, b=b, ranker=w)
        if case["launch"] == "graph":
            s["graph"] = ctx.graph(case["op"], a, b, precision=case["precision"], order=case["order"],
                                   ranker=w, tile=case["tile"])
    elif case["kind"] == "segments":
        R = 50.0
        seg = synth.drill_holes(case["holes"], case["segs"], int(seed), 1.5 * R, 1.3 * R + 5.0)
        m = _blobs(g, [case["freq"]], R, np.zeros((1, 3)))
        if case["mem"] == "host":
            m = sd3.Batch(m.xyz.cpu().numpy(), m.tri.cpu().numpy(), m.v_off, m.t_off)
        s.update(mesh=m, seg=seg if case["mem"] == "host" else torch.from_numpy(seg).to(DEV))
    elif case["kind"] == "volume":
        R = case["rows"]
        s["g"] = _blobs(g, _ore_freqs(g, R), 5.0, g.uniform(-100.0, 100.0, size=(R, 3)))
    else:
        # some hundred steps into a training: the moments are those of gradients
        n, P = case["n"], sd3.MLP_NPARAM
        x = g.normal(size=(n, sd3.MLP_NIN))
        t = x[:, 0] - 0.5 * np.abs(x[:, 1]) + 0.1 * g.normal(size=n)
        s.update(r=sd3.Ranker(ctx), p=_gpu(ranker.init_params(int(seed) % 1000), torch.float32),
                 x=_gpu(x, torch.float32), t=_gpu(t, torch.float32),
                 m=_gpu(0.01 * g.normal(size=P), torch.float32),
                 v=_gpu(1e-4 * g.uniform(0.5, 2.0, size=P), torch.float32), step=500)
    return s


def run(s):
    c, ctx = s["case"], s["ctx"]
    if c["kind"] == "mesh":
        if c["launch"] == "graph":
            gr = s["graph"]
            gr.launch()
            return (gr.dist, gr.hit) if c["op"] == "distance" else gr.hit
        if c["op"] == "distance":
            return ctx.distance(s["a"], s["b"], precision=c["precision"], order=c["order"], ranker=s["ranker"],
                                tile=c["tile"], semantics=c["semantics"])
        return ctx.intersects(s["a"], s["b"], precision=c["precision"], tile=c["tile"], semantics=c["semantics"])
    if c["kind"] == "segments":
        return ctx.segments(c["op"], s["seg"], s["mesh"], r=c["r"])
    if c["kind"] == "volume":
        return ctx.volume(s["g"])
    loss, grad = s["r"].loss_grad(s["p"], s["x"], s["t"])
    s["r"].adam(s["p"], grad, s["m"], s["v"], s["step"], lr=2e-3)
    s["step"] += 1
    return loss, grad, s["p"], s["m"], s["v"]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _mean_ore():
    """Triangles of a row's ore body on average, and of its drill hole."""
    return 199000 / math.log(200.0), 19800 / math.log(100.0)


def work(case):
    """Bytes: every input once, every output once (a closed mesh and a grid have half as many
    vertices as triangles).  Operations: the tests of one triangle pair a row (or one
    segment and triangle), 700 each, the terms of a volume, the products of the network."""
    k = case["kind"]
    if k == "ranker":
        n, P = case["n"], sd3.MLP_NPARAM
        return {"bytes": 4 * (n * 11 + 8 * P), "flops": 6 * 9024 * n}
    if k == "segments":
        n = case["holes"] * case["segs"]
        return {"bytes": 48 * n + (9 if case["op"] == "distance" else 1) * n + 24 * 20 * case["freq"] ** 2,
                "flops": 700 * n}
    if k == "volume":
        nt = case["rows"] * _mean_ore()[0]
        return {"bytes": 24 * nt + 8 * case["rows"], "flops": 20 * nt}
    rows = case.get("rows", 1)
    d = case["data"]
    if d == "ico":
        nt = 2560 * rows
    elif d == "tin":
        nt = 4 * case["cells"] ** 2
    elif d == "terrain_blob":
        nt = 2 * case["nx"] * case["ny"] + 20 * case["freq"] ** 2
    elif d == "tubes":
        nt = rows * sum(_mean_ore())
    else:
        nt = rows * 20 * (29 + 53)
    return {"bytes": 24 * nt + 9 * rows, "flops": 700 * rows}


# ---------------------------------------------------------------------------
# 64-bit values in plain torch
# ---------------------------------------------------------------------------
def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _sub(a, b):
    return [x - y for x, y in zip(a, b)]


def _crs(a, b):
    return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]


def _div(a, b):
    return a / torch.where(b == 0, 1.0, b)


def _seg_seg(p, d1, q, d2):
    """Squared distance of p + s d1 and q + t d2, s and t in [0, 1]."""
    r = _sub(p, q)
    a, e, b, c, f = _dot(d1, d1), _dot(d2, d2), _dot(d1, d2), _dot(d1, r), _dot(d2, r)
    s = _div(b * f - c * e, a * e - b * b).clamp(0, 1)
    t = _div(b * s + f, e)
    tc = t.clamp(0, 1)
    s = torch.where(t == tc, s, _div(b * tc - c, a).clamp(0, 1))
    w = [r[i] + s * d1[i] - tc * d2[i] for i in range(3)]
    return _dot(w, w)


def _point_face(p, v, e1, e2, n, nn):
    """Squared distance of p to the triangle's plane where its foot lies inside, else inf."""
    r = _sub(p, v)
    u, w = _dot(_crs(r, e2), n), _dot(_crs(e1, r), n)
    h = _dot(r, n)
    inside = (u >= 0) & (w >= 0) & (u + w <= nn)
    return torch.where(inside & (nn > 0), h * h / torch.where(nn > 0, nn, 1.0), math.inf)


def _crosses(p, q, v, e1, e2, n, nn):
    """Whether the segment p q meets the triangle (in general position)."""
    d = _sub(q, p)
    hp, hq = _dot(_sub(p, v), n), _dot(_sub(q, v), n)
    s = _div(hp, hp - hq)
    r = [p[i] + s * d[i] - v[i] for i in range(3)]
    u, w = _dot(_crs(r, e2), n), _dot(_crs(e1, r), n)
    return (hp * hq <= 0) & (hp != hq) & (u >= 0) & (w >= 0) & (u + w <= nn)


def _tri_parts(v):
    e1, e2 = _sub(v[1], v[0]), _sub(v[2], v[0])
    n = _crs(e1, e2)
    return e1, e2, n, _dot(n, n)


def _pairs(A, B):
    """(smallest distance, whether they meet) over all of A's triangles, for each of B's.
    A: 3 corners (or the 2 of a segment) of 3 coordinates [na, 1]; B: 3 of [1, nb]."""
    d2, hit = None, None
    ea = [(0, 1)] if len(A) == 2 else [(0, 1), (1, 2), (2, 0)]
    tb = _tri_parts(B)

    def low(x):
        nonlocal d2
        d2 = x if d2 is None else torch.minimum(d2, x)

    def meets(x):
        nonlocal hit
        hit = x if hit is None else hit | x

    for i, j in ea:
        da = _sub(A[j], A[i])
        for k, m in ((0, 1), (1, 2), (2, 0)):
            low(_seg_seg(A[i], da, B[k], _sub(B[m], B[k])))
        meets(_crosses(A[i], A[j], B[0], *tb))
    for p in A:
        low(_point_face(p, B[0], *tb))
    if len(A) == 3:
        ta = _tri_parts(A)
        for p in B:
            low(_point_face(p, A[0], *ta))
        for k, m in ((0, 1), (1, 2), (2, 0)):
            meets(_crosses(B[k], B[m], A[0], *ta))
    return torch.where(hit, 0.0, d2.clamp(min=0).sqrt())


def _corners(b, g):
    xyz = b.xyz.view(-1, 3)[int(b.v_off[g]):int(b.v_off[g + 1])]
    return xyz[b.tri.view(-1, 3)[int(b.t_off[g]):int(b.t_off[g + 1])].long()]


def _inside(p, T):
    """Winding number of the closed mesh T [n, 3, 3] about p, as a truth value."""
    r = T - p
    ln = r.norm(dim=2)
    a, b, c = r[:, 0], r[:, 1], r[:, 2]
    num = (a * torch.linalg.cross(b, c)).sum(1)
    den = (ln.prod(1) + (a * b).sum(1) * ln[:, 2] + (b * c).sum(1) * ln[:, 0] + (c * a).sum(1) * ln[:, 1])
    return float(torch.atan2(num, den).sum().abs()) > math.pi


def _lanes(T, first):
    return [[T[:, k, i][:, None] if first else T[:, k, i][None] for i in range(3)] for k in range(T.shape[1])]


def exact(case, seed):
    g = np.random.Generator(np.random.PCG64(int(seed)))
    k = case["kind"]
    if k == "mesh":
        if case["op"] != "distance" or case["data"] not in ("ico", "bodies"):
            return None  # whole numbers, or too many triangle pairs
        a, b = _meshes(case, g)
        out = []
        for r in range(case["rows"]):
            A, B = _corners(a, r), _corners(b, r)
            d = min(float(_pairs(_lanes(A[i:i + 512], True), _lanes(B, False)).min()) for i in range(0, len(A), 512))
            if case["semantics"] == "solid" and (_inside(A[0, 0], B) or _inside(B[0, 0], A)):
                d = 0.0
            out.append(d)
        return torch.tensor(out, dtype=F64), None
    if k == "segments":
        if case["op"] != "distance":
            return None
        seg = torch.from_numpy(synth.drill_holes(case["holes"], case["segs"], int(seed), 75.0, 70.0)).to(DEV)
        T = _lanes(_corners(_blobs(g, [case["freq"]], 50.0, np.zeros((1, 3))), 0), False)
        if len(seg) * 20 * case["freq"] ** 2 > 3e9:
            return None
        n = max(1, 30_000_000 // (20 * case["freq"] ** 2))
        return torch.cat([_pairs(_lanes(seg[i:i + n], True), T).amin(1) for i in range(0, len(seg), n)]), None
    if k == "volume":
        R = case["rows"]
        b = _blobs(g, _ore_freqs(g, R), 5.0, g.uniform(-100.0, 100.0, size=(R, 3)))
        out = []
        for r in range(R):
            T = _corners(b, r)
            o = T[0, 0].clone()  # any origin: near the body the terms hardly cancel
            u, v, w = (T[:, i] - o for i in range(3))
            out.append((u * torch.linalg.cross(v, w)).sum() / 6)
        return torch.stack(out)
    s = prepare(case, seed)
    p, x, t, m, v = (s[q].double() for q in ("p", "x", "t", "m", "v"))
    p.requires_grad_(True)
    h, at = x, 0
    for i, (o, q) in enumerate(((64, 10), (64, 64), (64, 64), (1, 64))):
        w = p[at:at + o * q].view(o, q)
        h = h @ w.T + p[at + o * q:at + o * q + o]
        h = h.relu() if i < 3 else h
        at += o * q + o
    loss = (h[:, 0] - t).square().mean()
    (gr,) = torch.autograd.grad(loss, p)
    m = 0.9 * m + 0.1 * gr
    v = 0.999 * v + 0.001 * gr * gr
    step = s["step"]
    p = p.detach() - 2e-3 * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
    return loss.detach().view(1), gr, p, m, v
