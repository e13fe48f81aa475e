"""Segments whose squared length or offsets leave FP32's range in units of the
mesh, and meshes whose box is not that of their triangles.  Bar: flags equal
the oracle's over all triangles, distances have the bits sd3_distance gives
for the degenerate triangles (P0, P1, P1) on the plain FP64 path, and the
threshold filter equals the returned distance's.  Above 2^127, where the
mesh path has no distances, the bar is its error model: 32 u of the extent.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1808_09571_amd import sd3, synth
from test_gpu_segment_tree import TRI1, _check


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def _through(seed, size):
    """Segments of about `size` through a body at the origin, along axes and
    across them, and such that lie on one side of it."""
    g = np.random.default_rng(seed)
    out = []
    for k in range(24):
        u = g.normal(size=3)
        u /= np.linalg.norm(u)
        if k % 3 == 0:
            u = np.eye(3)[k // 3 % 3] * (1 if k % 2 else -1)
        out.append([-u * size * g.uniform(1.0, 1.4), u * size * g.uniform(1.0, 1.4)])
        out.append([u * size * 1.5, u * size * 2.8])
        out.append([u * 0.1, u * size])
    return np.array(out)


@pytest.mark.parametrize("lo,hi,step", [(20.0, 28.0, 1.0), (30.0, 60.0, 5.0), (61.0, 65.0, 0.25), (70.0, 110.0, 20.0)])
def test_long_segments(ctx, lo, hi, step):
    x, t = synth.icosphere(2, radius=0.5)
    seg = np.concatenate([_through(int(8 * e), 2.0 ** e) for e in np.arange(lo, hi + step / 2, step)])
    _check(ctx, seg, (x, t), 0.25)


@pytest.mark.parametrize("size", [130.0, 190.0, 250.0])
def test_longest_segments(ctx, size):
    import torch
    x, t = synth.icosphere(2, radius=0.5)
    seg = _through(int(size), 2.0 ** size)
    mb = sd3.Batch.from_packed(synth.pack([(x, t)]), "cuda:0")
    sg = torch.from_numpy(seg).to("cuda:0")
    d, h = (v.cpu().numpy() for v in ctx.segments("distance", sg, mb))
    hi = ctx.segments("intersects", sg, mb).cpu().numpy()
    w = ctx.segments("within", sg, mb, r=0.25).cpu().numpy()
    for i, (p, q) in enumerate(seg):
        do, ho, _ = oracle.mesh((np.array([p, q, q]), TRI1), (x, t))
        assert bool(h[i]) == ho and bool(hi[i]) == ho and bool(w[i]) == (d[i] <= 0.25), i
        assert abs(d[i] - do) <= 2e-12 * do + 32 * 2.0 ** -53 * 4.2 * 2.0 ** size, (i, d[i], do)


@pytest.mark.parametrize("far", [10.0, 1e3, 1e9])
def test_vertices_of_no_triangle(ctx, far):
    # a vertex that no triangle uses changes nothing: not the results, nor how
    # many triangles are compared
    import torch
    x, t = synth.icosphere(3)
    g = np.random.default_rng(2)
    p = g.uniform(-1.5, 1.5, size=(500, 3))
    seg = np.stack([p, p + g.normal(size=(500, 3)) * 0.3], axis=1)
    sg = torch.from_numpy(seg).to("cuda:0")
    out = []
    for y in (x, np.vstack([x, [[far, -far, 0.0]]])):
        mb = sd3.Batch.from_packed(synth.pack([(y, t)]), "cuda:0")
        for op in ("distance", "intersects", "within"):
            r, st = ctx.segments(op, sg, mb, r=0.1, stats=True)
            out.append((r if op == "distance" else (r,), st["tri_pairs_boxed"], st["tri_pairs_fp64"]))
    for a, b in zip(out[:3], out[3:]):
        assert all(torch.equal(u, v) for u, v in zip(a[0], b[0])) and a[1:] == b[1:]


def test_exact_tests_of_long_segments(ctx):
    # intersects settles near misses without exact arithmetic as distance does
    import torch
    x, t = synth.icosphere(4)
    g = np.random.default_rng(1)
    u = g.normal(size=(500, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    a = g.uniform(-1.2, 1.2, size=(500, 3))
    sg = torch.from_numpy(np.stack([a - 2e6 * u, a + 2e6 * u], axis=1)).to("cuda:0")
    mb = sd3.Batch.from_packed(synth.pack([(x, t)]), "cuda:0")
    (_, h), sd = ctx.segments("distance", sg, mb, stats=True)
    f, si = ctx.segments("intersects", sg, mb, stats=True)
    assert torch.equal(h, f) and si["exact"] <= 2 * sd["exact"], (si["exact"], sd["exact"])
