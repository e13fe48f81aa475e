"""Long segments against the box that intersects and within cut them to: lines
through and just beside its corners, edges and faces, along its axes, of every
length about the one from which they are cut, and thresholds that are some
segment's own distance.  Bar: flags equal the oracle's over all triangles,
distances have the bits sd3_distance gives for the degenerate triangles
(P0, P1, P1) on the plain FP64 path, and the threshold filter equals the
returned distance's.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1808_09571_amd import sd3, synth
from test_gpu_segment_tree import _check


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def _grazing(seed, lo, hi):
    """Lines through points of the box's surface (corners, edges, faces) moved
    by nothing, by little or by some of the box."""
    g = np.random.default_rng(seed)
    out = []
    for k in range(220):
        on = g.integers(0, 3, size=3)             # a face's own plane or between
        p = np.where(on == 0, lo, np.where(on == 1, hi, g.uniform(lo, hi)))
        u = np.eye(3)[k % 3] if k % 4 == 0 else g.normal(size=3)
        u = u / np.linalg.norm(u)
        p = p + g.normal(size=3) * (0.0, 1e-9, 1e-3, 0.3)[k // 4 % 4]
        n = (0.4, 0.51, 1.0, 3.0, 40.0, 1e4, 1e7)[k % 7]
        t = g.uniform(-0.1, 1.1)
        out.append([p - t * n * u, p + (1.0 - t) * n * u])
    return np.array(out)


def _own(ctx, seg, mesh):
    import torch
    mb = sd3.Batch.from_packed(synth.pack([mesh]), "cuda:0")
    d = np.sort(ctx.segments("distance", torch.from_numpy(seg).to("cuda:0"), mb)[0].cpu().numpy())
    d = d[d > 0.0]
    return [0.0, d[0], d[len(d) // 3], d[2 * len(d) // 3], d[-1]]


@pytest.mark.parametrize("kind", ["cube", "body", "plane", "line"])
def test_lines_about_the_box(ctx, kind):
    if kind == "cube":
        mesh = synth.cube((-0.5, -0.5, -0.5), 1.0)
    elif kind == "body":
        mesh = synth.blob(300, 1.0, (3.0, -2.0, 1.0), 4)
    elif kind == "plane":      # a box without height
        x, t = synth.heightfield(9, 7, 2.0, 1.0, 1, amplitude=0.0)
        mesh = (x - 0.5, t)
    else:                      # triangles without area along an axis
        x = np.zeros((20, 3))
        x[:, 1] = np.linspace(-1.0, 1.0, 20)
        k = np.arange(19, dtype=np.int32)
        mesh = (x, np.stack([k, k + 1, k + 1], axis=1))
    seg = _grazing(7, mesh[0].min(axis=0), mesh[0].max(axis=0))
    for r in _own(ctx, seg, mesh):
        _check(ctx, seg, mesh, r)


def test_a_long_segment_beside_many_triangles(ctx):
    # one that leaves the box is compared with few of its triangles
    import torch
    mesh = synth.random_triangle_soup(20000, 3, scale=1.0, size=0.3)
    mb = sd3.Batch.from_packed(synth.pack([mesh]), "cuda:0")
    p = mesh[0].max(axis=0) + 0.05
    sg = torch.from_numpy(np.array([[p, p + 20.0], [p * [1, 0, 0], p * [40, 0, 0] + [0, 9, 9]]])).to("cuda:0")
    for op in ("intersects", "within"):
        f, st = ctx.segments(op, sg, mb, r=0.01, stats=True)
        assert not f.cpu().numpy().any() and st["tri_pairs_fp64"] <= 200, st
