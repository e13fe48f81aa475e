"""The segment path's tree of bounding cylinders: mesh sizes at the edges of
its levels (8, 64, 512, ... triangles a node, at most 16 nodes at the top),
segment counts at the edges of a wave, long, far, tiny and zero-length
segments, and meshes far from the origin or of extreme
scale.  Bar: flags equal the oracle's over all triangles, distances have the
bits sd3_distance gives for the degenerate triangles (P0, P1, P1) on the plain
FP64 path, and the threshold filter equals the returned distance's.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1808_09571_amd import sd3, synth

TRI1 = np.array([[0, 1, 2]], np.int32)


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def _check(ctx, seg, mesh, r):
    import torch
    mb = sd3.Batch.from_packed(synth.pack([mesh]), "cuda:0")
    sg = torch.from_numpy(np.ascontiguousarray(seg)).to("cuda:0")
    d, h = (x.cpu().numpy() for x in ctx.segments("distance", sg, mb))
    hi = ctx.segments("intersects", sg, mb).cpu().numpy().astype(bool)
    w = ctx.segments("within", sg, mb, r=r).cpu().numpy().astype(bool)
    ba = sd3.Batch.from_packed(synth.pack([(np.array([p, q, q]), TRI1) for p, q in seg]), "cuda:0")
    bb = sd3.Batch.from_packed(synth.pack([mesh] * len(seg)), "cuda:0")
    dm, hm = (x.cpu().numpy() for x in ctx.distance(ba, bb, precision="fp64"))
    assert np.array_equal(d.view(np.int64), dm.view(np.int64)), np.nonzero(d != dm)
    ho = np.array([oracle.mesh((np.array([p, q, q]), TRI1), mesh)[1] for p, q in seg])
    assert np.array_equal(h.astype(bool), ho) and np.array_equal(hi, ho) and np.array_equal(hm.astype(bool), ho)
    assert np.array_equal(w, d <= r)


def _segments(seed, n, scale):
    g = np.random.default_rng(seed)
    p = g.uniform(-1.6, 1.6, size=(n, 3)) * scale
    q = p + g.normal(size=(n, 3)) * g.uniform(0.0, 1.0, size=(n, 1)) * scale
    k = max(1, n // 8)
    q[:k] = p[:k]                                        # points
    q[k:2 * k] = p[k:2 * k] + 300.0 * (q - p)[k:2 * k]   # far longer than the mesh
    p[2 * k:3 * k] *= 1000.0                             # far away
    q[2 * k:3 * k] = p[2 * k:3 * k] + g.normal(size=(len(p[2 * k:3 * k]), 3)) * scale
    return np.stack([p, q], axis=1)


@pytest.mark.parametrize("nt,n", [(1, 1), (2, 63), (7, 64), (8, 65), (9, 40), (64, 40), (65, 129), (127, 40),
                                  (128, 40), (129, 40), (513, 40), (1024, 65), (1025, 65), (8193, 65)])
def test_level_edges_against_oracle(ctx, nt, n):
    mesh = synth.random_triangle_soup(nt, 100 + nt, scale=1.0, size=0.6 / nt ** (1 / 3))
    _check(ctx, _segments(nt, n, 1.0), mesh, 0.25)


@pytest.mark.parametrize("scale,shift", [(1.0, 1e6), (2.0 ** 60, 0.0), (2.0 ** -60, 0.0), (1e-3, 1e3)])
def test_scales_against_oracle(ctx, scale, shift):
    x, t = synth.blob(500, 1.0, (0.0, 0.0, 0.0), 5)
    seg = _segments(3, 70, 1.0)
    _check(ctx, seg * scale + shift, (x * scale + shift, t), 0.3 * scale)


def test_flat_and_degenerate_meshes(ctx):
    # a plane grid (cylinders without height), and triangles of no area (a
    # polyline and a single point, whose box has no extent)
    x, t = synth.heightfield(12, 9, 2.0, 2.0, 1, amplitude=0.0)
    seg = _segments(9, 70, 1.0)
    _check(ctx, seg, (x - 1.0, t), 0.2)
    line = np.stack([np.linspace(-1, 1, 30)] * 3, axis=1)
    k = np.arange(29, dtype=np.int32)
    _check(ctx, seg, (line, np.stack([k, k + 1, k + 1], axis=1)), 0.2)
    _check(ctx, seg, (np.array([[0.25, 0.5, -0.125]]), np.zeros((3, 3), np.int32)), 0.2)


@pytest.mark.parametrize("nt,n", [(2047, 17), (2048, 64), (2049, 17), (4097, 17)])
def test_runs_of_the_order(ctx, nt, n):
    # the tree takes each 2048 triangles in the order of a curve: the edges of
    # a run, triangles in no order at all
    mesh = synth.random_triangle_soup(nt, nt, scale=1.0, size=0.05)
    _check(ctx, _segments(nt, n, 1.0), mesh, 0.25)


def test_every_triangle_as_near_as_any(ctx):
    # points and short segments at the centre of a sphere, where no bound
    # tells one triangle from another: the list of pairs to test runs full
    x, t = synth.blob(2000, 1.0, (0.0, 0.0, 0.0), 3)
    x = x / np.linalg.norm(x, axis=1, keepdims=True)
    g = np.random.default_rng(5)
    p = g.normal(size=(130, 3)) * np.array([0.0, 1e-9, 1e-6, 1e-3, 1e-2])[np.arange(130) % 5, None]
    q = p + g.normal(size=(130, 3)) * np.array([0.0, 1e-7, 1e-3])[np.arange(130) % 3, None]
    _check(ctx, np.stack([p, q], axis=1), (x, t), 0.99)


@pytest.mark.parametrize("bad,name", [(np.nan, "SD3_E_NONFINITE"), (-np.inf, "SD3_E_NONFINITE"),
                                      (np.nextafter(2.0 ** 256, np.inf), "SD3_E_RANGE"),
                                      (np.nextafter(2.0 ** -256, 0.0), "SD3_E_RANGE"), (5e-324, "SD3_E_RANGE")])
def test_refused_host_segments(ctx, bad, name):
    # host segments are checked while the kernels run on them: the first one
    # refused is named, no output is written, and the next call is unharmed
    import ctypes
    mb = sd3.Batch.from_packed(synth.pack([synth.blob(100, 1.0, (0.0, 0.0, 0.0), 2)]))
    seg = _segments(4, 70, 1.0)
    good = ctx.segments("distance", seg, mb)
    wrong = seg.copy()
    wrong[66, 1, 2] = wrong[69, 0, 0] = bad
    d, f = np.full(70, 7.0), np.full(70, 7, np.uint8)
    g = mb.geoms()
    st = ctx.lib.sd3_segments(ctx.handle, sd3.SEG_OP["distance"], wrong.ctypes.data, 70, sd3.MEM_HOST,
                              ctypes.byref(g), 0.0, d.ctypes.data, f.ctypes.data, None, None)
    with pytest.raises(sd3.SD3Error, match="segment 66") as e:
        ctx._raise(st)
    assert e.value.name == name and (d == 7.0).all() and (f == 7).all()
    again = ctx.segments("distance", seg, mb)
    assert np.array_equal(good[0], again[0]) and np.array_equal(good[1], again[1])
