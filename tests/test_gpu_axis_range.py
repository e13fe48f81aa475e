"""The separating-axis culls of the triangle-pair pass where their arithmetic
leaves its range: rows far from the origin (the FP64 corners are absolute
coordinates, the row's margin only a part of its extent), and scales at which
products of FP32 coordinates overflow.

Bar, as for the culls at ordinary scales: flags exact, distances within
2e-12 d + 32 u S of the oracle's (twice the FP64 error model of a pair
distance), FP32 with rescue and plain FP64 the same bits.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1808_09571_amd import sd3, synth

U = 2.0 ** -53
TRI1 = np.array([[0, 1, 2]], np.int32)


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def _check(ctx, A, B, tile):
    ba = sd3.Batch.from_packed(synth.pack(A), "cuda:0")
    bb = sd3.Batch.from_packed(synth.pack(B), "cuda:0")
    out = {}
    for prec in ("fp64", "fp32"):
        d, h = (x.cpu().numpy() for x in ctx.distance(ba, bb, precision=prec, tile=tile))
        hi = ctx.intersects(ba, bb, precision=prec, tile=tile).cpu().numpy()
        assert np.array_equal(h, hi), prec
        for i in range(len(A)):
            do, ho, _ = oracle.mesh(A[i], B[i])
            pts = np.vstack([A[i][0], B[i][0]])
            S = float(np.max(pts.max(axis=0) - pts.min(axis=0)))
            assert bool(h[i]) == ho, (prec, i, d[i], do)
            assert abs(d[i] - do) <= 2e-12 * do + 32 * U * S, (prec, i, d[i], do, S)
        out[prec] = d
    assert np.array_equal(out["fp32"].view(np.int64), out["fp64"].view(np.int64))


def _far_rows(seed):
    """Rows whose nearest pair of triangles is the only one there is, and small
    bodies, up to 2^40 of their size from the origin."""
    g = np.random.default_rng(seed)
    A, B = [], []

    def unit():
        v = g.normal(size=3)
        return v / np.linalg.norm(v)

    for far in (1e3, 1e6, 7e6, 2.0 ** 40):
        for gap in (10.0, 1.0, 0.5):
            for _ in range(12):
                p = unit() * far
                q = p + unit() * gap
                A.append((np.array([p, p, p]), TRI1))  # points
                B.append((np.array([q, q, q]), TRI1))
                w = unit() * gap                       # facing first vertices
                s, t = unit(), unit()
                A.append((np.array([p, p - w + s, p - w + t]), TRI1))
                B.append((np.array([p + w, p + 2 * w + s, p + 2 * w + t]), TRI1))
        for _ in range(3):
            c = unit() * far
            x, t = synth.icosphere(1)
            y, s = synth.icosphere(1)
            A.append((x + c, t))
            B.append((y * 0.5 + c + unit() * 1.75, s))
    return A, B


@pytest.mark.parametrize("tile", [32, 64, 128])
def test_rows_far_from_the_origin(ctx, tile):
    A, B = _far_rows(tile)
    _check(ctx, A, B, tile)


def test_single_rows_far_from_the_origin(ctx):
    A, B = _far_rows(3)
    for i in range(72, 144, 5):  # (calls of one row bound it by other kernels)
        _check(ctx, A[i:i + 1], B[i:i + 1], 0)


def _scale_rows(s):
    """Gaps well below the bodies' size, off the centre of their tile: corners
    in the frame of a tile are some 2^0 s, the separations of single pairs
    some 2^-5 s to 2^-1 s."""
    t = np.array([[0, 0, 1], [0.1, 0, 1], [0, 0.1, 1]])
    two = (np.vstack([t, t * [1, 1, -1]]), np.array([[0, 1, 2], [3, 4, 5]], np.int32))
    A, B = [], []
    for gap in (0.05, 0.1, 0.2, 0.3, 0.6):
        A.append(two)
        B.append((t + [0, 0, gap], TRI1))
    x, f = synth.icosphere(2)
    A += [(x, f)] * 3
    B += [(x * 1.03125, f), (x[f[0]] * 1.015625, TRI1), synth.blob(500, 0.8, (1.7, 0.9, 0.2), 1)]
    return [(x * s, f) for x, f in A], [(x * s, f) for x, f in B]


# every product of two corners leaves FP32's range near 2^64, every corner
# near 2^128
@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("lo,hi,step", [(58.0, 68.0, 0.25), (119.0, 127.0, 0.5), (-50.0, -40.0, 2.0)])
def test_scales(ctx, lo, hi, step, tile):
    A, B = [], []
    for e in np.arange(lo, hi + step, step):
        a, b = _scale_rows(2.0 ** e)
        A += a
        B += b
    _check(ctx, A, B, tile)


def _small_rows(seed):
    """Single triangles that cross, miss each other closely, or lie far apart."""
    g = np.random.default_rng(seed)
    A, B = [], []
    for k in range(60):
        x, y = g.normal(size=(2, 3, 3))
        A.append((x, TRI1))
        B.append((y * 0.5 + [0.0, 0.0, (0.0, 0.5, 2.5)[k % 3]], TRI1))
    return A, B


# the FP32 pass's squares lose bits to underflow from about 2^-50 on, an axis
# decides nothing below 2^-60, the triple products of the flags are denormal
# near 2^-44
@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("lo,hi,step", [(-56.0, -38.0, 2.0), (-76.0, -57.0, 1.0), (-110.0, -80.0, 10.0)])
def test_small_scales(ctx, lo, hi, step, tile):
    A, B = [], []
    for e in np.arange(lo, hi + step / 2, step):
        for a, b in (_scale_rows(1.0), _small_rows(int(-e))):
            A += [(x * 2.0 ** e, t) for x, t in a]
            B += [(x * 2.0 ** e, t) for x, t in b]
    _check(ctx, A, B, tile)
