"""Columns of small rows (every row within one sort block: keys and sort in one
launch, a block per row box) against the general path: the same rows with one
longer row beside them take the general path and must give the same bits, for
row sizes at the edges of a block's rounds, empty sides, vertices no triangle
uses, both precisions and every tile size.  A few rows are checked against the
oracle, and what is refused stays refused.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1808_09571_amd import sd3, synth

EMPTY = (np.zeros((0, 3)), np.zeros((0, 3), np.int32))


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def _soup(n, seed, center=(0.0, 0.0, 0.0), extra=0):
    x, t = synth.random_triangle_soup(n, seed, scale=1.0, center=center, size=0.15)
    if extra:  # vertices no triangle uses, inside the box
        x = np.vstack([np.random.default_rng(seed).uniform(-0.5, 0.5, size=(extra, 3)) + np.asarray(center), x])
        t = t + extra
    return x, t.astype(np.int32)


def _rows():
    sizes = [1, 2, 63, 64, 65, 255, 1023, 1024, 1025, 2047, 2048]
    A, B = [], []
    for i, n in enumerate(sizes):
        A.append(_soup(n, 10 + i, extra=300 if i == 3 else 0))
        B.append(_soup(sizes[-1 - i], 50 + i, center=(2.4 if i % 2 else 0.8, 0.1 * i, 0.2)))
    A += [EMPTY, _soup(5, 3), (np.ones((4, 3)), np.zeros((0, 3), np.int32))]
    B += [_soup(7, 4), EMPTY, _soup(9, 5)]
    return A, B


def _batch(meshes):
    return sd3.Batch.from_packed(synth.pack(meshes), "cuda:0")


@pytest.mark.parametrize("beside", ["triangles", "vertices"])
@pytest.mark.parametrize("tile", [32, 64, 128])
def test_small_rows_equal_the_general_path(ctx, tile, beside):
    A, B = _rows()
    n = len(A)
    # one longer row takes the whole call off the small-row path: by its
    # triangles (keys, sort and boxes) or its vertices alone (boxes)
    long_row = _soup(2049, 99) if beside == "triangles" else _soup(40, 98, extra=8193)
    for prec in ("fp32", "fp64"):
        d, h = (x.cpu().numpy() for x in ctx.distance(_batch(A), _batch(B), precision=prec, tile=tile))
        hi = ctx.intersects(_batch(A), _batch(B), precision=prec, tile=tile).cpu().numpy()
        dg, hg = (x.cpu().numpy() for x in ctx.distance(_batch(A + [long_row]), _batch(B + [_soup(3, 1)]),
                                                        precision=prec, tile=tile))
        assert np.array_equal(d.view(np.int64), dg[:n].view(np.int64))
        assert np.array_equal(h, hg[:n]) and np.array_equal(h, hi)
    for i in (0, 3, 5, 10):
        do, ho, _ = oracle.mesh(A[i], B[i])
        assert bool(h[i]) == ho and abs(d[i] - do) <= 1e-12 * do
    assert np.all(np.isinf(d[11:])) and not h[11:].any()


def test_small_rows_replayed(ctx):
    import torch
    A, B = _rows()
    ba, bb = _batch(A), _batch(B)
    d, h = ctx.distance(ba, bb)
    g = ctx.graph("distance", ba, bb)
    for _ in range(3):
        g.launch()
        g.result()
        assert torch.equal(g.dist, d) and torch.equal(g.hit, h)
        ctx.distance(bb, ba)  # the program's own work between the replays
    g.close()


def test_small_rows_refuse_bad_contents(ctx):
    A, B = _rows()
    lone = (np.array([[0.0, np.inf, 1.0]]), np.zeros((0, 3), np.int32))
    for bad, name in ((lone, "SD3_E_NONFINITE"),
                      ((A[5][0], np.full((3, 3), len(A[5][0]), np.int32)), "SD3_E_INDEX_RANGE"),
                      ((A[5][0] * 2.0 ** 300, A[5][1]), "SD3_E_RANGE")):
        for side in (0, 1):
            rows = [_batch(A + [bad]), _batch(B + [_soup(3, 1)])]
            with pytest.raises(sd3.SD3Error) as e:
                ctx.distance(*(rows if side == 0 else rows[::-1]))
            assert e.value.name == name


@pytest.mark.parametrize("nt", [2048, 2049])
def test_stats_report_the_scatter_passes_that_ran(ctx, nt):
    a, b = _batch([_soup(nt, 1)]), _batch([_soup(9, 2)])
    _, _, st = ctx.distance(a, b, stats=True, timing=True)
    assert st["sort_passes"] == st["n_kernel"]["scatter"] == (0 if nt <= 2048 else 2)
    assert st["sort_item_bytes"] == (0 if nt <= 2048 else 20) and st["sort_items"] == nt + 9


def test_rows_ranked_by_counting_equal_the_general_path(ctx):
    # up to 128 triangles a row; fans share their first vertices, so that every
    # key of the row is the same
    A, B = [], []
    for n in (3, 127, 128, 129, 190):
        x, t = _soup(n, n)
        A += [(x, t), (x, np.stack([np.full(n, t[0, 0]), t[:, 1], t[:, 2]], axis=1).astype(np.int32))]
        B += [_soup(131 - n % 3, n + 1, center=(1.3, 0.2, 0.1))] * 2
    d, h = ctx.distance(_batch(A), _batch(B))
    dg, hg = ctx.distance(_batch(A + [_soup(2049, 99)]), _batch(B + [_soup(3, 1)]))
    assert np.array_equal(d.cpu().numpy(), dg.cpu().numpy()[:len(A)])
    assert np.array_equal(h.cpu().numpy(), hg.cpu().numpy()[:len(A)])
    for i in range(len(A)):
        do, ho, _ = oracle.mesh(A[i], B[i])
        assert bool(h[i]) == ho and abs(float(d[i]) - do) <= 1e-12 * do
