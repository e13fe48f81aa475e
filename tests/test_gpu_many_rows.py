"""Columns of more rows than one launch has threads for a block per row: a
launch takes fewer than 2^32 threads, 2^24 blocks of 256.  Bar: the rows of a
small column at the ends and in the middle have the bits they have alone.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1808_09571_amd import sd3, synth


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def test_volume_of_2_24_rows(ctx):
    import torch
    # bodies at rows 0, n / 2 and n - 1, a triangle through the origin (of
    # volume 0) in every other row
    n = (1 << 24) + 5
    bodies = [synth.icosphere(2, radius=1.5), synth.blob(5000, 2.0, (1.0, 2.0, 3.0), 4), synth.cube((0, 0, 0), 1.0)]
    at = [0, n // 2, n - 1]
    nv, nt = np.full(n, 3, np.int64), np.full(n, 1, np.int64)
    for r, (x, t) in zip(at, bodies):
        nv[r], nt[r] = len(x), len(t)
    v_off, t_off = (np.concatenate([[0], np.cumsum(c)]) for c in (nv, nt))
    flat = torch.tensor([0.0, 0.0, 0.0, 1.0, 0.5, 0.25, 0.25, 1.0, 0.5], dtype=torch.float64, device="cuda:0")
    one = torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda:0")
    px, pt = [], []
    for k, (x, t) in enumerate(bodies):
        px.append(torch.from_numpy(np.ascontiguousarray(x).reshape(-1)).to("cuda:0"))
        pt.append(torch.from_numpy(np.ascontiguousarray(t, np.int32).reshape(-1)).to("cuda:0"))
        if k < 2:
            px.append(flat.repeat(at[k + 1] - at[k] - 1))
            pt.append(one.repeat(at[k + 1] - at[k] - 1))
    xyz, tri = torch.cat(px), torch.cat(pt)
    v = ctx.volume(sd3.Batch(xyz, tri, v_off, t_off))
    alone = ctx.volume(sd3.Batch.from_packed(synth.pack(bodies), "cuda:0"))
    assert torch.equal(v[torch.tensor(at, device="cuda:0")], alone)
    v[torch.tensor(at, device="cuda:0")] = 0.0
    assert not bool(v.any())


def test_distance_of_a_sparse_column_of_2_23_rows(ctx):
    import torch
    # three rows of bodies, every other row empty on both sides
    n = (1 << 23) + 3
    at = np.array([0, n // 2, n - 1])
    A, B = zip(*(synth.config_icospheres(k) for k in range(3)))

    def sparse(meshes):
        p = synth.pack(list(meshes))
        nv, nt = np.zeros(n, np.int64), np.zeros(n, np.int64)
        nv[at], nt[at] = np.diff(p.v_off), np.diff(p.t_off)
        b = sd3.Batch.from_packed(p, "cuda:0")
        return b, sd3.Batch(b.xyz, b.tri, *(np.concatenate([[0], np.cumsum(c)]) for c in (nv, nt)))

    (a3, a), (b3, b) = sparse(A), sparse(B)
    d, h = ctx.distance(a, b)
    d3, h3 = ctx.distance(a3, b3)
    rows = torch.from_numpy(at).to("cuda:0")
    assert torch.equal(d[rows], d3) and torch.equal(h[rows], h3)
    d[rows] = float("inf")
    h[rows] = 0
    assert bool(torch.isinf(d).all()) and not bool(h.any())
