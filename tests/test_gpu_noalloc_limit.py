"""Allocation-free calls at the limit of their static scratch: 128 MiB of a
call's buffers with one copy of the counters, which the replicas (4096 bytes of
them) do not take from.
"""
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1808_09571_amd import sd3, synth

LIMIT = (128 << 20) + 4096


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sd3.Context(0)


def _need(ctx, a, b, **kw):
    """(bytes the call is refused for, None) or (None, its results)."""
    try:
        return None, ctx.distance_noalloc(a, b, **kw)
    except sd3.SD3Error as e:
        assert e.name == "SD3_E_CAPACITY"
        need, limit = map(int, re.search(r"at least (\d+) bytes.* limit is (\d+)", str(e)).groups())
        assert limit == LIMIT
        return need, None


def test_calls_of_128_mib(ctx):
    import torch
    for n in range(400_000, 1_000_000, 50_000):
        a, b = (sd3.Batch.from_packed(synth.pack([synth.random_triangle_soup(
            n, s, scale=10.0, center=(30.0 * s, 0.0, 0.0), size=0.2)]), "cuda:0") for s in (0, 1))
        need, _ = _need(ctx, a, b)
        if need is not None:
            break
    # the rescue list (2^20 entries of 16 bytes) takes up the difference
    cap = (1 << 20) - -(-(need - LIMIT) // 16)
    assert cap > 0
    most = next(c for c in range(cap + 32, cap - 32, -1) if _need(ctx, a, b, rescue_cap=c)[0] is None)
    need, _ = _need(ctx, a, b, rescue_cap=most + 1)
    assert LIMIT < need <= LIMIT + 256
    _, (d, h) = _need(ctx, a, b, rescue_cap=most)
    e, f = ctx.distance(a, b)
    assert torch.equal(d, e) and torch.equal(h, f)
