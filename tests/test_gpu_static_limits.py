"""mk_count_static where its scratch gets tight: the largest graph of 4,096
vertices it takes at k = 3 (counted in place) and one a little larger, disjoint
cliques on both sides of the size at which the slices of costly children no
longer fit beside the histogram's work array, and hubs whose children are cut into slices, all into a destination
that is not clear."""

import math

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _static(ctx, g, t):
    import torch
    d = torch.full((t.num_classes,), 7, dtype=torch.int64, device="cuda:0")
    torch.cuda.synchronize()  # the library's stream does not wait for torch's default one
    ctx.count_static(g, t, d, torch.cuda.current_stream())
    return d.cpu().numpy().astype(np.uint64)


def _pairs(n, count, rng):
    """A digraph of n vertices and `count` adjacent pairs."""
    code = rng.choice(n * (n - 1) // 2, size=count, replace=False)
    v = ((1 + np.sqrt(1 + 8.0 * code)) / 2).astype(np.int64)
    v -= v * (v - 1) // 2 > code
    v += v * (v + 1) // 2 <= code
    u = code - v * (v - 1) // 2
    flip = rng.random(count) < 0.5
    return I.csr_from_arcs(n, np.where(flip, u, v), np.where(flip, v, u))


# 32 bytes an adjacency entry (lists, planner slots, half a unit) beside 4 MiB
# of bit matrices
@pytest.mark.parametrize("pairs,fits", [(982720, True), (982800, False)])
def test_last_graph_that_fits(ctx, pairs, fits):
    t = ctx.table(3)
    g = ctx.load_graph(*_pairs(4096, pairs, np.random.default_rng(67)))
    try:
        if fits:
            assert np.array_equal(_static(ctx, g, t), ctx.count(g, t)[0])
        else:
            with pytest.raises(M.MotifsError) as e:
                _static(ctx, g, t)
            assert e.value.status == M.MK_ERANGE
    finally:
        g.free()


@pytest.mark.parametrize("size", [99, 147, 160])
def test_cliques(ctx, size):
    """8,192 vertices in cliques: 0.8 to 1.3 million adjacency entries."""
    c = M.MK_LDS_MARKS_MAX_VERTICES // size
    v, u = np.tril_indices(size, -1)
    at = np.repeat(np.arange(c) * size, len(u))
    flip = np.random.default_rng([68, size]).random(len(at)) < 0.5
    u, v = np.tile(u, c) + at, np.tile(v, c) + at
    spec = I.csr_from_arcs(M.MK_LDS_MARKS_MAX_VERTICES, np.where(flip, u, v), np.where(flip, v, u))
    g = ctx.load_graph(*spec)
    try:
        for k in (4, 5):
            t = ctx.table(k)
            got = _static(ctx, g, t)
            assert int(got.sum()) == c * math.comb(size, k)
            assert np.array_equal(got, ctx.count(g, t)[0])
    finally:
        g.free()


@pytest.mark.parametrize("k,leaves", [(5, 80), (5, 120), (6, 26), (6, 45)])
def test_hubs(ctx, k, leaves):
    rng = np.random.default_rng([69, leaves])
    arcs = {(0, v) if v % 3 else (v, 0) for v in range(1, leaves + 1)}
    arcs |= {(v, 1) for v in range(2, leaves // 3 + 2)}
    while len(arcs) < leaves + leaves // 2:
        arcs.add(tuple(map(int, rng.choice(leaves + 1, 2, replace=False))))
    src, dst = np.array(sorted(arcs)).T
    t = ctx.table(k)
    for perm in (np.arange(leaves + 1), np.arange(leaves, -1, -1)):
        spec = I.relabel(*I.csr_from_arcs(leaves + 1, src, dst), perm)
        g = ctx.load_graph(*spec)
        try:
            assert_hist_equals_oracle(_static(ctx, g, t), t.class_codes(), *spec, k)
        finally:
            g.free()
