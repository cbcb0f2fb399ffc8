"""The library's choice of method at k = 6 on both sides of its rule (the
degrees of the batch, its vertex count, and the number of graphs), on loaded
and on device-made graphs, against the oracle."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _q(row_ptr, col):
    """sum d^2 / sum d over the undirected degrees d."""
    src, dst = I.arcs_from_csr(row_ptr, col)
    n = len(row_ptr) - 1
    key = np.unique(np.minimum(src, dst) * n + np.maximum(src, dst))
    d = np.bincount(np.concatenate([key // n, key % n]), minlength=n)
    return float((d ** 2).sum()) / d.sum()


def _union(spec, n):
    """spec and isolated vertices up to n in all."""
    rp, col = spec
    return np.concatenate([rp, np.full(n - len(rp) + 1, rp[-1], rp.dtype)]), col


# a hub-heavy core graph padded with isolated vertices past the rule's n
@pytest.mark.parametrize("pad,randoms,method", [
    (0, 0, M.METHOD_ESU), (1199, 0, M.METHOD_ESU), (1200, 0, M.METHOD_CORES),
    (900, 6, M.METHOD_ESU), (900, 7, M.METHOD_CORES), (899, 7, M.METHOD_ESU),
    (0, 15, M.METHOD_ESU), (8192, 0, M.METHOD_CORES), (8193, 0, M.METHOD_ESU)])
def test_choice_and_counts(ctx, pad, randoms, method):
    spec = I.chung_lu_digraph(80, 190, 2.1, 40, 0.2, np.random.default_rng([61, 3]))
    q = _q(*spec)
    assert 7.5 < q
    if pad:
        spec = _union(spec, pad)
    t = ctx.table(6)
    cc = t.class_codes()
    g = ctx.load_graph(*spec)
    gs = [g] + (ctx.randomise(g, randoms, 5, 3)[0] if randoms else [])
    b = ctx.batch(gs, t)
    try:
        assert b.stats()["method"] == method
        b.run()
        hist, _ = b.read()
        for i in (0, randoms):
            assert_hist_equals_oracle(hist[i], cc, *gs[i].read(), 6)
    finally:
        b.free()
        for h in gs:
            h.free()


def test_light_graphs_enumerate(ctx):
    spec = _union(I.er_digraph(300, 500, np.random.default_rng(8)), 1200)
    assert _q(*spec) < 7.5
    t = ctx.table(6)
    gs = [ctx.load_graph(*spec) for _ in range(8)]
    try:
        for ng in (1, 8):
            b = ctx.batch(gs[:ng], t)
            assert b.stats()["method"] == M.METHOD_ESU
            b.free()
    finally:
        for g in gs:
            g.free()
