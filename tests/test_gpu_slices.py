"""Costly children cut into slices of their own children: a hub and a few
cross arcs, relabelled so that the hub comes first, last and between, at
sizes on both sides of the least slice and with hundreds of slices a child,
by every kernel that takes slices, against the oracle."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from oracle import oracle as O
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _hubs(leaves, hub_at, seed=0):
    """A vertex with `leaves` neighbours, a second hub with a third of them,
    and `leaves` / 4 arcs more; the first hub has label hub_at."""
    rng = np.random.default_rng([71, leaves, seed])
    arcs = {(0, v) if v % 3 else (v, 0) for v in range(1, leaves + 1)}
    arcs |= {(v, 1) for v in range(2, leaves // 3 + 2)}
    while len(arcs) < leaves + leaves // 3 + leaves // 4:
        u, v = map(int, rng.choice(leaves + 1, 2, replace=False))
        arcs.add((u, v))
    src, dst = np.array(sorted(arcs)).T
    perm = np.arange(leaves + 1)
    perm[[0, hub_at]] = perm[[hub_at, 0]]
    return I.relabel(*I.csr_from_arcs(leaves + 1, src, dst), perm)


# leaves: below and above the first sliced child, and far above (k, method,
# adjacency); a split threshold of 1 leaves the slices to their least cost
@pytest.mark.parametrize("k,method,lists,sizes", [
    (5, M.METHOD_ESU, False, (80, 100, 120)), (5, M.METHOD_ESU, True, (100,)),
    (6, M.METHOD_ESU, False, (26, 34, 45)), (6, M.METHOD_ESU, True, (34,)),
    (6, M.METHOD_CORES, False, (28, 36, 45))])
@pytest.mark.parametrize("threshold", [0, 1])
def test_dense_histograms(ctx, k, method, lists, sizes, threshold):
    t = ctx.table(k)
    specs = [_hubs(n, at) for n in sizes for at in (0, n // 2, n)]
    gs = [ctx.load_graph(*s) for s in specs]
    opts = {"adjacency": M.ADJ_LISTS, "marks": M.MARKS_GLOBAL} if lists else {}
    b = ctx.batch(gs, t, method=method, split_threshold=threshold, **opts)
    try:
        for _ in range(2):
            b.run()
            hist, _ = b.read()
            for h, s in zip(hist, specs):
                assert_hist_equals_oracle(h, t.class_codes(), *s, k)
    finally:
        b.free()
        for g in gs:
            g.free()


@pytest.mark.parametrize("leaves", [24, 30, 36])
def test_k7(ctx, leaves):
    specs = [_hubs(leaves, at) for at in (0, leaves // 2, leaves)]
    gs = [ctx.load_graph(*s) for s in specs]
    out, totals, _ = ctx.count7(gs)
    for got, total, s in zip(out, totals, specs):
        exp = O.count(*s, 7)
        assert dict(zip(map(int, got[0]), map(int, got[1]))) == exp
        assert int(total) == sum(exp.values())
    for g in gs:
        g.free()
