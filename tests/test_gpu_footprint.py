"""What a count takes of device memory: mk_graph_footprint covers a one-graph
batch (its units as planned), and a batch kept to a limit keeps to it, with
fewer units, shorter arc lists, no work array and, at k = 6, the 4-sets where
their lists fit, and counts the same."""

import numpy as np
import pytest

from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _hubs(leaves, rng):
    """A hub, a second one with a third of its neighbours, and arcs across."""
    arcs = {(0, v) if v % 3 else (v, 0) for v in range(1, leaves + 1)}
    arcs |= {(v, 1) for v in range(2, leaves // 3 + 2)}
    while len(arcs) < 2 * leaves:
        arcs.add(tuple(map(int, rng.choice(leaves + 1, 2, replace=False))))
    src, dst = np.array(sorted(arcs)).T
    return I.csr_from_arcs(leaves + 1, src, dst)


def _specs():
    rng = np.random.default_rng(63)
    return {"path": I.directed_path(3000), "star": I.out_star(150), "hubs": _hubs(60, rng),
            "hubs2": _hubs(110, rng), "dense": I.er_digraph(50, 900, rng),
            "powerlaw": I.chung_lu_digraph(700, 1500, 2.2, 25, 0.2, rng),
            "powerlaw2": I.chung_lu_digraph(2600, 5200, 2.2, 60, 0.0, rng),
            "empty": I.empty_graph(20), "big": I.er_digraph(9000, 9000, rng)}


SPECS = _specs()


def _nnz(spec):
    src, dst = I.arcs_from_csr(*spec)
    n = len(spec[0])
    return 2 * len(np.unique(np.minimum(src, dst) * n + np.maximum(src, dst)))


@pytest.mark.parametrize("k", [3, 4, 5, 6])
@pytest.mark.parametrize("name", sorted(SPECS))
def test_footprint_and_least(ctx, k, name):
    t = ctx.table(k)
    g = ctx.load_graph(*SPECS[name])
    try:
        b = ctx.batch([g], t)
        b.run()
        ref, totals = b.read()
        over = 16 * max(0, b.stats()["units"] - 4 * _nnz(SPECS[name]))
        assert M.mk_batch_bytes(b.handle) <= g.footprint(k) + over
        b.free()
        least = M.mk_graph_least_footprint(g.handle, k)
        assert least <= g.footprint(k)
        for limit in (least, (least + g.footprint(k)) // 2):
            for method in (M.METHOD_AUTO, M.METHOD_ESU):
                b = ctx.batch([g], t, limit=limit, method=method)
                assert M.mk_batch_bytes(b.handle) <= limit
                b.run()
                hist, tot = b.read()
                assert np.array_equal(hist, ref) and np.array_equal(tot, totals)
                b.free()
        # a limit below the least: the same memory as at the least
        b = ctx.batch([g], t, limit=1)
        b.run()
        assert np.array_equal(b.read()[0], ref)
        assert M.mk_batch_bytes(b.handle) <= least
        b.free()
    finally:
        g.free()


@pytest.mark.parametrize("k", [4, 5, 6])
@pytest.mark.parametrize("lists", [False, True])
def test_batch_within_sum(ctx, k, lists):
    t = ctx.table(k)
    names = ("path", "hubs", "star", "hubs2", "dense", "empty", "powerlaw")
    gs = [ctx.load_graph(*SPECS[n]) for n in names]
    opts = dict(adjacency=M.ADJ_LISTS, method=M.METHOD_ESU) if lists else {}
    try:
        b = ctx.batch(gs, t, **opts)
        b.run()
        ref = b.read()[0]
        b.free()
        limit = sum(M.mk_graph_least_footprint(g.handle, k) for g in gs)
        b = ctx.batch(gs, t, limit=limit, **opts)
        assert M.mk_batch_bytes(b.handle) <= limit + 65536
        for _ in range(2):
            b.run()
            assert np.array_equal(b.read()[0], ref)
        b.free()
    finally:
        for g in gs:
            g.free()


def test_k6_keeps_the_cores_while_their_lists_fit(ctx):
    t = ctx.table(6)
    g = ctx.load_graph(*SPECS["powerlaw2"])
    try:
        least, full = M.mk_graph_least_footprint(g.handle, 6), g.footprint(6)
        work = 8 * (47 << 15)
        assert full > least + work
        seen = []
        hists = []
        for limit in (least, full - work, full):
            b = ctx.batch([g], t, limit=limit)
            seen.append(b.stats()["method"])
            assert M.mk_batch_bytes(b.handle) <= limit
            b.run()
            hists.append(b.read()[0])
            b.free()
        assert seen == [M.METHOD_ESU, M.METHOD_CORES, M.METHOD_CORES]
        assert np.array_equal(hists[0], hists[1]) and np.array_equal(hists[0], hists[2])
    finally:
        g.free()
