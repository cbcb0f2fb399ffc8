"""The library's choice of method at k = 6 on graphs whose neighbourhoods
overlap: unclustered graphs are counted from the 4-sets, small worlds,
communities and cliques of the same sizes and degrees enumerated; both methods
count the same."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _oriented(n, pairs, rng):
    a = np.array(sorted(pairs))
    flip = rng.random(len(a)) < 0.5
    return I.csr_from_arcs(n, np.where(flip, a[:, 0], a[:, 1]), np.where(flip, a[:, 1], a[:, 0]))


def _ring(n, d, rng):
    """Every vertex joined with its d nearest on a ring."""
    return _oriented(n, {tuple(sorted((v, (v + j) % n))) for v in range(n)
                         for j in range(1, d // 2 + 1)}, rng)


def _communities(n, size, p, rng):
    return _oriented(n, {(c * size + j, c * size + i) for c in range(n // size)
                         for i in range(size) for j in range(i) if rng.random() < p}, rng)


def _er(n, d, rng):
    pairs = set()
    while len(pairs) < n * d // 2:
        u, v = map(int, rng.integers(n, size=2))
        if u != v:
            pairs.add((min(u, v), max(u, v)))
    return _oriented(n, pairs, rng)


CASES = {  # name: (graphs, method)
    "random": (lambda r: [_er(1200, 8, r)], M.METHOD_CORES),
    "powerlaw": (lambda r: [I.chung_lu_digraph(2600, 5200, 2.2, 60, 0.0, r)], M.METHOD_CORES),
    "ring": (lambda r: [_ring(1200, 8, r)], M.METHOD_ESU),
    "ring12": (lambda r: [_ring(1500, 12, r)], M.METHOD_ESU),
    "communities": (lambda r: [_communities(1200, 20, 0.45, r)], M.METHOD_ESU),
    "cliques": (lambda r: [_communities(1206, 9, 1.1, r)], M.METHOD_ESU),
    "powerlaw8": (lambda r: [I.chung_lu_digraph(1000, 2500, 2.2, 60, 0.0, r) for _ in range(8)],
                  M.METHOD_CORES),
    "rings8": (lambda r: [_ring(900, 8, r) for _ in range(8)], M.METHOD_ESU),
    # 47 of 1,200 vertices on a ring: 376 adjacency entries, no look at links
    "few_entries": (lambda r: [_padded(_ring(47, 8, r), 1200)], M.METHOD_CORES),
    "more_entries": (lambda r: [_padded(_ring(48, 8, r), 1200)], M.METHOD_ESU),
    "few_entries8": (lambda r: [_padded(_ring(47, 8, r), 900) for _ in range(8)], M.METHOD_CORES),
    "more_entries9": (lambda r: [_padded(_ring(47, 8, r), 900) for _ in range(9)], M.METHOD_ESU),
}


def _padded(spec, n):
    rp, col = spec
    return np.concatenate([rp, np.full(n - len(rp) + 1, rp[-1], rp.dtype)]), col


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("adjacency", [M.ADJ_BITS, M.ADJ_LISTS])
def test_choice(ctx, name, adjacency):
    make, method = CASES[name]
    specs = make(np.random.default_rng([91, 7]))
    t = ctx.table(6)
    gs = [ctx.load_graph(*s) for s in specs]
    try:
        hists = {}
        for m in (M.METHOD_AUTO, M.METHOD_ESU, M.METHOD_CORES):
            b = ctx.batch(gs, t, method=m, adjacency=adjacency)
            if m == M.METHOD_AUTO:
                assert b.stats()["method"] == method
            for _ in range(2):
                b.run()
                hists[m], totals = b.read()
            b.free()
        assert totals.all()
        assert np.array_equal(hists[M.METHOD_AUTO], hists[M.METHOD_ESU])
        assert np.array_equal(hists[M.METHOD_AUTO], hists[M.METHOD_CORES])
        if name in ("ring", "few_entries", "cliques"):
            assert_hist_equals_oracle(hists[M.METHOD_AUTO][0], t.class_codes(), *specs[0], 6)
    finally:
        for g in gs:
            g.free()


def test_one_graph_of_many_entries_sampled(ctx):
    """More than 65,536 entries: every second or third one is looked at."""
    r = np.random.default_rng(5)
    for spec, method in ((_er(8000, 10, r), M.METHOD_CORES), (_ring(8000, 12, r), M.METHOD_ESU)):
        g = ctx.load_graph(*spec)
        b = ctx.batch([g], ctx.table(6))
        assert b.stats()["method"] == method
        b.free()
        g.free()
