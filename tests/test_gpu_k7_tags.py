"""k = 7 around the 63 extension vertices that the marks' tags hold (more are
counted pair by pair): stars of 60 to 72 leaves with the hub first, last and in
the middle, out, mixed, and with arcs between leaves, against closed forms."""

import math

import numpy as np
import pytest

from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _specs(leaves):
    """(arcs, counts of the classes, ascending) on vertices 0 (hub) .. leaves."""
    out = [(0, v) for v in range(1, leaves + 1)]
    total = math.comb(leaves, 6)
    yield out, [total]
    # a third of the leaves point at the hub
    a = leaves // 3
    mixed = [(v, 0) for v in range(1, a + 1)] + out[a:]
    yield mixed, sorted(math.comb(a, i) * math.comb(leaves - a, 6 - i) for i in range(7))
    # one arc between two leaves; two arcs in a two-way pair
    linked = math.comb(leaves - 2, 4)
    yield out + [(leaves, 1)], sorted([linked, total - linked])
    yield out + [(2, leaves - 1), (leaves - 1, 2)], sorted([linked, total - linked])


@pytest.mark.parametrize("leaves", [60, 63, 64, 65, 66, 67, 68, 69, 70, 72])
def test_stars(ctx, leaves):
    n = leaves + 1
    for arcs, counts in _specs(leaves):
        src, dst = np.array(arcs).T
        specs = []
        for at in (0, leaves // 2, leaves):
            perm = np.arange(n)
            perm[[0, at]] = perm[[at, 0]]
            specs.append(I.relabel(*I.csr_from_arcs(n, src, dst), perm))
        gs = [ctx.load_graph(*s) for s in specs]
        try:
            out, totals, _ = ctx.count7(gs)
        finally:
            for g in gs:
                g.free()
        for (codes, got), total in zip(out, totals):
            assert sorted(int(c) for c in got) == counts
            assert int(total) == sum(counts) == math.comb(leaves, 6)
            assert np.array_equal(codes, out[0][0]) and np.array_equal(got, out[0][1])
        if len(counts) == 1:
            assert [int(c) for c in out[0][0]] == [2**6 - 1]


def test_past_lds_marks(ctx):
    """The same with marks in device memory: the star beside isolated vertices."""
    leaves = 66
    arcs, counts = list(_specs(leaves))[1]
    src, dst = np.array(arcs).T
    g = ctx.load_graph(*I.csr_from_arcs(M.MK_LDS_MARKS_MAX_VERTICES + 10, src, dst))
    try:
        out, totals, _ = ctx.count7([g])
    finally:
        g.free()
    assert sorted(int(c) for c in out[0][1]) == counts
    assert int(totals[0]) == math.comb(leaves, 6)
