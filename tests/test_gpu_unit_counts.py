"""Plans for 2- and 3-sets, made without a sizing pass: the units a batch is
created with are the units its plan makes, on graphs with isolated vertices,
two-way arcs, device-made random versions and list-built adjacency."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _specs():
    rp, col = I.chung_lu_digraph(90, 200, 2.2, 30, 0.4, np.random.default_rng([81, 1]))
    far = np.concatenate([np.zeros(40, rp.dtype), rp, np.full(25, rp[-1], rp.dtype)])
    return [(rp, col), (far, (col + 40).astype(col.dtype)), I.empty_graph(7),
            I.complete_digraph(5), I.directed_path(2), I.out_star(70)]


@pytest.mark.parametrize("k,opts", [
    (3, {"method": M.METHOD_CORES}), (3, {"method": M.METHOD_ESU}),
    (4, {"method": M.METHOD_CORES}),
    (3, {"method": M.METHOD_ESU, "adjacency": M.ADJ_LISTS, "marks": M.MARKS_GLOBAL})])
def test_units(ctx, k, opts):
    t = ctx.table(k)
    gs = [ctx.load_graph(*s) for s in _specs()]
    gs += ctx.randomise(gs[1], 3, 5, 5)[0]
    for chosen in (gs, gs[2:3]):
        b = ctx.batch(chosen, t, **opts)
        try:
            before = b.stats()
            b.run()
            hist, _ = b.read()
            assert b.stats() == before
            for h, g in zip(hist, chosen):
                assert_hist_equals_oracle(h, t.class_codes(), *g.read(), k)
        finally:
            b.free()
    for g in gs:
        g.free()
