"""The core kernel's lists of a parent's arc pairs are no longer than the
graphs can need: their memory (which a blocking count allocates and frees) at
small degrees, and the counts at k = 5 and 6 where a parent's arc pairs come
near the bound, far below it, and past the longest list."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _batch(ctx, specs, k, **opts):
    gs = [ctx.load_graph(*s) for s in specs]
    return gs, ctx.batch(gs, ctx.table(k), method=M.METHOD_CORES, **opts)


@pytest.mark.parametrize("specs", [
    [I.directed_path(5000)],
    [I.er_digraph(3000, 4500, np.random.default_rng(5))],
    [I.chung_lu_digraph(100, 200, 2.2, 15, 0.2, np.random.default_rng([9, i])) for i in range(40)]])
def test_bytes_at_small_degrees(ctx, specs):
    gs, b = _batch(ctx, specs, 5)
    try:
        st = b.stats()
        words = sum(2 * (len(rp) - 1) * ((len(rp) + 30) // 32) for rp, _ in specs)
        nnz = 2 * sum(len(col) for _, col in specs)
        rest = 4 * words + 64 * nnz + 16 * st["units"] + 9364 * 8 * len(specs) + 32 * 2**20 // 8
        # a list a wave, of 2,048 arc pairs at the most, here under a tenth of them
        assert M.mk_batch_bytes(b.handle) < rest + st["grid"] * 4 * 205 + len(specs) * 2**19
    finally:
        b.free()
        for g in gs:
            g.free()


@pytest.mark.parametrize("k", [5, 6])
@pytest.mark.parametrize("spec", [
    I.complete_digraph(14), I.complete_digraph(3), I.directed_path(40), I.out_star(40),
    I.er_digraph(60, 700, np.random.default_rng(3))], ids=["K14", "K3", "path", "star", "dense"])
def test_counts(ctx, k, spec):
    gs, b = _batch(ctx, [spec, I.directed_cycle(9)], k)
    try:
        for _ in range(2):
            b.run()
            hist, _ = b.read()
        if spec[1].size < 700 or k == 5:
            assert_hist_equals_oracle(hist[0], ctx.table(k).class_codes(), *spec, k)
        assert_hist_equals_oracle(hist[1], ctx.table(k).class_codes(), *I.directed_cycle(9), k)
    finally:
        b.free()
        for g in gs:
            g.free()


def test_parents_past_the_longest_list(ctx):
    """A bidirected hub over a dense graph: adj(P) holds about 20,000 arc pairs."""
    rng = np.random.default_rng(11)
    n = 320
    rp, col = I.er_digraph(n, 42000, rng)
    src, dst = I.arcs_from_csr(rp, col)
    spec = I.csr_from_arcs(n + 2, np.concatenate([src, np.full(n, n), [n + 1]]),
                           np.concatenate([dst, np.arange(n), [n]]))
    gs, b = _batch(ctx, [spec], 5)
    e = ctx.batch(gs, ctx.table(5), method=M.METHOD_ESU)
    try:
        b.run()
        e.run()
        assert np.array_equal(b.read()[0], e.read()[0])
    finally:
        b.free()
        e.free()
        gs[0].free()
