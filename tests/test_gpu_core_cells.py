"""The counting from (k-2)-sets around its table sizes: cores with fewer,
exactly as many and more cells than the arc-pair table holds (15, 16 at
k = 6), up to hundreds, and lists at and past one wave's 64 entries."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _hist(ctx, spec, k, method):
    t = ctx.table(k)
    g = ctx.load_graph(*spec)
    b = ctx.batch([g], t, method=method)
    try:
        b.run()
        return b.read()[0][0], t.class_codes()
    finally:
        b.free()
        g.free()


# dense digraphs: n - k + 2 vertices around every core, nearly all of
# different relation
@pytest.mark.parametrize("k,n", [(5, 17), (5, 18), (5, 19), (5, 26), (6, 19), (6, 20), (6, 21),
                                 (6, 23)])
def test_many_cells_equal_oracle(ctx, k, n):
    spec = I.er_digraph(n, n * (n - 1) * 2 // 5, np.random.default_rng([31, k, n]))
    hist, cc = _hist(ctx, spec, k, M.METHOD_CORES)
    assert_hist_equals_oracle(hist, cc, *spec, k)


@pytest.mark.parametrize("k,n,m", [(3, 300, 9000), (4, 130, 5000), (5, 90, 2500), (6, 66, 1300)])
def test_hundreds_of_cells_equal_esu(ctx, k, n, m):
    spec = I.er_digraph(n, m, np.random.default_rng([32, k]))
    a, _ = _hist(ctx, spec, k, M.METHOD_CORES)
    b, _ = _hist(ctx, spec, k, M.METHOD_ESU)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("k", [4, 5, 6])
@pytest.mark.parametrize("leaves", [62, 63, 64, 65])
def test_list_of_a_wave(ctx, k, leaves):
    """Hub lists of 63 to 66 entries: the wave's held list and the long one."""
    src = [0] * leaves + [1, leaves + 1]
    dst = list(range(1, leaves + 1)) + [0, 1]
    spec = I.csr_from_arcs(leaves + 2, src, dst)
    if k == 6:
        a, _ = _hist(ctx, spec, k, M.METHOD_CORES)
        b, _ = _hist(ctx, spec, k, M.METHOD_ESU)
        assert np.array_equal(a, b)
    else:
        hist, cc = _hist(ctx, spec, k, M.METHOD_CORES)
        assert_hist_equals_oracle(hist, cc, *spec, k)
