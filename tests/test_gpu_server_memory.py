"""The server's budget: finished batches give their memory back before a group
has to do with less, arc lists are charged once a group, and what is charged
stays within the budget."""

import numpy as np
import pytest

from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _serve(ctx, specs, ks, budget):
    """(groups, short groups, peak bytes) after serving everything at once;
    every histogram equals the same request's alone."""
    tables = {k: ctx.table(k) for k in set(ks)}
    gs = [ctx.load_graph(*s) for s in specs]
    alone = [ctx.count(g, tables[k])[0] for g, k in zip(gs, ks)]
    srv = ctx.server(hbm_budget_bytes=budget)
    try:
        tickets = [srv.submit(g, k) for g, k in zip(gs, ks)]
        for tk, k, ref in zip(tickets, ks, alone):
            assert np.array_equal(srv.wait(tk, k)[0], ref)
        return M.mk_server_counts(srv.handle)
    finally:
        srv.stop()
        for g in gs:
            g.free()


def test_finished_batches_make_room(ctx):
    """A long request stays in flight while others finish, whose memory
    together is several times the budget; each can use all it needs."""
    rng = np.random.default_rng(64)
    specs = [I.chung_lu_digraph(5000, 22000, 2.3, 60, 0.0, rng)]
    specs += [I.chung_lu_digraph(1300 + 40 * i, 3000, 2.2, 60, 0.0, rng) for i in range(40)]
    groups, short, peak = _serve(ctx, specs, [6] * len(specs), 2048 * MIB)
    assert groups >= 2 and short == 0
    assert peak <= 2048 * MIB


@pytest.mark.parametrize("budget", [320 * MIB, 128 * MIB])
def test_arc_lists_once_a_group(ctx, budget):
    """32 requests whose arc lists alone would fill the budget five at a time."""
    rng = np.random.default_rng(65)
    specs = [I.chung_lu_digraph(2000, 6000, 2.1, 150, 0.1, rng) for _ in range(32)]
    groups, _, peak = _serve(ctx, specs, [5] * 32, budget)
    assert groups <= (6 if budget > 200 * MIB else 20)
    assert peak <= budget


@pytest.mark.parametrize("budget_mib", [96, 24])
def test_short_groups_count_the_same(ctx, budget_mib):
    rng = np.random.default_rng(66)
    ks = [3, 4, 5, 6] * 5
    specs = [I.chung_lu_digraph(int(rng.integers(100, 900)), 900, 2.2, 15, 0.1, rng) for _ in ks]
    _, _, peak = _serve(ctx, specs, ks, budget_mib * MIB)
    assert peak <= budget_mib * MIB


@pytest.mark.parametrize("k", [4, 5, 6])
def test_budget_of_one_request(ctx, k):
    """A budget of what the request's arrays take, without rounding, is enough;
    one of half of it is refused."""
    rng = np.random.default_rng([67, k])
    spec = I.chung_lu_digraph(500, 1200, 2.2, 15, 0.1, rng)
    g = ctx.load_graph(*spec)
    least = M.mk_graph_least_footprint(g.handle, k)
    g.free()
    _serve(ctx, [spec, spec], [k, k], least - 4096)
    with pytest.raises(M.MotifsError) as e:
        _serve(ctx, [spec], [k], least // 2)
    assert e.value.status == M.MK_EBUSY
