"""The kernels that prepare a pass, at the edges of their tiles: bit rows of
one word, of a wave of words and of more; adjacency slots around a workgroup's
64; hubs whose child ranges cross the teams' 16 lanes; batches around the
windows of 512 workgroups and past the 14,336 that plan without a scan; and a
destination that is 8-byte aligned only."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


def _check(ctx, specs, k, look, **opts):
    """Two passes of a batch into a buffer one bin past its start."""
    import torch
    t = ctx.table(k)
    gs = [ctx.load_graph(*s) for s in specs]
    b = ctx.batch(gs, t, **opts)
    try:
        flat = torch.full((len(specs) * t.num_classes + 2,), 7, dtype=torch.int64, device="cuda:0")
        d = flat[1:-1].view(len(specs), t.num_classes)
        for _ in range(2):
            b.run(d, torch.cuda.current_stream())
            hist, totals = b.read()
            assert np.array_equal(hist, d.cpu().numpy().astype(np.uint64))
            assert np.array_equal(hist.sum(axis=1), totals)
        assert flat[0].item() == 7 and flat[-1].item() == 7
        for i in look:
            assert_hist_equals_oracle(hist[i], t.class_codes(), *specs[i], k)
        return hist
    finally:
        b.free()
        for g in gs:
            g.free()


# words of a row 1, 2, 16, 17, 64, 65, 256
@pytest.mark.parametrize("n", [2, 31, 32, 33, 512, 513, 2048, 2049, 8192])
@pytest.mark.parametrize("k", [3, 4])
def test_rows(ctx, n, k):
    rng = np.random.default_rng([51, n])
    if n == 2:
        spec = I.complete_digraph(2)
    else:
        spec = I.chung_lu_digraph(n, 2 * n, 2.2, 25, 0.2, rng)
    _check(ctx, [spec], k, [0])


# a ring of n vertices has 2 n slots, of which n are nodes
@pytest.mark.parametrize("n", [31, 32, 33, 64, 128, 257])
@pytest.mark.parametrize("k", [3, 5])
def test_slots(ctx, n, k):
    _check(ctx, [I.directed_cycle(n), I.bidirected_cycle(n)], k, [0, 1])


# a hub with `leaves` children on both sides of a team's 16 and of a wave,
# whole and in ranges down to single children
@pytest.mark.parametrize("leaves", [15, 16, 17, 18, 65])
@pytest.mark.parametrize("k", [4, 5])
@pytest.mark.parametrize("threshold", [1, 40, 1 << 30])
def test_ranges(ctx, leaves, k, threshold):
    rng = np.random.default_rng([52, leaves])
    hub = [(0, v) for v in range(1, leaves + 1)]
    more = [tuple(map(int, rng.choice(leaves + 1, 2, replace=False))) for _ in range(leaves)]
    src, dst = np.array(sorted(set(hub + more))).T
    spec = I.csr_from_arcs(leaves + 1, src, dst)
    _check(ctx, [spec, I.relabel(*spec, np.arange(leaves, -1, -1))], k, [0, 1],
           split_threshold=threshold)


# 2 workgroups a graph (33 vertices on a ring), or 1
@pytest.mark.parametrize("ring,ng", [(33, 255), (33, 256), (33, 257), (33, 600), (5, 14336),
                                     (5, 14337)])
def test_windows(ctx, ring, ng):
    specs = [I.directed_cycle(ring) if i % 3 else I.bidirected_cycle(ring - i % 2)
             for i in range(ng)]
    hist = _check(ctx, specs, 4, [0, 1, 2, 3, ng - 2, ng - 1])
    for i in range(6, ng):  # the six kinds repeat
        assert np.array_equal(hist[i], hist[i % 6])
