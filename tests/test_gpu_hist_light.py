"""Light launches count into the caller's histograms, heavy ones into the work
array: both sides of the rule on units a graph, into a buffer that is not
clear, and the memory each takes."""

import numpy as np
import pytest

from gpu_helpers import assert_hist_equals_oracle
from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu

WORK = {5: 8 << 16, 6: 47 * 8 << 15}  # bytes of a graph's work array, one copy


@pytest.mark.parametrize("method", [M.METHOD_ESU, M.METHOD_CORES])
@pytest.mark.parametrize("k,n,m,cap,ng,work", [
    (5, 40, 80, 10, 8, False), (5, 700, 1500, 25, 2, True),
    (6, 60, 130, 15, 3, False), (6, 700, 1500, 25, 2, True)])
def test_both_sides(ctx, k, n, m, cap, ng, work, method):
    import torch
    t = ctx.table(k)
    specs = [I.chung_lu_digraph(n, m, 2.2, cap, 0.2, np.random.default_rng([61, n, i]))
             for i in range(ng)]
    gs = [ctx.load_graph(*s) for s in specs]
    b = ctx.batch(gs, t, method=method)
    try:
        st = b.stats()
        assert (st["units"] >= WORK[k] * ng // (8 * (128 if k == 5 else 900))) == work
        rest = ng * t.num_classes * 8 + 16 * st["units"]
        slots = 2 * sum(len(s[1]) for s in specs)
        lists = 4 * 8192 * st["grid"] if method == M.METHOD_CORES else 0
        words = ng * 2 * n * ((n + 31) // 32)
        most = rest + 4 * words + 64 * slots + lists + (1 << 20)
        assert (M.mk_batch_bytes(b.handle) >= rest + ng * WORK[k]) == work or lists
        if not work:
            assert M.mk_batch_bytes(b.handle) < most
        for _ in range(2):
            d = torch.full((ng, t.num_classes), 5, dtype=torch.int64, device="cuda:0")
            torch.cuda.synchronize()  # the library's stream does not wait for torch's default one
            b.run(d, torch.cuda.current_stream())
            hist, totals = b.read()
            assert np.array_equal(hist, d.cpu().numpy().astype(np.uint64))
            assert np.array_equal(hist.sum(axis=1), totals)
        for i in (0, ng - 1):
            if n < 100 or k == 5:
                assert_hist_equals_oracle(hist[i], t.class_codes(), *specs[i], k)
    finally:
        b.free()
        for g in gs:
            g.free()
