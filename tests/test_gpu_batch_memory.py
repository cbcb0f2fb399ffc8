"""A batch short of device memory counts without the histograms' work array,
whether it is missing when the batch is made or when its own histograms are
(the first run without a caller's buffer), and fails only where what it needs
does not fit."""

import numpy as np
import pytest

from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,method", [(5, M.METHOD_ESU), (5, M.METHOD_CORES), (6, M.METHOD_ESU),
                                      (6, M.METHOD_CORES)])
@pytest.mark.parametrize("use_graph", [-1, 1, 2])
def test_work_array_goes_first(ctx, k, method, use_graph):
    import torch
    t = ctx.table(k)
    specs = [I.chung_lu_digraph(700, 1500, 2.2, 25, 0.2, np.random.default_rng([62, i]))
             for i in range(2)]
    gs = [ctx.load_graph(*s) for s in specs]
    stream = torch.cuda.current_stream()
    opts = dict(method=method, use_graph=use_graph)
    own = 8 * len(gs) * t.num_classes
    work = 8 * len(gs) * (1 << 16 if k == 5 else 47 << 15)  # one copy (of two at k = 5)
    try:
        b = ctx.batch(gs, t, **opts)
        full = M.mk_batch_bytes(b.handle)
        b.run()
        ref = b.read()[0]
        assert M.mk_batch_bytes(b.handle) == full
        b.free()
        for cap in (full - 1, full - own - 1):
            b = ctx.batch(gs, t, most_bytes=cap, **opts)
            d = torch.full((len(gs), t.num_classes), 3, dtype=torch.int64, device="cuda:0")
            torch.cuda.synchronize()  # the library's stream does not wait for torch's default one
            b.run(d, stream)
            assert np.array_equal(b.read()[0], ref)
            for _ in range(2):
                b.run()
                assert np.array_equal(b.read()[0], ref)
            least = M.mk_batch_bytes(b.handle)
            assert least <= full - work
            d.fill_(5)
            torch.cuda.synchronize()
            b.run(d, stream)
            assert np.array_equal(b.read()[0], ref)
            assert np.array_equal(d.cpu().numpy().astype(np.uint64), ref)
            b.free()
        # neither the work array nor the batch's own histograms fit
        b = ctx.batch(gs, t, most_bytes=least - own // 2, **opts)
        d = torch.full((len(gs), t.num_classes), 3, dtype=torch.int64, device="cuda:0")
        torch.cuda.synchronize()
        with pytest.raises(M.MotifsError) as e:
            b.run()
        assert e.value.status == M.MK_ENOMEM
        b.run(d, stream)
        assert np.array_equal(b.read()[0], ref)
        b.free()
        with pytest.raises(M.MotifsError) as e:
            ctx.batch(gs, t, most_bytes=10000, **opts)
        assert e.value.status == M.MK_ENOMEM
    finally:
        for g in gs:
            g.free()
