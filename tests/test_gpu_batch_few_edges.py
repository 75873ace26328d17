"""GPU parity of wc_sssp_batch for instances of fewer than four edges at the wave
and block levels, whose children load four edges at once: their buffered items
take the grid-wide child, whose loads stay inside the arrays.  Against the
oracle, exactly; the arrays lie at every element of an allocation."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev_to_u32, say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["wave", "block"])
@pytest.mark.parametrize("m", [2, 3])
def test_few_edges(ctx, mode, m):
    n = 300  # two instances: their sources lie in windows of different workgroups
    rng = np.random.default_rng(m)
    ptr = np.full(n + 1, m, dtype=np.int32)
    ptr[0] = 0
    tune = wc.make_tune(threshold=m - 1, block_threads=64)
    for off in range(4):
        graphs, weights, refs = [], [], []
        for _ in range(2):
            col, w = rng.integers(1, 5, m).astype(np.int32), rng.integers(1, 100, m, dtype=np.uint32)
            dc = torch.zeros(m + 8, dtype=torch.int32, device="cuda")
            dw = torch.zeros_like(dc)
            dc[off:off + m] = torch.from_numpy(col).cuda()
            dw[off:off + m] = u32_to_dev(w)
            graphs.append(wc.DeviceCSR(n, torch.from_numpy(ptr).cuda(), dc[off:off + m]))
            weights.append(dw[off:off + m])
            refs.append(oracle.sssp_dijkstra(ptr, col, w, 0))
        say(f"batch of few edges: mode={mode} m={m} element {off}")
        outs, st = ctx.sssp_batch(graphs, weights, [0, 0], modes=[mode] * 2, tunes=[tune] * 2, stats=True)
        torch.cuda.synchronize()
        for o, r in zip(outs, refs):
            assert np.array_equal(dev_to_u32(o), r), (mode, m, off)
        # both items in the one grid-wide child, none in a wave's or a workgroup's own
        assert (st["items_buffered"], st["dispatches"], st["edges_buffered"]) == (2, 1, 2 * m)
