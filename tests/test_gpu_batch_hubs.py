"""GPU parity of wc_sssp_batch with vertices of very many chunks, which their wave
writes, beside vertices whose lane writes a few (up to four) in the same
workgroup; several of both in a wave, at every level, without and with captured
rounds; against the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev_to_u32, say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


def star(n):
    return synth.symmetrize(synth.graph_from_edges(n, [(0, i) for i in range(1, n)])[0])


def of_degrees(deg, seed):
    ptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    return synth.CSR(len(deg), ptr, np.random.default_rng(seed).integers(0, len(deg), int(ptr[-1])).astype(np.int32))


def joined(n, hubs, seed):
    """`hubs` vertices joined with all, both ways."""
    h = np.random.default_rng(seed).choice(n, hubs, replace=False)
    e = np.stack([np.repeat(h, n), np.tile(np.arange(n), hubs)], 1)
    e = np.concatenate([e, e[:, ::-1]])
    e = e[np.lexsort((e[:, 1], e[:, 0]))]
    ptr = np.concatenate([[0], np.cumsum(np.bincount(e[:, 0], minlength=n))]).astype(np.int32)
    return synth.CSR(n, ptr, e[:, 1].astype(np.int32))


@pytest.mark.parametrize("mode", ["grid", "wave", "block", "mixed"])
def test_long_rows(ctx, mode):
    rng = np.random.default_rng(1)
    long = [255, 256, 257, 319, 320, 321, 511, 512, 513, 639, 640, 641, 5000, 1, 40000, 9, 64]
    gs = [star(50000), of_degrees(rng.permutation(long * 4), 2), of_degrees(rng.permutation(long + [3] * 500), 3),
          joined(3000, 5, 4), joined(20011, 4, 5), star(9)]
    ws = [rng.integers(1, 1 << (4 + 3 * k), g.m, dtype=np.uint32) for k, g in enumerate(gs)]
    srcs = [int(np.argmax(g.degrees())) for g in gs]
    refs = [oracle.sssp_dijkstra(g.row_ptr, g.col, w, s) for g, w, s in zip(gs, ws, srcs)]
    dgs, dws = [wc.DeviceCSR.from_host(g.row_ptr, g.col) for g in gs], [u32_to_dev(w) for w in ws]
    modes = [["grid", "wave", "block", "flat"][i % 4] if mode == "mixed" else mode for i in range(len(gs))]
    for block, items in ((256, 1), (64, 2), (1024, 1)):
        for rounds in (0, 12):
            say(f"batch of long rows: mode={mode} block={block} items={items} graph_rounds={rounds}")
            tunes = [wc.make_tune(block_threads=block, items_per_lane=items)] * len(gs)
            outs = ctx.sssp_batch(dgs, dws, srcs, modes=modes, tunes=tunes, graph_rounds=rounds)
            torch.cuda.synchronize()
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert np.array_equal(dev_to_u32(o), r), (i, mode, block, rounds)
