"""GPU parity of wc_sssp_batch at the edges of its kernels: degrees on both sides
of the inline, short, long and chunk limits (8, 32 and 128 edges), rows at every
alignment, instances of fewer than four edges, windows that end inside an
instance, more than 256 rounds (the frontier marks keep eight bits of the round),
distances over all octaves of the byte that bounds them; every level and mixtures,
with and without captured rounds; against the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev_to_u32, say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
MODES = ["flat", "wave", "block", "grid"]


def of_degrees(deg, seed):
    ptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    return synth.CSR(len(deg), ptr,
                     np.random.default_rng(seed).integers(0, len(deg), int(ptr[-1])).astype(np.int32))


def chain(n):
    return synth.CSR(n, np.minimum(np.arange(n + 1), n - 1).astype(np.int32), np.arange(1, n, dtype=np.int32))


@pytest.fixture(scope="module")
def batch():
    rng = np.random.default_rng(11)
    edge = [0, 1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1500]
    gs = [of_degrees([off] + edge + [2] * 30, off) for off in range(4)]
    gs += [of_degrees(rng.permutation(edge * 60), 4), of_degrees([33] * 1023, 5), of_degrees([9] * 4097, 6)]
    gs += [of_degrees([k], 7 + k) for k in range(5)] + [of_degrees([3, 0], 12), of_degrees([1, 1, 1], 13), chain(700)]
    gs += [synth.rmat_csr(13, 1 << 17, seed=3), of_degrees([40] * 255, 14)]
    ws = []
    for k, g in enumerate(gs):
        top = (16, 1000, 1 << 20, 1 << 30)[k % 4] if g.n != 700 else 100
        ws.append(rng.integers(1, top, g.m, dtype=np.uint32) >> rng.integers(0, 20 if top > 1000 else 1, g.m).astype(np.uint32) | np.uint32(1))
    srcs = [int(np.argmax(g.degrees() > 0)) for g in gs]
    refs = [oracle.sssp_dijkstra(g.row_ptr, g.col, w, s) for g, w, s in zip(gs, ws, srcs)]
    return [wc.DeviceCSR.from_host(g.row_ptr, g.col) for g in gs], [u32_to_dev(w) for w in ws], srcs, refs


@pytest.mark.parametrize("mode", MODES + ["mixed"])
@pytest.mark.parametrize("block", [64, 256, 1024])
def test_levels(ctx, batch, mode, block):
    graphs, weights, srcs, refs = batch
    k = len(graphs)
    modes = [MODES[i % 4] if mode == "mixed" else mode for i in range(k)]
    for rounds, items in ((0, 2), (20, 1)):
        say(f"batch paths mode={mode} block={block} graph_rounds={rounds} items={items}")
        tunes = [wc.make_tune(block_threads=block, items_per_lane=items, threshold=2 if items == 1 else 8)] * k
        outs = ctx.sssp_batch(graphs, weights, srcs, modes=modes, tunes=tunes, graph_rounds=rounds)
        torch.cuda.synchronize()
        for i, (o, r) in enumerate(zip(outs, refs)):
            assert np.array_equal(dev_to_u32(o), r), (i, mode, block, rounds)
