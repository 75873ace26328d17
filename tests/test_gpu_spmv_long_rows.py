"""GPU parity of products with rows of many chunks, whose chunks are counted in
groups of 64 entries of the buffer: rows of 63 to 65, 127 to 129 and some
thousand chunks side by side, so that groups of two rows share a run of 64
entries, few and many workgroups, every mode that splits rows, and buffers that
serve several products (PageRank's sweeps); against the oracle, and bitwise
against another grid."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f32_to_dev, say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
CHUNK = 64  # items_per_lane 1


def matrix(n, seed):
    rng = np.random.default_rng(seed)
    chunks = [63, 64, 65, 1, 127, 128, 129, 2, 3000, 66, 66, 66, 191, 192, 193, 70, 5000]
    lens = rng.integers(0, 12, n)
    lens[rng.choice(n, len(chunks), replace=False)] = [CHUNK * c - int(rng.integers(0, CHUNK - 1)) for c in chunks]
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return synth.CSR(n, ptr, rng.integers(0, n, int(ptr[-1])).astype(np.int32))


@pytest.mark.parametrize("mode", ["wave", "block", "grid"])
def test_products(ctx, mode):
    for n, seed in ((40, 1), (900, 2), (50000, 3)):
        g = matrix(n, seed)
        val, x = synth.values(g.m, seed=4), synth.vector_x(g.n, seed=5)
        y_ref, b = oracle.spmv_f64(g.row_ptr, g.col, val, x)
        dg, dv, dx = wc.DeviceCSR.from_host(g.row_ptr, g.col), f32_to_dev(val), f32_to_dev(x)
        want = None
        for blocks in (0, 3, 100):
            tune = wc.make_tune(items_per_lane=1, grid_blocks=blocks)
            say(f"long rows: n={n} m={g.m} mode={mode} grid_blocks={blocks}")
            for _ in range(2):
                y = ctx.spmv(dg, dv, dx, mode=mode, tune=tune).cpu().numpy()
                assert oracle.spmv_check(y_ref, b, y) == (0, -1), (n, blocks)
                want = y if want is None else want
                assert np.array_equal(y.view(np.uint32), want.view(np.uint32)), (n, blocks)


def test_reused_buffers(ctx):
    g = matrix(3000, 6)
    od = np.bincount(g.col, minlength=g.n).astype(np.int32)
    dg, dod = wc.DeviceCSR.from_host(g.row_ptr, g.col), torch.from_numpy(od).cuda()
    for blocks in (0, 2):
        for it in (1, 2, 5):
            say(f"long rows: pagerank grid_blocks={blocks} sweeps={it}")
            tune = wc.make_tune(items_per_lane=1, grid_blocks=blocks)
            r = ctx.pagerank(dg, dod, it, mode="grid", tune=tune).cpu().numpy()
            assert oracle.pagerank_check(oracle.pagerank_f64(g.row_ptr, g.col, od, it), r)[0] == 0
            # a call with counters bins the rows in every sweep
            s, _ = ctx.pagerank(dg, dod, it, mode="grid", tune=tune, stats=True)
            assert np.array_equal(r.view(np.uint32), s.cpu().numpy().view(np.uint32))
