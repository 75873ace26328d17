"""GPU tests of the ways a grid-mode product can take: the one-launch kernel of
small matrices sums every row in the general path's order (bitwise the same, at
its edges: workgroups of 8 rows, the largest size, rows of many chunks), and the
general path's drain combines split rows whichever wave finishes them, also
where a wave holds more than 64 chunks."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f32_to_dev, say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
SMALL = 1 << 18
# the library's own values, given explicitly: the general path
GENERAL = dict(threshold=8, items_per_lane=8, block_threads=512)


def rows_of(lens, n, seed):
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return synth.CSR(n, ptr, rng.integers(0, n, int(ptr[-1])).astype(np.int32))


def matrices():
    for n in (1, 7, 8, 9, 64, 1000):
        yield f"rows {n}", rows_of(np.arange(n) % 40, n, n)
    edges = [0, 1, 8, 9, 16, 17, 128, 129, 511, 512, 513, 1024, 1025, 40 * 512 + 3]
    yield "every bin", rows_of(np.random.default_rng(5).permutation(edges * 3), 3 * len(edges), 6)
    yield "one row", rows_of([SMALL], 1, 7)
    hub = np.full(4096, 4)
    hub[77] = SMALL - 4 * 4095
    yield "a hub, largest small", rows_of(hub, 4096, 8)
    hub[78] += 1
    yield "a hub, smallest general", rows_of(hub, 4096, 9)
    yield "rmat", synth.rmat_csr(14, SMALL, seed=10)


def run(ctx, g, val, x, **tune):
    y = ctx.spmv(wc.DeviceCSR.from_host(g.row_ptr, g.col), f32_to_dev(val), f32_to_dev(x), mode="grid",
                 tune=wc.make_tune(**tune) if tune else None)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def test_small_and_general_path_agree(ctx):
    for name, g in matrices():
        say(f"spmv paths: {name} n={g.n} m={g.m}")
        val, x = synth.values(g.m, seed=11), synth.vector_x(g.n, seed=12)
        y_ref, b = oracle.spmv_f64(g.row_ptr, g.col, val, x)
        y = run(ctx, g, val, x)
        assert oracle.spmv_check(y_ref, b, y) == (0, -1), name
        general = run(ctx, g, val, x, **GENERAL)
        assert np.array_equal(y.view(np.uint32), general.view(np.uint32)), name


@pytest.mark.parametrize("blocks", [1, 3])
def test_many_chunks_a_wave(ctx, blocks):
    """One or three workgroups of one wave and chunks of 64 entries: hundreds of
    chunks a wave, rows split between waves."""
    g = rows_of([30000, 5, 64, 65, 0, 12000, 129, 4000, 1], 9, 13)
    val, x = synth.values(g.m, seed=14), synth.vector_x(g.n, seed=15)
    y_ref, b = oracle.spmv_f64(g.row_ptr, g.col, val, x)
    say(f"spmv drain: {blocks} workgroups of one wave")
    y = run(ctx, g, val, x, grid_blocks=blocks, block_threads=64, items_per_lane=1)
    assert oracle.spmv_check(y_ref, b, y) == (0, -1)
    wide = run(ctx, g, val, x, items_per_lane=1)
    assert np.array_equal(y.view(np.uint32), wide.view(np.uint32))


def test_pagerank_paths_agree(ctx):
    """PageRank's sweeps through the one-launch kernel and through reused buffers
    give the same ranks."""
    g = synth.transpose(synth.rmat_csr(11, 1 << 15, seed=16))
    od = torch.from_numpy(np.bincount(g.col, minlength=g.n).astype(np.int32)).cuda()
    dg = wc.DeviceCSR.from_host(g.row_ptr, g.col)
    for it in (0, 1, 2, 7):
        say(f"pagerank paths: {it} sweeps")
        a = ctx.pagerank(dg, od, it, mode="grid").cpu().numpy()
        b = ctx.pagerank(dg, od, it, mode="grid", tune=wc.make_tune(**GENERAL)).cpu().numpy()
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), it
        assert oracle.pagerank_check(oracle.pagerank_f64(g.row_ptr, g.col, od.cpu().numpy(), it), a)[0] == 0
