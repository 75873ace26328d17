"""GPU parity of grid-mode products whose number of rows, not of entries, sets
their size: both sides of the row limit of the one-launch kernel and of its limit
for short matrices with many entries (bitwise the general path's sums), more rows
than a launch of eight rows to a workgroup could cover, and both sides of the
limits of PageRank, which depend on the number of sweeps."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import f32_to_dev, say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
# the library's own values, given explicitly: the general path
GENERAL = dict(threshold=8, items_per_lane=8, block_threads=512)


@pytest.mark.parametrize("n,m", [(32768, 5000), (32769, 5000), (32767, 1 << 18), (32769, 1 << 18), (200000, 3000),
                                 (181, 32768), (181, 32769), (182, 33124), (182, 33125), (3, 32768), (3, 32769)])
def test_both_sides_of_the_row_limits(ctx, n, m):
    rng = np.random.default_rng(n + m)
    # half the entries in few rows
    rows = np.where(rng.random(m) < 0.5, rng.integers(0, n, m), rng.integers(0, min(n, 40), m) * (n // min(n, 40)))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    g = synth.CSR(n, ptr, rng.integers(0, n, m).astype(np.int32))
    val, x = synth.values(m, seed=1), synth.vector_x(n, seed=2)
    y_ref, b = oracle.spmv_f64(g.row_ptr, g.col, val, x)
    dg, dv, dx = wc.DeviceCSR.from_host(g.row_ptr, g.col), f32_to_dev(val), f32_to_dev(x)
    say(f"spmv by rows: n={n} m={m}")
    y = ctx.spmv(dg, dv, dx).cpu().numpy()
    assert oracle.spmv_check(y_ref, b, y) == (0, -1)
    general = ctx.spmv(dg, dv, dx, tune=wc.make_tune(**GENERAL)).cpu().numpy()
    assert np.array_equal(y.view(np.uint32), general.view(np.uint32))


def test_more_rows_than_threads_of_a_launch(ctx):
    """2^26 + 9 rows, 1,000 entries in the first and the last of them."""
    n, m = (1 << 26) + 9, 1000
    ptr = torch.full((n + 1,), m // 2, dtype=torch.int32, device="cuda")
    ptr[0], ptr[n] = 0, m
    gen = torch.Generator(device="cuda").manual_seed(3)
    col = torch.randint(0, n, (m,), dtype=torch.int32, device="cuda", generator=gen)
    val = torch.rand(m, device="cuda", generator=gen)
    x = torch.rand(n, device="cuda", generator=gen)
    say(f"spmv by rows: n={n} m={m}")
    y = ctx.spmv(wc.DeviceCSR(n, ptr, col), val, x, out=torch.full((n,), 7.0, device="cuda"))
    torch.cuda.synchronize()
    want = (val.double() * x[col.long()].double()).view(2, -1).sum(1)
    got = torch.stack([y[0], y[-1]]).double()
    # all terms are positive: the documented bound of 1e-5 of their sum
    assert ((got - want).abs() <= 1e-5 * want).all()
    assert not y[1:-1].any()


@pytest.mark.parametrize("iterations,n", [(1, 32768), (2, 24576), (2, 24577), (4, 12288), (4, 12289), (9, 5461), (9, 5462)])
def test_pagerank_by_sweeps(ctx, iterations, n):
    m = 50000
    rng = np.random.default_rng(n)
    rows = np.where(rng.random(m) < 0.8, rng.integers(0, n, m), 17)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    col = rng.integers(0, n - 5, m).astype(np.int32)
    od = np.bincount(col, minlength=n).astype(np.int32)
    dg, dod = wc.DeviceCSR.from_host(ptr, col), torch.from_numpy(od).cuda()
    say(f"pagerank by sweeps: {iterations} n={n}")
    r = ctx.pagerank(dg, dod, iterations).cpu().numpy()
    assert oracle.pagerank_check(oracle.pagerank_f64(ptr, col, od, iterations), r)[0] == 0
    general = ctx.pagerank(dg, dod, iterations, tune=wc.make_tune(**GENERAL)).cpu().numpy()
    assert np.array_equal(r.view(np.uint32), general.view(np.uint32))
