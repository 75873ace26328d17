"""GPU parity of grid-mode coloring where rounds change between the one workgroup
and the grid: a round is the workgroup's up to 256 chunks (a chunk: up to 128
entries of a row), the first of a launch up to 160 chunks and 8,192 entries; a
round that readies more than 256 vertices ends a launch, and up to 64 vertices
have 16 lanes each; runs of large rounds are the grid's alone.  Layers of every
size around these limits, rows of 127 to 129 entries, in turn and at random;
against the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, u32_to_dev
from paper_1606_08150_amd import wc
from test_gpu_color_narrow import layers

pytestmark = pytest.mark.gpu


def sequences():
    for limit in (16, 32, 64, 160, 256):  # chunks a wave takes, vertices and chunks of a round
        one = [s for k in (-1, 0, 1) for s in (limit + k, 1, 2)]
        yield f"around {limit}", [1] + one + [1]
        yield f"around {limit} after a large round", [s for k in (-1, 0, 1) for s in (400, limit + k, 1, 1)]
    yield "rows of 127 to 129 entries", [1, 100, 27, 100, 28, 100, 29, 1, 127, 128, 129, 1, 3]
    yield "entries of a first round", [400, 10, 409, 1, 400, 10, 419, 1, 400, 10, 419, 10, 410, 2]
    yield "large rounds, then small ones, and again", [300] * 9 + [1] * 9 + [270] * 7 + [2, 1, 300, 1, 300, 300, 300, 300, 1, 1]
    yield "starts with small rounds", [5, 4, 3, 600, 600, 600, 600, 600, 1, 1, 1]
    rng = np.random.default_rng(1)
    for k in range(4):
        size = np.exp(rng.uniform(0, np.log(500), 60)).astype(int) + 1
        yield f"random {k}", np.sort(size).tolist() if k == 3 else size.tolist()


def test_rounds_around_the_limits(ctx):
    for name, sizes in sequences():
        g, prio = layers([int(s) for s in sizes], len(sizes))
        assert g.n <= 65536
        ref, _ = oracle.color_jp(g.row_ptr, g.col, prio)
        dg, dp = wc.DeviceCSR.from_host(g.row_ptr, g.col), u32_to_dev(prio)
        for rep in range(3):
            say(f"coloring phases: {name} n={g.n} m={g.m} run {rep}")
            got = ctx.color(dg, dp, mode="grid")
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), ref), (name, rep)


@pytest.mark.parametrize("n,degree", [(300, 3), (2000, 40), (16384, 16), (50000, 8), (65536, 3)])
def test_random_graphs(ctx, n, degree):
    """Rounds that shrink slowly past the limits."""
    import synth
    rng = np.random.default_rng(n)
    e = rng.integers(0, n, (n * degree // 2, 2))
    e = np.concatenate([e, e[:, ::-1]])
    e = e[np.lexsort((e[:, 1], e[:, 0]))]
    ptr = np.concatenate([[0], np.cumsum(np.bincount(e[:, 0], minlength=n))]).astype(np.int32)
    g = synth.CSR(n, ptr, e[:, 1].astype(np.int32))
    prio = synth.priorities(n)
    ref, _ = oracle.color_jp(g.row_ptr, g.col, prio)
    dg, dp = wc.DeviceCSR.from_host(g.row_ptr, g.col), u32_to_dev(prio)
    for rep in range(3):
        say(f"coloring phases: random n={n} degree={degree} run {rep}")
        got = ctx.color(dg, dp, mode="grid")
        assert np.array_equal(got.cpu().numpy(), ref), rep
