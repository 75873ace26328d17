"""GPU parity of grid mode's one-launch path for small graphs (up to 8,192
vertices and 4 to 131,072 edges, library tune): both sides of its limits, the
edges of its degree classes (32 and 256 edges), rows that start at every
alignment, edge arrays that end inside a load of four, long chains, saturating
distances; against the oracle and the general path (a caller's threshold),
exactly."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev_to_u32, say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


def of_degrees(deg, seed):
    """Row u has deg[u] edges to random vertices (loops and repeats included)."""
    ptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    rng = np.random.default_rng(seed)
    return synth.CSR(len(deg), ptr, rng.integers(0, len(deg), int(ptr[-1])).astype(np.int32))


def with_edges(n, m, seed):
    return of_degrees(np.bincount(np.random.default_rng(seed).integers(0, n, m), minlength=n), seed + 1)


def chain(n):
    return synth.CSR(n, np.minimum(np.arange(n + 1), n - 1).astype(np.int32), np.arange(1, n, dtype=np.int32))


def cases():
    for n, m in [(1, 4), (2, 3), (2, 4), (3, 5), (63, 250), (1023, 9000), (1024, 9001), (1025, 9002), (8191, 65537),
                 (8192, 131071), (8192, 131072), (8192, 131073), (8193, 40000)]:
        yield f"random {n} {m}", with_edges(n, m, n + m)
    for off in range(4):
        deg = [off, 1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 255, 256, 257, 0, 1023, 1025] + [3] * 40
        yield f"degrees, offset {off}", of_degrees(deg, off)
    yield "one hub", of_degrees([131072] + [0] * 8191, 5)
    yield "wave-wide vertices", of_degrees([257] * 510 + [0] * 100, 6)
    yield "chain", chain(2500)
    yield "rmat", synth.rmat_csr(12, 1 << 16, seed=8)


def test_small_graphs(ctx):
    for name, g in cases():
        dg = wc.DeviceCSR.from_host(g.row_ptr, g.col)
        rng = np.random.default_rng(9)
        for top in (16, 1 << 16, 0xFFFFFFF0):
            w = rng.integers(1, top, g.m, dtype=np.uint32)
            dw = u32_to_dev(w)
            for src in {0, g.n - 1}:
                say(f"small sssp {name} n={g.n} m={g.m} top={top} src={src}")
                d = dev_to_u32(ctx.sssp(dg, dw, src))
                same = dev_to_u32(ctx.sssp(dg, dw, src, tune=wc.make_tune(threshold=24)))
                assert np.array_equal(d, same), (name, top, src)
                if top < 1 << 20:  # the oracle's distances must stay below 2^32
                    assert np.array_equal(d, oracle.sssp_dijkstra(g.row_ptr, g.col, w, src)), (name, top, src)
        say(f"small bfs {name}")
        assert np.array_equal(dev_to_u32(ctx.bfs(dg, 0)), oracle.bfs(g.row_ptr, g.col, 0)), name


@pytest.mark.parametrize("n", [4097, 10007])
@pytest.mark.parametrize("off", [1, 2, 3])
def test_arrays_at_any_element(ctx, n, off):
    """Columns, weights and distances that start at any element of an allocation,
    on both paths; nothing is written beside the distances."""
    g = with_edges(n, 5 * n + 1, n)
    w = np.random.default_rng(off).integers(1, 1000, g.m, dtype=np.uint32)
    col = torch.zeros(g.m + 8, dtype=torch.int32, device="cuda")
    wt, out = torch.zeros_like(col), torch.full((n + 8,), 77, dtype=torch.int32, device="cuda")
    col[off:off + g.m] = torch.from_numpy(g.col).cuda()
    wt[off:off + g.m] = u32_to_dev(w)
    dg = wc.DeviceCSR(n, torch.from_numpy(g.row_ptr).cuda(), col[off:off + g.m])
    say(f"sssp arrays at element {off} n={n}")
    ctx.sssp(dg, wt[off:off + g.m], 3, out=out[off:off + n])
    torch.cuda.synchronize()
    assert np.array_equal(dev_to_u32(out[off:off + n]), oracle.sssp_dijkstra(g.row_ptr, g.col, w, 3))
    assert (out[:off] == 77).all() and (out[off + n:] == 77).all()
