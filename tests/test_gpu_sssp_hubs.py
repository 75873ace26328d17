"""GPU parity of grid-mode shortest paths and levels where many vertices share
their targets: hubs joined with all vertices and in-hubs that all point at, with
rows short enough for a lane each, whose lanes then make one offer a wave;
repeated edges, waves that are not full, weights that let many offers pass and
weights that saturate; against the oracle and against flat mode, exactly."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev_to_u32, say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


def graph(n, hubs, extra, both, repeat, seed):
    rng = np.random.default_rng(seed)
    v = np.repeat(np.arange(n), hubs)
    h = np.tile(rng.choice(n, hubs, replace=False), n)
    src, dst = [v] * repeat, [h] * repeat
    if both:
        src.append(h), dst.append(v)
    src.append(rng.integers(0, n, extra * n)), dst.append(rng.integers(0, n, extra * n))
    src, dst = np.concatenate(src), np.concatenate(dst)
    order = np.lexsort((dst, src))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int32)
    return synth.CSR(n, ptr, dst[order].astype(np.int32))


@pytest.mark.parametrize("n,hubs,extra,both,repeat", [(8193, 1, 0, True, 1), (9001, 3, 0, True, 1), (30011, 4, 0, True, 1),
                                                      (9001, 2, 3, True, 2), (20000, 8, 0, True, 1), (9999, 2, 4, False, 1),
                                                      (9999, 3, 12, True, 1), (8200, 1, 1, False, 3)])
def test_shared_targets(ctx, n, hubs, extra, both, repeat):
    g = graph(n, hubs, extra, both, repeat, n + hubs)
    dg = wc.DeviceCSR.from_host(g.row_ptr, g.col)
    rng = np.random.default_rng(1)
    for top in (3, 101, 1 << 20, 0xFFFFFFF0):
        w = rng.integers(1, top, g.m, dtype=np.uint32)
        dw = u32_to_dev(w)
        for src in (int(np.argmax(g.degrees())), n - 1):
            for threshold in (0, 2, 64):
                say(f"shared targets n={n} hubs={hubs} extra={extra} top={top} src={src} threshold={threshold}")
                d = dev_to_u32(ctx.sssp(dg, dw, src, tune=wc.make_tune(threshold=threshold)))
                if top < 1 << 21:
                    assert np.array_equal(d, oracle.sssp_dijkstra(g.row_ptr, g.col, w, src)), (top, src, threshold)
                else:
                    assert np.array_equal(d, dev_to_u32(ctx.sssp(dg, dw, src, mode="flat"))), (src, threshold)
    assert np.array_equal(dev_to_u32(ctx.bfs(dg, 0)), oracle.bfs(g.row_ptr, g.col, 0))
