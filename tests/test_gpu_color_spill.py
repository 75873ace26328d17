"""GPU parity of grid-mode coloring where a small round readies more chunks than
the workgroup's list of 1,024 holds: rows made long by self-loops (ignored, but
entries of the row), around the list's end and far beyond it, in graphs with
hardly any other entries, so that the chunk buffers have no room to spare;
against the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
CHUNK, LIST = 128, 1024


def star(chunks, leaves):
    """Vertex 0 outranks `leaves` leaves, each of which outranks a vertex of its
    own at the end of its row; leaf k has rows of chunks[k] chunks by self-loops."""
    e = []
    for k in range(leaves):
        leaf, pendant = 1 + k, 1 + leaves + k
        loops = CHUNK * chunks[k] - 2 if k < len(chunks) else 0
        e.append(np.array([(0, leaf), (leaf, 0)] + [(leaf, pendant), (pendant, leaf)]))
        e.append(np.full((loops, 2), leaf))
    e = np.concatenate(e)
    n = 1 + 2 * leaves
    e = e[np.lexsort((e[:, 1], e[:, 0]))]
    ptr = np.concatenate([[0], np.cumsum(np.bincount(e[:, 0], minlength=n))]).astype(np.int32)
    return synth.CSR(n, ptr, e[:, 1].astype(np.int32)), np.arange(n, dtype=np.uint32)[::-1].copy()


@pytest.mark.parametrize("leaves", [1, 2, 64])
@pytest.mark.parametrize("total", [LIST - 1, LIST, LIST + 1, LIST + 64, 3 * LIST + 7])
def test_rows_beyond_the_list(ctx, leaves, total):
    rest = total - leaves
    for chunks in ([rest + 1], [rest // 2 + 1, rest - rest // 2 + 1]):
        if len(chunks) > leaves:
            continue
        g, prio = star(chunks, leaves)
        assert int(((g.degrees()[1:1 + leaves] + CHUNK - 1) // CHUNK).sum()) == total
        ref, _ = oracle.color_jp(g.row_ptr, g.col, prio)
        dg = wc.DeviceCSR.from_host(g.row_ptr, g.col)
        for rep in range(3):
            say(f"narrow rounds: {leaves} leaves, {total} chunks in rows of {chunks}, run {rep}")
            got = ctx.color(dg, u32_to_dev(prio), mode="grid")
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), ref)
