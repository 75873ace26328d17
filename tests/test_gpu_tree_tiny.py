"""Batches of very many small trees: the workspace of the fold tiles follows the
nodes and the trees, not a whole tile for every tree, also where trees of some
tiles stand between them; against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


def test_workspace_and_results(ctx):
    kinds = [synth.random_tree(n, seed=n) for n in list(range(1, 10)) + [1023, 1024, 1025, 1026, 5000]]
    refs = [(oracle.tree_descendants(t.child_ptr, t.child), oracle.tree_height(t.child_ptr, t.child)) for t in kinds]
    dev = [wc.DeviceTree.from_host(t.parent, t.child_ptr, t.child) for t in kinds]
    which = [i % 9 if i % 500 else 9 + i // 500 % 5 for i in range(20000)]
    trees = [dev[k] for k in which]
    room = torch.full((sum(t.n for t in trees) + 1,), -7, dtype=torch.int32, device="cuda")
    ends = np.cumsum([0] + [t.n for t in trees]).tolist()
    outs = [room[a:b] for a, b in zip(ends, ends[1:])]
    want = [np.concatenate([refs[k][j] for k in which]) for j in range(2)]
    for j, name in enumerate(("tree_descendants_batch", "tree_height_batch")):
        need = ctx.workspace_bytes(lambda c: getattr(c, name)(trees, mode="grid", outs=outs))
        say(f"many small trees: {name} {ends[-1]} nodes, {need} bytes")
        assert need <= 64 * (ends[-1] + len(trees)) + (1 << 16)  # a tile a tree: 82 MB
        getattr(ctx, name)(trees, mode="grid", outs=outs)
        torch.cuda.synchronize()
        got = room.cpu().numpy()
        assert np.array_equal(got[:-1], want[j]) and got[-1] == -7, name
