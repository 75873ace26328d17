"""GPU parity of grid-mode trees on both sides of the size from which a bit a node
tells the nodes with children (2^20), with node counts that end inside a word of
bits and inside a wave's words; against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
LIMIT = 1 << 20


def broom(n, handle):
    """A chain of `handle` edges whose last node has all other nodes as children."""
    parent = np.full(n, handle, dtype=np.int64)
    parent[0] = -1
    parent[1:handle + 1] = np.arange(handle)
    return synth.tree_from_parent(parent)


@pytest.mark.parametrize("n", [LIMIT, LIMIT + 1, LIMIT + 63, LIMIT + 64, LIMIT + 257])
def test_large_trees(ctx, n):
    for name, t in (("random", synth.random_tree(n, seed=n)), ("broom", broom(n, 700))):
        say(f"tree inner bits: {name} n={n}")
        d = wc.DeviceTree.from_host(t.parent, t.child_ptr, t.child)
        desc, height = ctx.tree_descendants(d, mode="grid"), ctx.tree_height(d, mode="grid")
        torch.cuda.synchronize()
        assert np.array_equal(desc.cpu().numpy(), oracle.tree_descendants(t.child_ptr, t.child)), (name, n)
        assert np.array_equal(height.cpu().numpy(), oracle.tree_height(t.child_ptr, t.child)), (name, n)
