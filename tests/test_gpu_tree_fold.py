"""GPU parity of the trees' fold tiles (grid mode without work counters): trees
whose work list (child entries and nodes, 2n - 1 in all) ends on, before and
after a tile's edge, hubs and runs of leaves that span several tiles, chains,
and batches that mix one-node trees with ones of many tiles; against the
oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
TILE = 2048  # work-list entries a tile


def shuffled(t, seed):
    """The same tree with the non-root ids permuted."""
    perm = np.concatenate([[0], 1 + np.random.default_rng(seed).permutation(t.n - 1)]).astype(np.int64)
    parent = np.full(t.n, -1, dtype=np.int64)
    parent[perm[1:]] = perm[t.parent[1:]]
    return synth.tree_from_parent(parent)


def broom(n, handle):
    """A chain of `handle` edges whose last node has all other nodes as children."""
    return synth.tree_from_parent([-1] + list(range(handle)) + [handle] * (n - handle - 1))


def trees():
    for n in (1, 2, 3, 64, TILE // 2, TILE // 2 + 1, TILE, TILE + 1, 3 * TILE // 2, 3 * TILE // 2 + 1, 50001):
        yield f"random {n}", synth.random_tree(n, seed=n)
    for n in (TILE // 2 + 1, TILE, 5 * TILE + 3):
        yield f"star {n}", synth.star_tree(n)
        yield f"star shuffled {n}", shuffled(synth.star_tree(n), n)
        yield f"broom {n}", broom(n, n // 3)
        yield f"broom shuffled {n}", shuffled(broom(n, n // 3), n)
    yield "chain", synth.chain_tree(2 * TILE + 1)
    yield "binary", shuffled(synth.kary_tree(2, 12), 1)
    yield "wide inner", shuffled(synth.kary_tree(130, 2), 2)
    yield "layered", synth.layered_tree(2, 128, 256, 0.5, seed=3)


def dev(t):
    return wc.DeviceTree.from_host(t.parent, t.child_ptr, t.child)


def test_single_trees(ctx):
    for name, t in trees():
        say(f"fold tiles: {name} n={t.n}")
        dt = dev(t)
        d = ctx.tree_descendants(dt, mode="grid")
        h = ctx.tree_height(dt, mode="grid")
        torch.cuda.synchronize()
        assert np.array_equal(d.cpu().numpy(), oracle.tree_descendants(t.child_ptr, t.child)), name
        assert np.array_equal(h.cpu().numpy(), oracle.tree_height(t.child_ptr, t.child)), name


def test_one_batch_of_all(ctx):
    ts = [t for _, t in trees()]
    say(f"fold tiles: a batch of {len(ts)} trees")
    dts = [dev(t) for t in ts]
    for rep in range(3):
        for t, got in zip(ts, ctx.tree_descendants_batch(dts, mode="grid")):
            assert np.array_equal(got.cpu().numpy(), oracle.tree_descendants(t.child_ptr, t.child)), (rep, t.n)
        for t, got in zip(ts, ctx.tree_height_batch(dts, mode="grid")):
            assert np.array_equal(got.cpu().numpy(), oracle.tree_height(t.child_ptr, t.child)), (rep, t.n)
