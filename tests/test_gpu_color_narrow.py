"""GPU parity of grid-mode coloring's small rounds (many rounds a launch by one
workgroup, without work counters): more rounds than one launch takes, rounds on
both sides of its limits (1,024 vertices, 8,192 neighbour entries) in turn, so
that the work goes back and forth between the workgroup and the grid, and the
starts with many vertices; against the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import say, u32_to_dev
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


def layers(sizes, seed):
    """Consecutive layers fully connected, every layer outranking the next: one
    round a layer.  Ids shuffled."""
    first = np.concatenate([[0], np.cumsum(sizes)])
    n = int(first[-1])
    perm = np.random.default_rng(seed).permutation(n)
    edges = []
    for k in range(len(sizes) - 1):
        u, v = np.meshgrid(np.arange(first[k], first[k + 1]), np.arange(first[k + 1], first[k + 2]))
        edges.append(np.stack([perm[u.ravel()], perm[v.ravel()]], 1))
    e = np.concatenate(edges)
    e = np.concatenate([e, e[:, ::-1]])
    order = np.lexsort((e[:, 1], e[:, 0]))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(e[:, 0], minlength=n))]).astype(np.int32)
    prio = np.zeros(n, np.uint32)
    for k in range(len(sizes)):
        prio[perm[first[k]:first[k + 1]]] = 10 * (len(sizes) - k)
    return synth.CSR(n, ptr, e[order, 1].astype(np.int32)), prio


def path(n):
    g = synth.symmetrize(synth.graph_from_edges(n, [(i, i + 1) for i in range(n - 1)])[0])
    return g, np.arange(n, dtype=np.uint32)


def cases():
    yield "path of 9,000", *path(9000)
    yield "wide and narrow in turn", *layers([1, 1500, 2, 1023, 1, 1024, 1, 1025, 3, 2000, 1], 1)
    yield "entries at the limit", *layers([2, 4094, 1, 2, 4095, 1, 2, 4096, 1, 2], 2)
    yield "many starts", *layers([3000, 1, 1, 40, 1], 3)
    yield "one after another", *layers([1] * 300, 4)
    g = synth.symmetrize(synth.rmat_csr(12, 1 << 17, seed=5))
    yield "rmat", g, synth.priorities(g.n)
    yield "rmat, equal priorities", g, np.zeros(g.n, np.uint32)
    yield "no edges", synth.graph_from_edges(5, [])[0], np.arange(5, dtype=np.uint32)


def test_narrow_rounds(ctx):
    for name, g, prio in cases():
        say(f"narrow rounds: {name} n={g.n} m={g.m}")
        ref, _ = oracle.color_jp(g.row_ptr, g.col, prio)
        dg = wc.DeviceCSR.from_host(g.row_ptr, g.col)
        for rep in range(2):
            got = ctx.color(dg, u32_to_dev(prio), mode="grid")
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), ref), (name, rep)


def test_counts_of_more_than_16_bits(ctx):
    """Multi-edges: a vertex outranked along 70,000 edges, more than the packed
    counts hold, next to an ordinary graph."""
    e = [(0, 1), (1, 0)] * 70000 + [(i, j) for i in range(2, 40) for j in range(2, 40) if i != j]
    g = synth.graph_from_edges(40, e)[0]
    prio = np.arange(40, dtype=np.uint32)[::-1].copy()
    ref, _ = oracle.color_jp(g.row_ptr, g.col, prio)
    say("narrow rounds: counts of more than 16 bits")
    got = ctx.color(wc.DeviceCSR.from_host(g.row_ptr, g.col), u32_to_dev(prio), mode="grid")
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), ref)


def test_asymmetric_graph_takes_the_general_path(ctx):
    """Edges without their reverse release vertices that never counted them: the
    packed counts would go below zero, so the call is done again round by round,
    with the status and the colors that a call with counters gives."""
    rng = np.random.default_rng(6)
    n = 300
    # a symmetric graph, and edges from high to low priority without a reverse
    sym = synth.symmetrize(synth.graph_from_edges(n, [tuple(p) for p in rng.integers(0, n, (2000, 2))])[0])
    src = np.repeat(np.arange(n), np.diff(sym.row_ptr))
    extra = [(n - 1, v) for v in range(50)] + [(n - 2, v) for v in range(50)]
    g = synth.graph_from_edges(n, list(zip(src.tolist(), sym.col.tolist())) + extra * 3)[0]
    prio = np.arange(n, dtype=np.uint32)
    dg, dp = wc.DeviceCSR.from_host(g.row_ptr, g.col), u32_to_dev(prio)

    def outcome(**kw):
        try:
            got = ctx.color(dg, dp, mode="grid", **kw)
            torch.cuda.synchronize()
            return (got[0] if kw.get("stats") else got).cpu().numpy().tolist()
        except wc.WcError as e:
            torch.cuda.synchronize()
            return e.status
    say("narrow rounds: an asymmetric graph")
    want = outcome(stats=True)
    assert outcome() == want
    # the library stays usable
    ref, _ = oracle.color_jp(sym.row_ptr, sym.col, prio)
    got = ctx.color(wc.DeviceCSR.from_host(sym.row_ptr, sym.col), dp, mode="grid")
    assert np.array_equal(got.cpu().numpy(), ref)
