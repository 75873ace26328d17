"""The work this library is timed on: calls a user makes through ``paper_1606_08150_amd.wc.Context``.

Graphs are R-MAT with quadrant probabilities 0.57 / 0.19 / 0.19 / 0.05 and about 16 edges a vertex, weights 1..100,
values and vectors in [-1, 1): the workload of the benchmark, the tests and the request server.  Trees have the
truncated power-law fanout, the depth limit of 24 and the shuffled node ids of the synthetic trees.  Everything is
generated on the GPU from the seed.  A case's kinds:

  spmv, sssp, bfs    one product, one shortest-path or one breadth-first call over a resident graph
  pagerank           `iterations` sweeps over the in-edges of a graph
  color              Jones-Plassmann colors of a symmetric graph
  tree               descendants or heights of one resident tree
  tree_batch         descendants or heights of many trees in one call
  sssp_batch         many shortest-path instances in one call, as the request server issues them
"""
import math

import torch

from paper_1606_08150_amd import wc

QUADRANTS = (0.57, 0.19, 0.19)
KMAX, ALPHA, MAX_DEPTH = 4096, 2.0, 24
LARGEST = 1 << 26  # edges of the largest graph

_context = None


def context():
    """The process's one library context, as a program that serves calls one after another keeps it."""
    global _context
    if _context is None:
        _context = wc.Context(0)
    return _context


def listed():
    return [
        # one product with a small resident matrix: what a latency-bound caller waits for
        {"name": "spmv-4k", "kind": "spmv", "n": 4096, "degree": 16, "mode": "grid"},
        # a product of the request server, whose graphs have 2^14 to 2^20 vertices of no round number
        {"name": "spmv-200k", "kind": "spmv", "n": 200003, "degree": 16, "mode": "grid"},
        # the benchmark's product: scale 22, 67M nonzeros
        {"name": "spmv-4m", "kind": "spmv", "n": 1 << 22, "degree": 16, "mode": "grid"},
        # shortest paths on a small graph: a handful of short rounds
        {"name": "sssp-4k", "kind": "sssp", "n": 4096, "degree": 16, "mode": "grid"},
        # a shortest-path request of the server
        {"name": "sssp-150k", "kind": "sssp", "n": 150001, "degree": 16, "mode": "grid"},
        # the benchmark's headline: shortest paths at scale 22
        {"name": "sssp-4m", "kind": "sssp", "n": 1 << 22, "degree": 16, "mode": "grid"},
        # breadth-first levels of a large graph
        {"name": "bfs-1m", "kind": "bfs", "n": 1 << 20, "degree": 16, "mode": "grid"},
        # ten sweeps of PageRank, the benchmark's number of sweeps
        {"name": "pagerank-1m", "kind": "pagerank", "n": 1 << 20, "degree": 16, "iterations": 10, "mode": "grid"},
        # coloring of the symmetrised scale-16 graph: hundreds of short dependent rounds
        {"name": "color-65k", "kind": "color", "n": 1 << 16, "degree": 32, "mode": "grid"},
        # the benchmark's tree: 2^22 nodes, two dozen levels
        {"name": "tree-4m", "kind": "tree", "op": "descendants", "n": 1 << 22, "mode": "grid"},
        # a forest of small and middling trees in one call
        {"name": "tree-batch-64", "kind": "tree_batch", "op": "height", "count": 64, "lo": 1 << 10, "hi": 1 << 17,
         "mode": "grid"},
        # many shortest-path requests admitted together, at the level the batch tuner chooses
        {"name": "sssp-batch-64", "kind": "sssp_batch", "count": 64, "lo": 1 << 10, "hi": 1 << 17, "degree": 16,
         "mode": "block"},
    ]


def _between(rng, lo, hi):
    """A size between lo and hi, even over its logarithm; mostly an odd or ragged one."""
    n = int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))
    return max(lo, min(hi, n | 1 if rng.random() < 0.7 else n))


def draw(rng):
    kind = rng.choice(["spmv", "spmv", "spmv", "sssp", "sssp", "sssp", "bfs", "pagerank", "color", "tree", "tree",
                       "tree_batch", "sssp_batch"])
    degree = rng.randint(8, 24)
    mode = rng.choice(["grid"] * 8 + ["block", "wave"])
    if kind in ("spmv", "sssp", "bfs"):
        n = _between(rng, 1 << 10, 1 << 22)
        return {"kind": kind, "n": n, "degree": min(degree, LARGEST // n), "mode": mode if kind != "bfs" else "grid"}
    if kind == "pagerank":
        return {"kind": kind, "n": _between(rng, 1 << 10, 1 << 20), "degree": min(degree, 16),
                "iterations": rng.randint(2, 10), "mode": "grid"}
    if kind == "color":
        return {"kind": kind, "n": _between(rng, 1 << 10, 1 << 16), "degree": degree, "mode": "grid"}
    op = rng.choice(["descendants", "height"])
    if kind == "tree":
        return {"kind": kind, "op": op, "n": _between(rng, 1 << 10, 1 << 22),
                "mode": rng.choice(["grid"] * 4 + ["block"])}
    count, hi = rng.randint(4, 64), _between(rng, 1 << 12, 1 << 17)
    if kind == "tree_batch":
        return {"kind": kind, "op": op, "count": count, "lo": 1 << 10, "hi": hi, "mode": "grid"}
    return {"kind": kind, "count": count, "lo": 1 << 10, "hi": hi, "degree": min(degree, 16),
            "mode": rng.choice(["block", "grid"])}


# ---- inputs --------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rmat(n, m, gen):
    """m R-MAT edges over n vertices: the endpoints' bits are drawn from the top, and where n is no power of two
    the pair is scaled onto [0, n)."""
    bits = max(1, math.ceil(math.log2(n)))
    scaled = (1 << bits) != n
    bits += 2 if scaled else 0
    a, ab, abc = QUADRANTS[0], QUADRANTS[0] + QUADRANTS[1], sum(QUADRANTS)
    s = torch.zeros(m, dtype=torch.int64, device="cuda")
    t = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(bits):
        u = torch.rand(m, device="cuda", generator=gen)
        s.mul_(2).add_(u >= ab)
        t.mul_(2).add_(((u >= a) & (u < ab)) | (u >= abc))
    if scaled:
        s = (s * n) >> bits
        t = (t * n) >> bits
    return s, t


def _csr_of_keys(key, n):
    """CSR arrays of the sorted keys row * n + column."""
    row = torch.div(key, n, rounding_mode="floor")
    col = (key - row * n).to(torch.int32)
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return ptr.to(torch.int32), col


def _graph(n, m, gen):
    s, t = _rmat(n, m, gen)
    ptr, col = _csr_of_keys(torch.sort(s * n + t)[0], n)
    return wc.DeviceCSR(n, ptr, col)


def _symmetric(n, m, gen):
    s, t = _rmat(n, m, gen)
    keep = s != t
    s, t = s[keep], t[keep]
    ptr, col = _csr_of_keys(torch.unique(torch.cat([s * n + t, t * n + s])), n)
    return wc.DeviceCSR(n, ptr, col)


def _weights(m, gen):
    return torch.randint(1, 101, (m,), dtype=torch.int32, device="cuda", generator=gen)


def _uniform(k, gen):
    return torch.rand(k, device="cuda", generator=gen) * 2 - 1


def _source(g, gen):
    """A vertex with out-edges: the source of a random edge."""
    e = torch.randint(0, g.m, (1,), dtype=torch.int64, device="cuda", generator=gen)
    return int(torch.searchsorted(g.row_ptr[1:].to(torch.int64), e, right=True))


def _tree(n, gen):
    """n nodes grown level by level, P(fanout = k) proportional to (k + 1)^-ALPHA, ids shuffled, child lists sorted."""
    cdf = torch.cumsum(torch.arange(1, KMAX + 2, dtype=torch.float64, device="cuda") ** -ALPHA, 0)
    cdf /= cdf[-1].clone()
    parents, first, size, made = [torch.full((1,), -1, dtype=torch.int64, device="cuda")], 0, 1, 1
    while made < n:
        u = torch.rand(size, dtype=torch.float64, device="cuda", generator=gen)
        if float(u.max()) < float(cdf[0]):  # no node of the level has children: the last one draws at least one
            u[-1] = cdf[0] + u[-1] / cdf[0] * (1 - cdf[0])
        if len(parents) == MAX_DEPTH:  # the last level takes the nodes that are still missing
            fan = torch.full((size,), -(-(n - made) // size), dtype=torch.int64, device="cuda")
        else:
            fan = torch.searchsorted(cdf, u, right=True).clamp_(max=KMAX)
        p = torch.repeat_interleave(torch.arange(first, first + size, device="cuda"), fan)[:n - made]
        parents.append(p)
        first, size, made = made, int(p.numel()), made + int(p.numel())
    old = torch.cat(parents)
    perm = torch.zeros(n, dtype=torch.int64, device="cuda")
    perm[1:] = torch.randperm(n - 1, device="cuda", generator=gen) + 1
    parent = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    parent[perm[1:]] = perm[old[1:]]
    child = torch.argsort(parent[1:], stable=True) + 1
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.bincount(parent[1:], minlength=n), 0)
    return wc.DeviceTree(n, parent.to(torch.int32), ptr.to(torch.int32), child.to(torch.int32))


def _sizes(case):
    """Instance sizes between lo and hi, even over their logarithm."""
    k, lo, hi = case["count"], math.log2(case["lo"]), math.log2(case["hi"])
    return [int(2.0 ** (lo + (hi - lo) * (i + 0.5) / k)) for i in range(k)]


def _inputs(case, seed):
    gen, kind = _generator(seed), case["kind"]
    s = {"case": dict(case)}
    if kind == "tree":
        s["t"] = _tree(case["n"], gen)
    elif kind == "tree_batch":
        s["t"] = [_tree(n, gen) for n in _sizes(case)]
    elif kind == "sssp_batch":
        s["g"] = [_graph(n, n * case["degree"], gen) for n in _sizes(case)]
        s["w"] = [_weights(g.m, gen) for g in s["g"]]
        s["src"] = [_source(g, gen) for g in s["g"]]
    elif kind == "color":
        s["g"] = _symmetric(case["n"], case["n"] * case["degree"], gen)
        s["prio"] = torch.randint(-(1 << 31), 1 << 31, (case["n"],), dtype=torch.int64, device="cuda",
                                  generator=gen).to(torch.int32)
    else:
        n = case["n"]
        s["g"] = _graph(n, n * case["degree"], gen)
        if kind == "spmv":
            s["val"], s["x"] = _uniform(s["g"].m, gen), _uniform(n, gen)
        elif kind == "pagerank":  # g holds the in-edges
            s["deg"] = torch.bincount(s["g"].col.to(torch.int64), minlength=n).to(torch.int32)
        else:
            s["w"] = _weights(s["g"].m, gen)
            s["src"] = _source(s["g"], gen)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["kind"] in ("tree_batch", "sssp_batch"):  # one result array, a slice for each instance
        sizes = _sizes(case)
        s["out"] = torch.empty(sum(sizes), dtype=torch.int32, device="cuda")
        s["outs"] = list(torch.split(s["out"], sizes))
    else:
        real = case["kind"] in ("spmv", "pagerank")
        s["out"] = torch.empty(case["n"], dtype=torch.float32 if real else torch.int32, device="cuda")
    s["ctx"] = context()
    return s


# ---- the calls -----------------------------------------------------------------------------------

def run(s):
    c, ctx, kind, mode = s["case"], s["ctx"], s["case"]["kind"], s["case"]["mode"]
    if kind == "spmv":
        return ctx.spmv(s["g"], s["val"], s["x"], mode=mode, out=s["out"])
    if kind == "sssp":
        return ctx.sssp(s["g"], s["w"], s["src"], mode=mode, out=s["out"])
    if kind == "bfs":
        return ctx.bfs(s["g"], s["src"], mode=mode, out=s["out"])
    if kind == "pagerank":
        return ctx.pagerank(s["g"], s["deg"], c["iterations"], mode=mode, out=s["out"])
    if kind == "color":
        return ctx.color(s["g"], s["prio"], mode=mode, out=s["out"])
    if kind == "tree":
        f = ctx.tree_descendants if c["op"] == "descendants" else ctx.tree_height
        return f(s["t"], mode=mode, out=s["out"])
    if kind == "tree_batch":
        f = ctx.tree_descendants_batch if c["op"] == "descendants" else ctx.tree_height_batch
        f(s["t"], mode=mode, outs=s["outs"])
        return s["out"]
    ctx.sssp_batch(s["g"], s["w"], s["src"], modes=[mode] * c["count"], outs=s["outs"])
    return s["out"]


def work(case):
    kind = case["kind"]
    if kind in ("tree", "tree_batch"):  # child ranges and child lists in, one number a node out
        n = case["n"] if kind == "tree" else sum(_sizes(case))
        return {"bytes": 12 * n, "flops": n}
    n = case["n"] if kind != "sssp_batch" else sum(_sizes(case))
    m = n * case["degree"]
    if kind == "spmv":
        return {"bytes": 8 * m + 12 * n, "flops": 2 * m}
    if kind == "bfs":
        return {"bytes": 4 * m + 8 * n, "flops": m}
    if kind == "pagerank":
        return {"bytes": case["iterations"] * (4 * m + 16 * n), "flops": case["iterations"] * (m + 4 * n)}
    if kind == "color":  # about 1.8 directed edges are left of each drawn edge
        return {"bytes": 4 * 1.8 * m + 12 * n, "flops": 1.8 * m}
    return {"bytes": 8 * m + 8 * n, "flops": m}


# ---- the same results in plain torch, 64 bits ----------------------------------------------------

def _rows(g):
    ptr = g.row_ptr.to(torch.int64)
    return torch.repeat_interleave(torch.arange(g.n, device="cuda"), ptr[1:] - ptr[:-1])


def _shortest(g, w, src):
    rows, cols = _rows(g), g.col.to(torch.int64)
    far = 1 << 40
    d = torch.full((g.n,), far, dtype=torch.int64, device="cuda")
    d[src] = 0
    while True:
        nd = d.scatter_reduce(0, cols, d[rows] + w, "amin")
        if torch.equal(nd, d):
            return torch.where(d >= far, -1, d)
        d = nd


def _subtrees(t, op):
    parent = t.parent.to(torch.int64)
    depth, at = torch.zeros(t.n, dtype=torch.int64, device="cuda"), torch.arange(t.n, device="cuda")
    while True:  # all nodes walk up together: a node's depth is the number of steps to the root
        at = torch.where(at >= 0, parent[at.clamp(min=0)], at)
        if not bool((at >= 0).any()):
            break
        depth += at >= 0
    out = torch.zeros(t.n, dtype=torch.int64, device="cuda")
    for d in range(int(depth.max()), 0, -1):
        v = torch.nonzero(depth == d).reshape(-1)
        if op == "descendants":
            out.scatter_add_(0, parent[v], out[v] + 1)
        else:
            out.scatter_reduce_(0, parent[v], out[v] + 1, "amax")
    return out


def _colors(g, prio):
    """color[v] = 0 without an outranking neighbour, else 1 + the largest color among those; -1 until it is known."""
    u, v = _rows(g), g.col.to(torch.int64)
    p = prio.to(torch.int64) & 0xFFFFFFFF
    above = (p[u] > p[v]) | ((p[u] == p[v]) & (u > v))
    u, v = u[above], v[above]  # u outranks v
    left = torch.bincount(v, minlength=g.n)
    color = torch.full((g.n,), -1, dtype=torch.int64, device="cuda")
    ready = torch.nonzero(left == 0).reshape(-1)
    order = torch.argsort(u, stable=True)
    u, v = u[order], v[order]
    first = torch.zeros(g.n + 1, dtype=torch.int64, device="cuda")
    first[1:] = torch.cumsum(torch.bincount(u, minlength=g.n), 0)
    r = 0
    while ready.numel():
        color[ready] = r
        count = first[ready + 1] - first[ready]
        at = torch.repeat_interleave(first[ready] - torch.cumsum(count, 0) + count, count)
        to = v[at + torch.arange(at.numel(), device="cuda")]
        left.scatter_add_(0, to, torch.full_like(to, -1))
        ready = torch.unique(to[left[to] == 0])
        r += 1
    return color


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "spmv":
        y = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
        return y.index_add_(0, _rows(s["g"]), s["val"].double() * s["x"].double()[s["g"].col.to(torch.int64)])
    if kind == "sssp":
        return _shortest(s["g"], s["w"].to(torch.int64), s["src"])
    if kind == "bfs":
        return _shortest(s["g"], 1, s["src"])
    if kind == "pagerank":
        n, d, deg = case["n"], 0.85, s["deg"].double()
        rows, cols = _rows(s["g"]), s["g"].col.to(torch.int64)
        rank = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
        for _ in range(case["iterations"]):
            give = torch.where(deg > 0, rank / deg.clamp(min=1), 0.0)
            got = torch.zeros_like(rank).index_add_(0, rows, give[cols])
            rank = (1 - d) / n + d * (got + rank[deg == 0].sum() / n)
        return rank
    if kind == "color":
        return _colors(s["g"], s["prio"])
    if kind == "tree":
        return _subtrees(s["t"], case["op"])
    if kind == "tree_batch":
        return torch.cat([_subtrees(t, case["op"]) for t in s["t"]])
    return torch.cat([_shortest(g, w.to(torch.int64), src) for g, w, src in zip(s["g"], s["w"], s["src"])])
