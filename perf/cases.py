"""Workloads that this framework's users run, one call (or one burst of served
requests) each: betweenness centrality on both paths, forward/backward levels,
SSSP, PageRank, triangle counting and serving, on the graph families of the
benchmark (uniform, RMAT, road-like), from 4,096 vertices to RMAT scale 22.

``listed()`` names the workloads; ``draw(rng)`` gives another of the same
ranges.  ``prepare`` builds a graph from the seed alone (on the GPU), uploads
it and draws sources; ``run`` is one call through the public entry points;
``exact`` is the same result in plain torch, binary64.

Every graph family follows the repository's own recipe (``graphs.py``): RMAT
with (0.57, 0.19, 0.19) and relabelled vertices, `edge_factor` draws per
vertex; road-like = the minimum spanning tree of a grid under random weights
plus 2% of the grid's edges; both directions stored, rows sorted, duplicates
and self-loops dropped.  An RMAT graph of n vertices, n not a power of two, is
the part of the next power of two's graph on n of its relabelled vertices.
"""
import math
import random

import torch

from paper_2305_03317_amd import sp

INT_MAX = 2**31 - 1


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # The smallest call: a few sources on a graph that fits the caches; launches and host checks count.
        dict(name="bc-uniform-4096", what="bc_batch", graph="uniform", n=4096, m=32768, sources=16),
        # The flagship: 1,024 sources on RMAT scale 22 (64 M edges), 16 grouped multi-source passes.
        dict(name="bc-rmat-22", what="bc_batch", graph="rmat", n=1 << 22, edge_factor=16, sources=1024),
        # A road network: thousands of small levels, one workgroup per source.
        dict(name="bc-road-2048", what="bc_batch", graph="road", width=2048, sources=64),
        # A directed graph (both row directions are read), one multi-source pass.
        dict(name="bc-directed-rmat-18", what="bc_batch", graph="rmat", n=1 << 18, edge_factor=16, sources=64,
             directed=True),
        # The per-source path, which callers use that want the paper's sums and source order as written.
        dict(name="bc-source-rmat-20", what="bc", graph="rmat", n=1 << 20, edge_factor=16, sources=16),
        # One source, forward and backward, on a ragged mid-size graph: distances, path counts, dependencies.
        dict(name="levels-rmat-200k", what="levels", graph="rmat", n=200_003, edge_factor=16),
        # Shortest paths on the skewed graph (few heavy rounds) and on a road grid of odd width (many light ones).
        dict(name="sssp-rmat-22", what="sssp", graph="rmat", n=1 << 22, edge_factor=16),
        dict(name="sssp-road-1501", what="sssp", graph="road", width=1501),
        # PageRank, 20 iterations at full size, and a small graph run with the defaults until it converges.
        dict(name="pagerank-rmat-22", what="pagerank", graph="rmat", n=1 << 22, edge_factor=16, beta=0.0, iters=20),
        dict(name="pagerank-rmat-15", what="pagerank", graph="rmat", n=1 << 15, edge_factor=16, beta=1e-6, iters=100),
        # Triangles of the benchmark graph.
        dict(name="triangles-rmat-22", what="triangles", graph="rmat", n=1 << 22, edge_factor=16, per_vertex=False),
        # A burst of requests over three resident graphs through the server.
        dict(name="serve-burst-24", what="serve", graph="mix", scale_a=16, scale_b=18, width=512, requests=24,
             most=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case: the work by its share of use, sizes log-uniform over each path's range."""
    what = rng.choice(["bc_batch", "bc_batch", "bc_road", "bc", "levels", "sssp", "sssp_road", "pagerank", "pagerank",
                       "triangles", "serve"])
    ef = rng.choice([8, 16, 16, 24])
    if what == "bc_batch":
        if rng.random() < 0.25:
            n = _log_int(rng, 4096, 300_000)
            return dict(what="bc_batch", graph="uniform", n=n, m=8 * n, sources=_log_int(rng, 4, 256))
        c = dict(what="bc_batch", graph="rmat", n=_log_int(rng, 4096, 1 << 22), edge_factor=min(ef, 16),
                 sources=_log_int(rng, 16, 512))
        if rng.random() < 0.25:
            c.update(n=_log_int(rng, 4096, 1 << 18), directed=True)
        return c
    if what == "bc_road":
        return dict(what="bc_batch", graph="road", width=_log_int(rng, 128, 2000), sources=_log_int(rng, 8, 64))
    if what == "bc":
        return dict(what="bc", graph="rmat", n=_log_int(rng, 4096, 1 << 21), edge_factor=ef, sources=_log_int(rng, 4, 32))
    if what == "levels":
        return dict(what="levels", graph="rmat", n=_log_int(rng, 4096, 1 << 22), edge_factor=min(ef, 16))
    if what == "sssp":
        return dict(what="sssp", graph="rmat", n=_log_int(rng, 8192, 1 << 22), edge_factor=min(ef, 16))
    if what == "sssp_road":
        return dict(what="sssp", graph="road", width=_log_int(rng, 128, 3000))
    if what == "pagerank":
        c = dict(what="pagerank", graph="rmat", n=_log_int(rng, 8192, 1 << 22), edge_factor=min(ef, 16), beta=1e-6,
                 iters=rng.randint(10, 100))
        if rng.random() < 0.3:
            c = dict(what="pagerank", graph="road", width=_log_int(rng, 128, 2500), beta=1e-6, iters=rng.randint(10, 60))
        return c
    if what == "triangles":
        return dict(what="triangles", graph="rmat", n=_log_int(rng, 8192, 1 << 22), edge_factor=min(ef, 16),
                    per_vertex=rng.random() < 0.5)
    return dict(what="serve", graph="mix", scale_a=rng.randint(13, 16), scale_b=rng.randint(17, 18),
                width=_log_int(rng, 128, 600), requests=rng.randint(4, 32), most=rng.randint(32, 160))


# ---------------------------------------------------------------------------
# Graphs, built on the GPU from a seed
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1_000_003 + 17)
    return g


def _csr(n, u, v, directed=False):
    """Sorted simple CSR (int32 row offsets, int32 ids) of the edges u-v."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = u * n + v if directed else torch.cat([u * n + v, v * n + u])
    key = torch.unique(key)
    row = torch.div(key, n, rounding_mode="floor")
    ci = (key - row * n).to(torch.int32)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return rp.to(torch.int32), ci


def _uniform(n, m, gen):
    k = m + m // 8 + 64
    u = torch.randint(n, (k,), generator=gen, device="cuda")
    v = torch.randint(n, (k,), generator=gen, device="cuda")
    ok = u != v
    key = torch.unique(torch.minimum(u, v)[ok] * n + torch.maximum(u, v)[ok])
    key = key[torch.randperm(key.numel(), generator=gen, device="cuda")[:m]]
    a = torch.div(key, n, rounding_mode="floor")
    return _csr(n, a, key - a * n)


def _rmat(n, edge_factor, gen, directed=False):
    scale = max(1, (n - 1).bit_length())
    draws = edge_factor << scale
    u = torch.zeros(draws, dtype=torch.int32, device="cuda")
    v = torch.zeros(draws, dtype=torch.int32, device="cuda")
    for _ in range(scale):
        r = torch.rand(draws, generator=gen, device="cuda")
        u = u * 2 + (r >= 0.76)
        v = v * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(1 << scale, generator=gen, device="cuda")
    u, v = perm[u.long()], perm[v.long()]
    if n < (1 << scale):
        keep = (u < n) & (v < n)
        u, v = u[keep], v[keep]
    if directed:  # each undirected edge once, its direction by a coin
        ok = u != v
        key = torch.unique(torch.minimum(u, v)[ok] * n + torch.maximum(u, v)[ok])
        a = torch.div(key, n, rounding_mode="floor")
        b = key - a * n
        flip = torch.rand(key.numel(), generator=gen, device="cuda") < 0.5
        u, v = torch.where(flip, b, a), torch.where(flip, a, b)
    return _csr(n, u, v, directed)


def _road(width, gen):
    """The grid's minimum spanning tree under distinct random weights (Boruvka rounds), plus 2% of its edges."""
    n = width * width
    at = torch.arange(n, device="cuda")
    right, down = at[at % width != width - 1], at[: n - width]
    eu = torch.cat([right, down])
    ev = torch.cat([right + 1, down + width])
    m = eu.numel()
    weight = torch.randperm(m, generator=gen, device="cuda")
    edge_of = torch.empty_like(weight)
    edge_of[weight] = torch.arange(m, device="cuda")
    tree = torch.zeros(m, dtype=torch.bool, device="cuda")
    comp = at.clone()
    live = torch.arange(m, device="cuda")
    while True:
        cu, cv = comp[eu[live]], comp[ev[live]]
        cross = cu != cv
        live, cu, cv = live[cross], cu[cross], cv[cross]
        if live.numel() == 0:
            break
        best = torch.full((n,), m, dtype=torch.int64, device="cuda")
        best.scatter_reduce_(0, cu, weight[live], "amin")
        best.scatter_reduce_(0, cv, weight[live], "amin")
        c = torch.nonzero(best < m).squeeze(1)
        e = edge_of[best[c]]
        tree[e] = True
        a, b = comp[eu[e]], comp[ev[e]]
        up = at.clone()
        up[c] = torch.where(a == c, b, a)
        both = (up[up] == at) & (at < up)  # two components that chose the same edge: the lower one stays the root
        up[both] = at[both]
        while True:
            nxt = up[up]
            if torch.equal(nxt, up):
                break
            up = nxt
        comp = up[comp]
    rest = torch.nonzero(~tree).squeeze(1)
    extra = rest[torch.randperm(rest.numel(), generator=gen, device="cuda")[: int(0.02 * m)]]
    pick = torch.cat([torch.nonzero(tree).squeeze(1), extra])
    return _csr(n, eu[pick], ev[pick])


def _graph(case, gen):
    if case["graph"] == "uniform":
        return _uniform(case["n"], case["m"], gen)
    if case["graph"] == "road":
        return _road(case["width"], gen)
    return _rmat(case["n"], case["edge_factor"], gen, bool(case.get("directed")))


def _sources(rp, count, gen):
    """Distinct vertices with at least one edge, as a host list (what the entry points take)."""
    cand = torch.nonzero(rp[1:] > rp[:-1]).squeeze(1)
    at = torch.randperm(cand.numel(), generator=gen, device="cuda")[:count]
    return cand[at].cpu().numpy().astype("int32")


def _rows(rp):
    deg = (rp[1:] - rp[:-1]).long()
    return torch.repeat_interleave(torch.arange(deg.numel(), device="cuda"), deg)


def _weights(rp, ci, seed):
    """Uniform on [1, 100], equal in both directions of an edge (a hash of the edge and the seed)."""
    u, v = _rows(rp), ci.long()
    x = torch.minimum(u, v) * (rp.numel() - 1) + torch.maximum(u, v) + int(seed) * 7_919
    for k in (0x2545F4914F6CDD1D, 0x5851F42D4C957F2D):
        x = x * k + 1_442_695_040_888_963_407
        x = x ^ ((x >> 29) & 0x7FFFFFFFF)
    return (((x >> 20) & 0x7FFFFFFF) % 100 + 1).to(torch.int32)


def _requests(case, rps, gen):
    """(graph, sources) of each request: the graph uniform, the source count log-uniform on 1..most (both by the
    case, so that every seed asks for the same amount of work); the sources by the seed."""
    r, out = random.Random(case["requests"] * 1000 + case["most"]), []
    for _ in range(case["requests"]):
        gi = r.randrange(len(rps))
        out.append((gi, _sources(rps[gi], max(1, int(math.exp(r.uniform(0, math.log(case["most"] + 1))))), gen)))
    return out


def _mix(case, gen):
    return [_rmat(1 << case["scale_a"], 16, gen), _rmat(1 << case["scale_b"], 16, gen), _road(case["width"], gen)]


class _Serving:
    """A server with its resident graphs; ends the server before its graphs go."""

    def __init__(self, graphs):
        self.graphs = [sp.sp_graph_upload(rp, ci) for rp, ci in graphs]
        self.server = sp.sp_server_create(memory_budget=24 << 30)
        self.ids = [self.server.add_graph(g) for g in self.graphs]

    def __del__(self):
        self.server.destroy()


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    gen = _gen(seed)
    s = dict(case)
    if case["what"] == "serve":
        graphs = _mix(case, gen)
        s["reqs"] = _requests(case, [rp for rp, _ in graphs], gen)
        s["serving"] = _Serving(graphs)
        s["outs"] = [torch.empty(graphs[gi][0].numel() - 1, dtype=torch.float64, device="cuda") for gi, _ in s["reqs"]]
        torch.cuda.synchronize()
        return s
    rp, ci = _graph(case, gen)
    g = s["g"] = sp.sp_graph_upload(rp, ci, directed=bool(case.get("directed")))
    if case["what"] == "sssp":
        sp.sp_graph_set_weights(g, _weights(rp, ci, seed))
    if case["what"] in ("bc", "bc_batch", "levels", "sssp"):
        s["src"] = _sources(rp, case.get("sources", 1), gen)
    if case["what"] in ("bc", "bc_batch", "pagerank"):
        s["out"] = torch.empty(g.n, dtype=torch.float64, device="cuda")
    elif case["what"] == "sssp":
        s["out"] = torch.empty(g.n, dtype=torch.int32, device="cuda")
    return s


def run(s):
    what = s["what"]
    if what == "bc_batch":
        return sp.sp_bc_batch(s["g"], s["src"], s["out"])[0]
    if what == "bc":
        return sp.sp_bc(s["g"], s["src"], s["out"])[0]
    if what == "levels":
        dist, sigma, delta, _ = sp.sp_bfs_levels(s["g"], int(s["src"][0]), with_sigma=True, with_delta=True)
        return dist, sigma, delta
    if what == "sssp":
        return sp.sp_sssp(s["g"], int(s["src"][0]), s["out"])
    if what == "pagerank":
        return sp.sp_pagerank(s["g"], s["beta"], 0.85, s["iters"], s["out"])
    if what == "triangles":
        count, per = sp.sp_triangle_count(s["g"], per_vertex=s["per_vertex"])
        return (count, per) if s["per_vertex"] else count
    srv = s["serving"]
    reqs = [srv.server.submit(srv.ids[gi], src, out) for (gi, src), out in zip(s["reqs"], s["outs"])]
    for r in reqs:
        r.wait()
        r.release()
    return s["outs"]


def _sizes(case):
    """(vertices, CSR entries) of the case's graph, by its recipe."""
    if case["graph"] == "uniform":
        return case["n"], 2 * case["m"]
    if case["graph"] == "road":
        n = case["width"] ** 2
        return n, int(2 * (n - 1 + 0.04 * n))
    full = 1 << max(1, (case["n"] - 1).bit_length())
    nnz = 2 * 0.95 * case["edge_factor"] * full * (case["n"] / full) ** 2
    return case["n"], int(nnz / 2 if case.get("directed") else nnz)


def work(case):
    """Each input read once and the outputs written once; the arithmetic that every (source, edge) pair needs."""
    what = case["what"]
    if what == "serve":
        sizes = [(1 << case["scale_a"], 30 << case["scale_a"]), (1 << case["scale_b"], 30 << case["scale_b"]),
                 (case["width"] ** 2, 2 * case["width"] ** 2)]
        each = (case["most"] - 1) / math.log(case["most"] + 1)  # mean sources of a request
        byte = sum(4 * e + 4 * v for v, e in sizes) + case["requests"] / 3 * sum(8 * v for v, _ in sizes)
        return dict(bytes=byte, flops=case["requests"] / 3 * each * sum(4 * e for _, e in sizes))
    v, e = _sizes(case)
    graph = 4 * (v + 1) + 4 * e
    if what in ("bc", "bc_batch"):
        rows = 2 if case.get("directed") else 1
        return dict(bytes=rows * graph + 8 * v, flops=4 * e * case["sources"])
    if what == "levels":
        return dict(bytes=graph + 20 * v, flops=4 * e)
    if what == "sssp":
        return dict(bytes=4 * v + 8 * e + 4 * v, flops=e)
    if what == "pagerank":  # every iteration reads the rows and the last values and writes new ones
        k = case["iters"] if case["beta"] == 0 else min(case["iters"], 20)
        return dict(bytes=k * (graph + 16 * v), flops=k * 2 * e)
    return dict(bytes=graph + (8 * v if case["per_vertex"] else 0), flops=e)


# ---------------------------------------------------------------------------
# The same results in plain torch, 64 bits
# ---------------------------------------------------------------------------
class _RowSums:
    """Sums over the rows of a CSR, by pieces of 128 entries first (no long chain of additions to one address)."""

    def __init__(self, rp, ci):
        self.n, self.row, self.col = rp.numel() - 1, _rows(rp), ci.long()
        deg = (rp[1:] - rp[:-1]).long()
        pieces = (deg + 127) // 128
        first = torch.cumsum(pieces, 0) - pieces
        self.piece = first[self.row] + (torch.arange(ci.numel(), device="cuda") - rp.long()[self.row]) // 128
        self.piece_row = torch.repeat_interleave(torch.arange(self.n, device="cuda"), pieces)

    def sums(self, x, at=None):
        """Per row, the sum of x over its entries (all, or those numbered `at`, ascending)."""
        part = torch.zeros(self.piece_row.numel(), dtype=torch.float64, device="cuda")
        part.index_add_(0, self.piece if at is None else self.piece[at], x)
        return torch.zeros(self.n, dtype=torch.float64, device="cuda").index_add_(0, self.piece_row, part)


def _reversed(rp, ci):
    n = rp.numel() - 1
    key = torch.sort(ci.long() * n + _rows(rp))[0]
    row = torch.div(key, n, rounding_mode="floor")
    back = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    back[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return back, key - row * n


def _brandes(out, inc, src):
    """dist, sigma, delta of one source; every level looks at every entry (few levels)."""
    n = out.n
    dist = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    sigma = torch.zeros(n, dtype=torch.float64, device="cuda")
    dist[src], sigma[src] = 0, 1.0
    level = 0
    while True:
        at = torch.nonzero((dist[inc.col] == level) & (dist[inc.row] < 0)).squeeze(1)
        if at.numel() == 0:
            break
        level += 1
        dist[inc.row[at]] = level
        sigma += inc.sums(sigma[inc.col[at]], at)
    delta = torch.zeros(n, dtype=torch.float64, device="cuda")
    for lv in range(level - 1, 0, -1):
        at = torch.nonzero((dist[out.row] == lv) & (dist[out.col] == lv + 1)).squeeze(1)
        v, w = out.row[at], out.col[at]
        delta += out.sums((sigma[v] / sigma[w]) * (1.0 + delta[w]), at)
    return dist, sigma, delta


def _bc_rows(rp, ci, src, directed=False):
    out = _RowSums(rp, ci)
    inc = _RowSums(*_reversed(rp, ci)) if directed else out
    bc = torch.zeros(out.n, dtype=torch.float64, device="cuda")
    for s in src:
        bc += _brandes(out, inc, int(s))[2]
    return bc


def _bc_road(rp, ci, src):
    """BC of a graph of short rows: all sources together, each level only its frontier (many levels)."""
    n, k = rp.numel() - 1, len(src)
    deg = (rp[1:] - rp[:-1]).long()
    width = int(deg.max())
    nb = torch.full((n, width), -1, dtype=torch.int64, device="cuda")
    row = _rows(rp)
    nb[row, torch.arange(ci.numel(), device="cuda") - rp.long()[row]] = ci.long()
    dist = torch.full((k * n,), -1, dtype=torch.int32, device="cuda")
    mark = torch.zeros(k * n, dtype=torch.int32, device="cuda")
    sigma = torch.zeros(k * n, dtype=torch.float64, device="cuda")
    front = torch.arange(k, device="cuda") * n + torch.as_tensor(src, device="cuda").long()
    dist[front], sigma[front] = 0, 1.0
    level, fronts = 0, [front]

    def edges(f):
        w = nb[f % n]
        u = f.unsqueeze(1).expand_as(w)[w >= 0]
        return u, u - u % n + w[w >= 0]

    while True:
        u, w = edges(front)
        new = w[dist[w] < 0]
        if new.numel() == 0:
            break
        dist[new] = level + 1
        at = torch.arange(new.numel(), dtype=torch.int32, device="cuda")
        mark[new] = at
        front = new[mark[new] == at]
        down = dist[w] == level + 1
        sigma.index_add_(0, w[down], sigma[u[down]])
        fronts.append(front)
        level += 1
    delta = torch.zeros(k * n, dtype=torch.float64, device="cuda")
    for lv in range(level - 1, 0, -1):
        u, w = edges(fronts[lv])
        down = dist[w] == lv + 1
        u, w = u[down], w[down]
        delta.index_add_(0, u, (sigma[u] / sigma[w]) * (1.0 + delta[w]))
    return delta.view(k, n).sum(0)


def _sssp(rp, ci, w, src):
    n = rp.numel() - 1
    start, deg = rp[:-1].long(), (rp[1:] - rp[:-1]).long()
    dist = torch.full((n,), INT_MAX, dtype=torch.int64, device="cuda")
    dist[src] = 0
    front = torch.tensor([src], device="cuda")
    while front.numel():
        d = deg[front]
        first = torch.cumsum(d, 0) - d
        own = torch.repeat_interleave(torch.arange(front.numel(), device="cuda"), d)
        e = start[front][own] + torch.arange(own.numel(), device="cuda") - first[own]
        to, nd = ci[e].long(), dist[front][own] + w[e]
        better = nd < dist[to]
        to, nd = to[better], nd[better]
        dist.scatter_reduce_(0, to, nd, "amin")
        front = torch.unique(to)
    return dist.to(torch.int32)


def _pagerank(rp, ci, beta, iters):
    rows = _RowSums(rp, ci)
    deg = (rp[1:] - rp[:-1]).double()
    pr = torch.full((rows.n,), 1.0 / rows.n, dtype=torch.float64, device="cuda")
    for _ in range(iters):
        share = torch.where(deg > 0, pr / deg.clamp(min=1.0), 0.0)
        val = rows.sums(share[rows.col]) * 0.85 + 0.15 / rows.n
        diff = float((val - pr).abs().sum())
        pr = val
        if not diff > beta:
            break
    return pr


def _triangles(rp, ci):
    """(count, per-vertex counts): pairs of each vertex's higher-ranked neighbours, tested against the edge list."""
    n = rp.numel() - 1
    deg = (rp[1:] - rp[:-1]).long()
    row, col = _rows(rp), ci.long()
    up = (deg[row] < deg[col]) | ((deg[row] == deg[col]) & (row < col))
    u, v = row[up], col[up]
    keys = u * n + v  # ascending: rows and their entries are sorted
    out = torch.bincount(u, minlength=n)
    off = torch.cumsum(out, 0) - out
    per = torch.zeros(n, dtype=torch.int64, device="cuda")
    total, step = 0, 1 << 27
    load = torch.cumsum(out[v], 0)  # an entry (u, v) tests u against every w that v points to
    if load.numel() == 0:
        return 0, per
    cuts = torch.searchsorted(load, torch.arange(0, int(load[-1]) + step, step, device="cuda")).tolist()
    for a, b in zip(cuts, cuts[1:] + [u.numel()]):
        uu, vv = u[a:b], v[a:b]
        k = out[vv]
        own = torch.repeat_interleave(torch.arange(b - a, device="cuda"), k)
        first = torch.cumsum(k, 0) - k
        ww = v[off[vv][own] + torch.arange(own.numel(), device="cuda") - first[own]]
        want = uu[own] * n + ww
        at = torch.searchsorted(keys, want).clamp(max=keys.numel() - 1)
        hit = keys[at] == want
        total += int(hit.sum())
        for x in (uu[own], vv[own], ww):
            per += torch.bincount(x[hit], minlength=n)
    return total, per


def exact(case, seed):
    gen = _gen(seed)
    what = case["what"]
    if what == "serve":
        graphs = _mix(case, gen)
        return [(_bc_road if gi == 2 else _bc_rows)(*graphs[gi], src)
                for gi, src in _requests(case, [rp for rp, _ in graphs], gen)]
    v, e = _sizes(case)
    if what in ("bc", "bc_batch"):
        road = case["graph"] == "road"
        if (v * case["sources"] > 1 << 28) if road else (e * case["sources"] > 1 << 32 or case["sources"] > 300):
            return None
        rp, ci = _graph(case, gen)
        src = _sources(rp, case["sources"], gen)
        return _bc_road(rp, ci, src) if road else _bc_rows(rp, ci, src, bool(case.get("directed")))
    if what == "triangles" and e > 40_000_000:
        return None
    rp, ci = _graph(case, gen)
    if what == "levels":
        rows = _RowSums(rp, ci)
        return _brandes(rows, rows, int(_sources(rp, 1, gen)[0]))
    if what == "sssp":
        return _sssp(rp, ci, _weights(rp, ci, seed), int(_sources(rp, 1, gen)[0]))
    if what == "pagerank":
        return _pagerank(rp, ci, case["beta"], case["iters"])
    count, per = _triangles(rp, ci)
    return (count, per) if case["per_vertex"] else count
