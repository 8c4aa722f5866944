"""SSSP against the Dijkstra oracle, bit for bit, where the push kernels' rows and
rings have their edges: fixed-width rows of 4 and 8, fan-outs that overflow a
wave's ring, rows across a wave's 256-entry steps and on both sides of a hub's
256, and a graph large and skewed enough to be numbered by rank."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu


def tree(arity: int, levels: int):
    """Every vertex of a level has `arity` children: rows of arity + 1."""
    n = (arity**levels - 1) // (arity - 1)
    child = np.arange(1, n)
    return graphs.from_edges(n, (child - 1) // arity, child)


def make(name: str):
    if name.startswith("tree"):
        arity = int(name[4:])
        return tree(arity, {3: 9, 7: 6}[arity])
    if name == "road":
        return graphs.road(73, 0.02, seed=3)
    if name == "path":
        return graphs.from_edges(3000, np.arange(2999), np.arange(1, 3000))
    rng = np.random.default_rng(9)
    if name == "stars":  # rows of 1, 63..65, 255..257, 511..513, 1025
        sizes = [1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1025] * 3
        src = np.concatenate([np.full(k, 5000 + i) for i, k in enumerate(sizes)])
        dst = np.concatenate([rng.choice(5000, k, replace=False) for k in sizes])
        return graphs.from_edges(5000 + len(sizes), src, dst)
    rp, ci = graphs.rmat(15, 16, seed=4)  # "ranked": isolated vertices up to 300,000 in all
    return np.concatenate([rp, np.full(300_000 - 32768, rp[-1], np.int32)]), ci


@pytest.mark.parametrize("name", ["tree3", "tree7", "road", "path", "stars", "ranked"])
@pytest.mark.parametrize("cfg", [{}, {"block_size": 512, "chunk_rounds": -3}, {"local_hops": 1}, {"local_hops": -1},
                                 {"max_blocks": 1, "block_size": 128}, {"direction": 2}])
def test_rows(name, cfg):
    from paper_2305_03317_amd import sp
    print(name, cfg, flush=True)
    rp, ci = make(name)
    w = graphs.weights(rp, ci, 12)
    g = sp.sp_graph_upload(rp, ci)
    sp.sp_graph_set_weights(g, w)
    for s in [0, *map(int, graphs.sources(rp, 2, 7, min_degree=1))]:
        got = sp.sp_sssp(g, s, config=cfg).cpu().numpy()
        assert np.array_equal(got, oracle.sssp(rp, ci, w, s)), s
    g.release()
