"""Weights replaced again and again on one graph, queries between some of the
replacements only: captured rounds must never run on the arrays of earlier
weights.  On a graph that is numbered by rank (over 2^18 vertices, skewed), on
one whose rows are kept at a fixed width, and on one that is neither.  Distances
bit for bit against the Dijkstra oracle; allocations of the same and other sizes
in between move the addresses that the allocator gives out."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu


def make(name: str):
    if name == "road":
        return graphs.road(90, 0.02, seed=3)
    rp, ci = graphs.rmat(14, 16, seed=4)
    if name == "rmat":
        return rp, ci
    return np.concatenate([rp, np.full(300_000 - 16384, rp[-1], np.int32)]), ci  # "ranked"


@pytest.mark.parametrize("name", ["ranked", "road", "rmat"])
@pytest.mark.parametrize("cfg", [{}, {"direction": 2}, {"alpha": 20.0}])
def test_queries_between_weights(name, cfg):
    import torch

    from paper_2305_03317_amd import sp
    print(name, cfg, flush=True)
    rp, ci = make(name)
    s = int(graphs.sources(rp, 1, 7, min_degree=1)[0])
    g = sp.sp_graph_upload(rp, ci)
    others = []
    for k in range(12):
        w = graphs.weights(rp, ci, 100 + k)
        sp.sp_graph_set_weights(g, w)
        if k % 3 == 1:  # a graph of the same size takes what was freed
            o = sp.sp_graph_upload(rp, ci)
            sp.sp_graph_set_weights(o, w)
            others.append(o)
        if k in (0, 2, 3, 6, 9, 11):
            for _ in range(2):
                assert np.array_equal(sp.sp_sssp(g, s, config=cfg).cpu().numpy(), oracle.sssp(rp, ci, w, s)), k
        if k % 4 == 3 and others:
            others.pop(0).release()
    torch.cuda.synchronize()
    for o in others:
        o.release()
    g.release()
