"""Weights replaced again and again on one graph, queries between some of the
replacements only: captured rounds must never run on the arrays of earlier
weights.  On a graph that is numbered by rank (over 2^20 vertices, skewed), on
one whose rows are kept at a fixed width, and on one that is neither.  Distances
bit for bit against the Dijkstra oracle; allocations of the same and other sizes
in between move the addresses that the allocator gives out."""
from __future__ import annotations

import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# Weights, a query (which keeps its workspace), other weights: whatever allocation of
# the second call fails, the graph answers by the weights that the status promises.
CHILD = r"""
import sys, numpy as np
sys.path.insert(0, %r)
import oracle
from paper_2305_03317_amd import graphs, sp
rp, ci = graphs.rmat(12, 16, seed=4)
rp = np.concatenate([rp, np.full(1_100_000 - 4096, rp[-1], np.int32)])   # numbered by rank
a, b = graphs.weights(rp, ci, 1), graphs.weights(rp, ci, 2)
s = int(graphs.sources(rp, 1, 7, min_degree=1)[0])
g = sp.sp_graph_upload(rp, ci)
sp.sp_graph_set_weights(g, a)
assert np.array_equal(sp.sp_sssp(g, s).cpu().numpy(), oracle.sssp(rp, ci, a, s))
try:
    sp.sp_graph_set_weights(g, b)
    now = b
except sp.SpError as e:
    assert e.status == sp.SP_ERR_OUT_OF_MEMORY, e
    now = a
for cfg in ({}, {"direction": 2}):
    assert np.array_equal(sp.sp_sssp(g, s, config=cfg).cpu().numpy(), oracle.sssp(rp, ci, now, s))
print("old" if now is a else "new")
""" % ROOT


def make(name: str):
    if name == "road":
        return graphs.road(90, 0.02, seed=3)
    rp, ci = graphs.rmat(14, 16, seed=4)
    if name == "rmat":
        return rp, ci
    return np.concatenate([rp, np.full(1_100_000 - 16384, rp[-1], np.int32)]), ci  # "ranked"


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


def test_failed_replacement_leaves_the_earlier_weights():
    seen = []
    for after in range(20, 27):  # 20 allocations come before the second call
        env = dict(os.environ, SP_TEST_FAIL_ALLOC_AFTER=str(after))
        r = subprocess.run([sys.executable, "-c", CHILD], env=env, capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, (after, r.stdout, r.stderr)
        print(after, r.stdout.strip(), flush=True)
        seen.append(r.stdout.split()[-1])
    assert seen[0] == "old" and seen[-1] == "new"
