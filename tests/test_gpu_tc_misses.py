"""Triangle counting where most tests miss, and rows that a count refuses:
disjoint complete multipartite graphs, whose counts are known in closed form
(parts of `size` vertices: C(parts, 3) size^3 triangles a copy, C(parts - 1, 2)
size^2 at every vertex); a vertex's neighbours in another neighbour's part are
no triangles.  Integers, so exact.  The copies put vertex ranks on both sides of
65,536, 262,144 and 524,288, and rows on both sides of what one route or the
other takes."""
from __future__ import annotations

import math
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import sys, numpy as np
sys.path.insert(0, %r)
import oracle
from paper_2305_03317_amd import graphs, sp
rp, ci = graphs.uniform(8192, 800000, 5)
g = sp.sp_graph_upload(rp, ci)
for per in (True, False, True):
    total, each = sp.sp_triangle_count(g, per_vertex=per)
    assert total == oracle.triangles(rp, ci)
    assert not per or np.array_equal(each.cpu().numpy().astype(np.int64), oracle.triangles_each(rp, ci))
print("ok", sp.sp_graph_info(g))
""" % ROOT


def multipartite(parts: int, size: int, copies: int):
    """CSR of the disjoint copies; copy c holds the vertices c + j * copies, j in part j % parts."""
    k = parts * size
    j, c = np.divmod(np.arange(k * copies, dtype=np.int64), copies)
    of = np.arange(k, dtype=np.int64)
    rows = np.stack([of[of % parts != p] for p in range(parts)])
    ci = (rows[j % parts] * copies + c[:, None]).astype(np.int32).ravel()
    return (np.arange(k * copies + 1, dtype=np.int64) * (k - size)).astype(np.int32), ci


@pytest.mark.parametrize("parts,size,copies", [(3, 1, 5), (3, 5, 10), (2, 30, 3000), (3, 16, 700), (3, 24, 700),
                                               (3, 25, 700), (4, 20, 8000), (5, 40, 400), (3, 300, 30),
                                               (3, 2100, 1)])
def test_multipartite(parts, size, copies):
    import torch

    from paper_2305_03317_amd import sp
    print(parts, size, copies, flush=True)
    g = sp.sp_graph_upload(*multipartite(parts, size, copies))
    want = copies * math.comb(parts, 3) * size**3
    assert sp.sp_triangle_count(g)[0] == want
    total, per = sp.sp_triangle_count(g, per_vertex=True)
    assert total == want and torch.all(per.to(torch.int64) == math.comb(parts - 1, 2) * size**2).item()
    assert sp.sp_triangle_count(g)[0] == want
    g.release()


def stars(sizes, one_way):
    """Stars whose centres come first, and entries between centres stored one way only."""
    centres = len(sizes)
    src = np.concatenate([np.full(k, i) for i, k in enumerate(sizes)])
    rp, ci = graphs.from_edges(centres + sum(sizes), src, centres + np.arange(sum(sizes)))
    rows = [list(ci[rp[v]:rp[v + 1]]) for v in range(centres)]
    for u, v in one_way:
        rows[u] = sorted(rows[u] + [v])
    head = np.concatenate([np.array(r, np.int32) for r in rows])
    rest = ci[rp[centres]:]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows]), rp[centres + 1:] + len(one_way)]).astype(np.int32)
    return rp, np.concatenate([head, rest]).astype(np.int32)


@pytest.mark.parametrize("copies", [1, 200])
def test_one_way_entries_are_refused_whatever_order_they_rise_in(copies):
    """Two entries without their reverse, one from the higher of two centres of about equal degree and one from the
    lower: half of them rise by (degree, id), as in a simple graph."""
    from paper_2305_03317_amd import sp
    rp, ci = stars([261, 257, 300, 400] + [300] * copies, [(0, 1), (2, 3)])
    g = sp.sp_graph_upload(rp, ci)
    with pytest.raises(sp.SpError) as e:
        sp.sp_triangle_count(g)
    assert e.value.status == sp.SP_ERR_INVALID_ARGUMENT
    g.release()


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("name", ["flat", "light", "small", "shuffled flat", "shuffled small", "skewed"])
def test_routes_against_the_oracle(name, first):
    """Both kinds of count on one graph, in either order; rows in any order within a row."""
    import oracle
    from paper_2305_03317_amd import sp
    print(name, first, flush=True)
    kind = name.split()[-1]
    rp, ci = {"flat": lambda: graphs.uniform(6000, 60000, 3), "light": lambda: graphs.uniform(3000, 110000, 3),
              "small": lambda: graphs.rmat(11, 8, seed=5), "skewed": lambda: graphs.rmat(14, 16, seed=5)}[kind]()
    total, each = oracle.triangles(rp, ci), oracle.triangles_each(rp, ci)
    if name.startswith("shuffled"):
        rng = np.random.default_rng(4)
        ci = np.concatenate([rng.permutation(ci[rp[v]:rp[v + 1]]) for v in range(len(rp) - 1)]).astype(np.int32)
    g = sp.sp_graph_upload(rp, ci)
    for per in (first, not first, first):
        got, seen = sp.sp_triangle_count(g, per_vertex=per)
        assert got == total
        if per:
            assert np.array_equal(seen.cpu().numpy().astype(np.int64), each)
    assert sp.sp_tc_get_last_stats()["oriented_edges"] * 2 == len(ci)
    g.release()


def test_index_that_does_not_fit():
    """No allocation over 9 MB: the rows alone (6.4 MB) serve where the index (12.8 MB) does not fit."""
    env = dict(os.environ, SP_TEST_FAIL_ALLOC_OVER="9000000")
    r = subprocess.run([sys.executable, "-c", CHILD], env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.stdout, r.stderr)
