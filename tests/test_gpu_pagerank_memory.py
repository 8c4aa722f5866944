"""PageRank on a directed graph whose renumbered copy does not fit: the graph's
own rows serve, with the same results."""
from __future__ import annotations

import ast
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = r"""
import sys, numpy as np
sys.path.insert(0, %r)
from oracle import pagerank
from paper_2305_03317_amd import graphs, sp
rp, ci = graphs.directed_from(*graphs.rmat(19, 10, seed=6), seed=7)
g = sp.sp_graph_upload(rp, ci, directed=True)
before = sp.sp_graph_info(g)["device_bytes"]
got = sp.sp_pagerank(g, 0.0, 0.85, 6).cpu().numpy()
want = pagerank(rp, ci, 0.0, 0.85, 6)[0]
assert np.max(np.abs(got - want) / want) < 1e-11
print((len(rp) - 1, len(ci), sp.sp_graph_info(g)["device_bytes"] - before))
""" % ROOT


def run(**env) -> tuple:
    r = subprocess.run([sys.executable, "-c", CHILD], env=dict(os.environ, **env), capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, (r.stdout, r.stderr)
    return ast.literal_eval(r.stdout.strip().splitlines()[-1])


def test_copy_that_does_not_fit():
    n, nnz, with_copy = run()
    # the copy shares a block with 16 bytes a vertex; the iterations take 32 bytes a vertex, the upload 4 an arc
    limit = 8 * n + 4 * nnz
    assert limit > 32 * n
    n, nnz, without = run(SP_TEST_FAIL_ALLOC_OVER=str(limit))
    assert with_copy - without >= 4 * nnz
