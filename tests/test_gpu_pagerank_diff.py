"""The summed |change| that stops PageRank, against the change itself: the
outputs of k and of k - 1 iterations, subtracted and summed in binary64, whose
own error is under 1e-15 of a sum that is at most 1e-9 here.  The header gives
it as accurate to about 1e-15: at small sums too, where each share of it is far
below that."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu


def make(name: str):
    if name == "uniform":  # rows of 9 to 32 entries
        return graphs.uniform(1 << 18, 1 << 21, 3)
    if name == "sparse":
        return graphs.uniform(1 << 18, 1 << 19, 3)
    return graphs.rmat(19, 8, seed=4)  # renumbered, rows cut into pieces


@pytest.mark.parametrize("block", [0, 128])
@pytest.mark.parametrize("name,delta", [("uniform", 0.85), ("sparse", 0.6), ("rmat", 0.6)])
def test_small_sums(name, delta, block):
    from paper_2305_03317_amd import sp
    print(name, block, flush=True)
    rp, ci = make(name)
    g = sp.sp_graph_upload(rp, ci)
    cfg = dict(block_size=block)
    seen = 0
    before = sp.sp_pagerank(g, 0.0, delta, 19, config=cfg)
    for k in range(20, 80):
        now = sp.sp_pagerank(g, 0.0, delta, k, config=cfg)
        st = sp.sp_pagerank_get_last_stats()
        want = (now - before).abs().sum().item()
        before = now
        if st["iterations"] < k:
            break
        if want > 1e-9:
            continue
        assert abs(st["diff"] - want) <= 1e-15, (k, st["diff"], want)
        seen += want < 1e-13
    assert seen >= 3
    g.release()
