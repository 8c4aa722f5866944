"""PageRank at the edges of its row classes, and on a renumbered graph, against
the oracle: relative error 1e-12 (a row of 20,000 doubles summed in another
order is off by at most 20,000 x 2^-53 = 2e-12 of itself if every rounding
went one way, a few 1e-14 when they do not; a few iterations multiply that by
less than one)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu

LENGTHS = [1, 8, 9, 32, 33, 128, 129, 256, 257, 511, 512, 513, 1024, 8191, 8192, 8193, 16384, 20000]


def hubs_graph(copies: int, leaves: int, seed: int):
    """`copies` hubs of each length in LENGTHS, their neighbours drawn from `leaves` other vertices."""
    rng = np.random.default_rng(seed)
    src, dst, hub = [], [], leaves
    for length in LENGTHS * copies:
        src.append(np.full(length, hub))
        dst.append(rng.choice(leaves, length, replace=False))
        hub += 1
    return graphs.from_edges(hub, np.concatenate(src), np.concatenate(dst))


@pytest.mark.parametrize("block", [0, 128, 256, 512])
@pytest.mark.parametrize("copies,leaves", [(1, 20001), (3, 40000), (8, 420_000)])
@pytest.mark.parametrize("directed", [False, True])
def test_row_classes(copies, leaves, block, directed):
    # 420,000 leaves, most of them without edges: past the size and the skew at which vertices are renumbered
    from paper_2305_03317_amd import sp
    print(copies, leaves, block, directed, flush=True)
    rp, ci = hubs_graph(copies, leaves, 5)
    if directed:
        rp, ci = graphs.directed_from(rp, ci, 6)
    g = sp.sp_graph_upload(rp, ci, directed=directed)
    got = sp.sp_pagerank(g, 0.0, 0.85, 6, config=dict(block_size=block)).cpu().numpy()
    ref, _, diff = oracle.pagerank(rp, ci, 0.0, 0.85, 6, iterations=6)
    assert np.max(np.abs(got - ref) / ref) <= 1e-12
    assert abs(sp.sp_pagerank_get_last_stats()["diff"] - diff) <= 1e-12 + 1e-9 * diff
    again = sp.sp_pagerank(g, 0.0, 0.85, 6, config=dict(block_size=block, chunk_iters=-2)).cpu().numpy()
    assert np.array_equal(got, again)
    g.release()
