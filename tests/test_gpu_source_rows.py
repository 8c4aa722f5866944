"""The per-source path at the edges of its row classes and hub chunks, and on
rows numbered by rank, against the oracle (distances and path counts exact,
dependencies and BC to 1e-9 relative and zero where the oracle is zero, the
bar of the parity tests).  sp_bc_noalloc never renumbers, so where sp_bc does
the two must still agree bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu

LENGTHS = [1, 8, 9, 32, 33, 64, 255, 256, 257, 512, 513, 2048, 2049, 4096, 4097, 9000]


def make(name: str):
    rng = np.random.default_rng(21)
    if name == "classes":  # hubs of every length over 9,500 others, which a sparse graph joins
        src = np.concatenate([np.full(k, 9500 + i) for i, k in enumerate(LENGTHS)] + [rng.integers(0, 9500, 12000)])
        dst = np.concatenate([rng.choice(9500, k, replace=False) for k in LENGTHS] + [rng.integers(0, 9500, 12000)])
        return graphs.from_edges(9500 + len(LENGTHS), src, dst)
    if name == "deep":  # more levels than come back with the control block
        return graphs.from_edges(2000, np.arange(1999), np.arange(1, 2000))
    rp, ci = graphs.rmat(14, 16, seed=4)  # "ranked": isolated vertices up to 2^20 in all
    return np.concatenate([rp, np.full((1 << 20) - 16384, rp[-1], np.int32)]), ci


def close(got, ref):
    zero = ref == 0
    assert np.all(got[zero] == 0)
    assert np.max(np.abs(got[~zero] - ref[~zero]) / np.abs(ref[~zero]), initial=0.0) <= 1e-9


@pytest.mark.parametrize("name", ["classes", "deep", "ranked"])
@pytest.mark.parametrize("directed", [False, True])
def test_rows(name, directed):
    from paper_2305_03317_amd import sp
    print(name, directed, flush=True)
    rp, ci = make(name)
    if directed:
        rp, ci = graphs.directed_from(rp, ci, 6)
    src = graphs.sources(rp, 9, 7, min_degree=1)
    g = sp.sp_graph_upload(rp, ci, directed=directed)
    got = sp.sp_bc(g, src)[0].cpu().numpy()
    close(got, oracle.bc(rp, ci, src))
    assert np.array_equal(got, sp.sp_bc_noalloc(g, src)[0].cpu().numpy())
    for s in map(int, src[:2]):
        dist, sigma, delta, _ = sp.sp_bfs_levels(g, s, with_delta=True)
        d, sg, dl = oracle.source_detail(rp, ci, s)
        assert np.array_equal(dist.cpu().numpy(), d) and np.array_equal(sigma.cpu().numpy(), sg)
        ref = dl.copy()
        ref[s] = 0.0
        close(delta.cpu().numpy(), ref)
    close(sp.sp_bc_batch(g, src)[0].cpu().numpy(), oracle.bc(rp, ci, src))
    g.release()
