"""The one-workgroup-per-source engine over fixed-width rows of an undirected
graph at the edges of what it holds on the chip: levels beyond its frontier
buffer, more shared children than its list, levels beyond 16-bit positions.
Against the oracle (distances and path counts exact, dependencies and BC to
1e-9 relative and zero where the oracle is zero, the bar of the parity
tests)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu


def tree(k: int, depth: int):
    n = sum(k ** i for i in range(depth + 1))
    child = np.arange(1, n)
    return n, (child - 1) // k, child


def make(name: str):
    if name == "tree-3":  # rows of 4, levels of up to 177,147
        return graphs.from_edges(*tree(3, 11))
    if name == "tree-7":  # rows of 8, levels of up to 117,649
        return graphs.from_edges(*tree(7, 6))
    # a tree whose leaves start layers of m vertices, each vertex of a layer with k parents in the one before
    k, fan, depth, layers = (2, 3, 7, 6) if name == "layers-4" else (4, 3, 7, 4)
    n, src, dst = tree(fan, depth)
    m = fan ** depth
    i = np.arange(m)
    src, dst = [src], [dst]
    for layer in range(layers):
        for j in range(k):
            src.append(n - m + layer * m + i)
            dst.append(n + layer * m + (i + j) % m)
    return graphs.from_edges(n + layers * m, np.concatenate(src), np.concatenate(dst))


def close(got, ref):
    zero = ref == 0
    assert np.all(got[zero] == 0)
    assert np.max(np.abs(got[~zero] - ref[~zero]) / np.abs(ref[~zero]), initial=0.0) <= 1e-9


@pytest.mark.parametrize("name,width", [("tree-3", 4), ("tree-7", 8), ("layers-4", 4), ("layers-8", 8)])
@pytest.mark.parametrize("block", [128, 1024])
def test_rows(name, width, block):
    from paper_2305_03317_amd import sp
    print(name, block, flush=True)
    rp, ci = make(name)
    n = len(rp) - 1
    assert width // 2 < np.diff(rp).max() <= width
    src = np.array([0, n // 2, n - 1, 0, 1], np.int32)
    g = sp.sp_graph_upload(rp, ci)
    cfg = {"engine": sp.SP_ENGINE_BLOCKS, "block_size": block, "batch_width": 3}  # odd: cells * 8 bytes
    close(sp.sp_bc_batch(g, src, config=cfg)[0].cpu().numpy(), oracle.bc(rp, ci, src))
    assert sp.sp_get_last_stats()["engine"] == sp.SP_ENGINE_BLOCKS
    out = sp.sp_batch_levels(g, src[:3], with_delta=True, config=cfg)
    for k, s in enumerate(map(int, src[:3])):
        d, sg, dl = oracle.source_detail(rp, ci, s)
        ref = dl.copy()
        ref[s] = 0.0
        assert np.array_equal(out[0][k].cpu().numpy(), d) and np.array_equal(out[1][k].cpu().numpy(), sg)
        close(out[2][k].cpu().numpy(), ref)
    g.release()
