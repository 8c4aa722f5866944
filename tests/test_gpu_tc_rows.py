"""Triangle counting at the edges of its row and bitmap classes: disjoint
complete graphs, whose counts are known in closed form (C(k, 3) triangles a
clique, C(k - 1, 2) at every vertex).  Integers, so exact.

The sizes put oriented rows on both sides of 64 entries (sorted by a wave, or
by a block), of 256 (a row's degree class) and of 4,096 (per-vertex counts
kept in LDS), and vertex ranks on both sides of 65,536 (16-bit ids), 262,144
(counted with a bitmap) and 524,288 (rows sorted through a bitmap)."""
from __future__ import annotations

import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def cliques(k: int, count: int):
    """CSR of `count` disjoint K_k; clique c holds the vertices c + j * count."""
    n = k * count
    j, c = np.divmod(np.arange(n, dtype=np.int64), count)
    others = np.arange(k - 1, dtype=np.int64)[None, :] + (np.arange(k - 1)[None, :] >= j[:, None])
    ci = (others * count + c[:, None]).astype(np.int32).ravel()
    return (np.arange(n + 1, dtype=np.int64) * (k - 1)).astype(np.int32), ci


@pytest.mark.parametrize("k,count", [(2, 3), (31, 50), (33, 70), (64, 9), (65, 9), (66, 40), (130, 5000), (258, 300),
                                     (300, 3), (1025, 2), (4097, 1), (4200, 1)])
def test_cliques(k, count):
    import torch

    from paper_2305_03317_amd import sp
    print(k, count, flush=True)
    rp, ci = cliques(k, count)
    g = sp.sp_graph_upload(rp, ci)
    total, per = sp.sp_triangle_count(g, per_vertex=True)
    assert total == count * math.comb(k, 3)
    assert torch.all(per.to(torch.int64) == math.comb(k - 1, 2)).item()
    assert sp.sp_triangle_count(g)[0] == total
    g.release()
