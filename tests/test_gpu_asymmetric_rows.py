"""Rows that are not symmetric, which an upload without `validate` accepts: the
one-workgroup-per-source engine over fixed-width rows against a host model of
what it computes on them.  Levels go along a vertex's row, sigma is the sum over
the vertex's own row of the level before, delta over its own row of the level
after; all sums in row order.  Distances and path counts exact, dependencies and
BC to 1e-9 relative (the bar of the parity tests), infinities and NaN (a vertex
without a parent in its own row counts no path) where the model has them."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu


def rows_of(rp, ci):
    return [list(map(int, ci[rp[v]:rp[v + 1]])) for v in range(len(rp) - 1)]


def make(name: str):
    """Rows as lists, at most 4 entries each (8 for names that end in 8)."""
    if name == "cycle":
        return [[(v + 1) % 5] for v in range(5)]
    if name == "cycle8":
        return [[(v + k) % 4099 for k in (1, 2, 3, 5, 8, 13)] for v in range(4099)]
    width = 40
    rows = rows_of(*graphs.road(width, 0.02, seed=3))
    room = [v for v in range(len(rows)) if len(rows[v]) < 4]
    if name == "grid":  # symmetric
        return rows
    if name == "one-way":  # an entry whose reverse is missing
        v = max(range(len(rows)), key=lambda x: len(rows[x]))
        rows[rows[v][0]].remove(v)
    elif name == "back":  # from everywhere to vertices reached long before
        for v in room[5:]:
            rows[v].append(room[v % 5])
    elif name == "back8":
        for v in range(len(rows)):
            rows[v] += [0, 1, (v * 7) % 1600, v][:8 - len(rows[v])]
    elif name == "multiple":  # the same edge twice in both rows, thrice and once
        v = room[0]
        rows[v].append(rows[v][0])
        rows[rows[v][0]].append(v)
        v = room[7]
        rows[v].append(rows[v][0])
    elif name == "loops":  # symmetric
        for v in room[:200]:
            rows[v].append(v)
    return rows


def model(rows, s):
    n = len(rows)
    dist, sigma, delta, rho = np.full(n, -1, np.int32), np.zeros(n), np.zeros(n), np.zeros(n)
    dist[s], sigma[s] = 0, 1.0
    levels = [[s]]
    while levels[-1]:
        nxt = []
        for v in levels[-1]:
            for u in rows[v]:
                if dist[u] < 0:
                    dist[u] = len(levels)
                    nxt.append(u)
        for u in nxt:
            for v in rows[u]:
                if dist[v] == len(levels) - 1:
                    sigma[u] += sigma[v]
        levels.append(nxt)
    with np.errstate(all="ignore"):
        for k in range(len(levels) - 1, 0, -1):
            for v in levels[k]:
                acc = np.float64(0.0)
                for u in rows[v]:
                    if dist[u] == k + 1:
                        acc += rho[u]
                delta[v] = sigma[v] * acc
                rho[v] = (1.0 + delta[v]) / sigma[v]
    return dist, sigma, delta


def close(got, ref):
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-9 * np.abs(ref[fin]))


@pytest.mark.parametrize("name", ["grid", "loops", "cycle", "cycle8", "one-way", "back", "back8", "multiple"])
@pytest.mark.parametrize("block", [128, 1024])
def test_rows(name, block):
    from paper_2305_03317_amd import sp
    print(name, block, flush=True)
    rows = make(name)
    n = len(rows)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate([np.array(r, np.int32) for r in rows])
    assert np.diff(rp).max() <= (8 if name.endswith("8") or name == "multiple" else 4)
    src = np.array([0, n // 2, n - 1, 0], np.int32)
    want = [model(rows, int(s)) for s in src]
    g = sp.sp_graph_upload(rp, ci)
    cfg = {"engine": sp.SP_ENGINE_BLOCKS, "block_size": block, "batch_width": 3}
    for _ in range(2):  # the first pass looks at the rows
        got = sp.sp_bc_batch(g, src, config=cfg)[0].cpu().numpy()
        with np.errstate(all="ignore"):
            close(got, sum(d for _, _, d in want))
    out = sp.sp_batch_levels(g, src[:3], with_delta=True, config=cfg)
    for k in range(3):
        assert np.array_equal(out[0][k].cpu().numpy(), want[k][0])
        assert np.array_equal(out[1][k].cpu().numpy(), want[k][1])
        close(out[2][k].cpu().numpy(), want[k][2])
    g.release()
