"""Which kernels a call launches, as sp_profile_read counts them."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2305_03317_amd import graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [40, 150])
def test_forced_pulls_on_short_rows_launch_no_push_rounds(size):
    from paper_2305_03317_amd import sp
    rp, ci = graphs.road(size, 0.02, seed=3)
    w = graphs.weights(rp, ci, 12)
    g = sp.sp_graph_upload(rp, ci)
    sp.sp_graph_set_weights(g, w)
    sp.sp_profile_read()
    sp.sp_profile_enable(sp.SP_PROFILE_TIMES)
    got = sp.sp_sssp(g, 0, config={"direction": 2}).cpu().numpy()
    sp.sp_profile_enable(False)
    seen = sp.sp_profile_read()
    assert np.array_equal(got, oracle.sssp(rp, ci, w, 0))
    assert "sssp_pull" in seen and "sssp_push" not in seen
    assert sp.sp_sssp_get_last_stats()["block_size"] == 256
    g.release()


def test_every_family_with_work_reports_its_launches_and_time():
    """Work that rows of long vertices do is counted where its time is: in both passes of both BC paths."""
    from paper_2305_03317_amd import sp
    rp, ci = graphs.rmat(13, 16, seed=8)
    src = graphs.sources(rp, 4, 7, min_degree=1)
    g = sp.sp_graph_upload(rp, ci)
    sp.sp_profile_read()
    want = oracle.bc(rp, ci, src)
    for call, families in ((sp.sp_bc, ("src_topdown", "src_bottomup", "src_sigma", "src_sigma_hub", "src_delta",
                                       "src_delta_hub")),
                           (sp.sp_bc_batch, ("ms_topdown", "ms_bottomup", "ms_sigma", "ms_sigma_hub", "ms_delta",
                                             "ms_delta_hub", "ms_bc"))):
        sp.sp_profile_enable(sp.SP_PROFILE_TIMES | sp.SP_PROFILE_COUNTS)
        got = call(g, src)[0].cpu().numpy()
        sp.sp_profile_enable(False)
        seen = sp.sp_profile_read()
        assert np.allclose(got, want, rtol=1e-9, atol=0)
        for f in families:
            assert f in seen and seen[f]["launches"] > 0 and seen[f]["total_ms"] > 0, f
        if call is sp.sp_bc:  # each row of a reached vertex but the source's is walked once in the reverse pass
            deg = np.diff(rp).astype(np.int64)
            walked = 0
            for s in map(int, src):
                dist, _, _ = oracle.source_detail(rp, ci, s)
                walked += int(deg[dist > 0].sum())
            assert seen["src_delta"]["edges"] + seen["src_delta_hub"]["edges"] == walked
            assert seen["src_delta_hub"]["edges"] > 0
    g.release()
