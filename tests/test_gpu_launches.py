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
