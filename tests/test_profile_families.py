"""Every kernel that the library launches under a profile family is found again
by the counter summary under the same family, without a GPU."""
from __future__ import annotations

import os
import re

from paper_2305_03317_amd import rocprof_summary as rs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def families():
    text = open(os.path.join(ROOT, "paper_2305_03317_amd", "csrc", "profile.hip")).read()
    return re.findall(r'"(\w+)"', re.search(r"kProfNames\[\w*\]\s*=\s*\{(.*?)\};", text, re.S).group(1))


def test_every_family_has_a_kernel():
    known = set(rs.FAMILY.values()) | {f for part in rs.PARTS.values() for f in part.values()}
    missing = [f for f in families() if f not in known]
    assert not missing, missing
    # and no kernel is put under one that is not reported (but the blocks engine's sum, timed as ms_bc)
    assert known - set(families()) <= {None, "wg_bc_sum"}


def test_kernel_names_exist_in_the_sources():
    text = "".join(open(os.path.join(rs.CSRC, f)).read() for f in os.listdir(rs.CSRC) if f.endswith(".hip"))
    for k in list(rs.FAMILY) + list(rs.PARTS):
        assert re.search(r"\b%s\(" % k, text), k


def test_parts_by_their_last_template_argument():
    name = "void sp::k_ms_sigma_rest<%d, %d>(sp::LevelCtl*, int const*)"
    assert rs.family_of(rs.short_name(name % (512, 1))) == "ms_sigma_push"
    assert rs.family_of(rs.short_name(name % (256, 2))) == "ms_sigma_hub"
    assert rs.family_of(rs.short_name(name % (256, 3))) is None
    assert rs.family_of("k_src_delta<512, 2>") == "src_delta_hub"
    assert rs.family_of("k_ms_delta_hub<512>") == "ms_delta_hub"
    assert rs.family_of("__amd_rocclr_copyBuffer") is None
