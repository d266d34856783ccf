"""What the rule for tiles on quads (csrc/tile_rule.h) rests on: host code alone."""
import json
import os
import re

import pytest

from paper_2408_11551_amd import build, lib_path


def test_workgroups_that_share_a_compute_unit():
    """Tiles of one group of four waves are priced with two workgroups to a compute unit: a wave of each on every SIMD, and their LDS together."""
    if not os.path.exists(build.RESOURCES) or os.path.getmtime(build.RESOURCES) + 60 < os.path.getmtime(lib_path()):
        pytest.skip("no report of this build")
    single = {}
    for name, use in json.load(open(build.RESOURCES)).items():
        m = re.search(r"spmm_quad_tile_kernelILi(\d)ELi(\d)ELi(\d)ELi1E", name)
        if m:
            single[m.groups()] = use
    assert set(single) == {(t, n, "4") for t in "24" for n in "468"}
    for use in single.values():
        assert use["Occupancy"] == 2 and 2 * use["LDS Size"] <= 160 * 1024, single
