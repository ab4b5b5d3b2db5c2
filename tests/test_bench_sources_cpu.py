"""bench.py reuses a kernel's stored counter readings while its sources are unchanged: the list of
those sources must name every file the stage's kernels are compiled from."""
import glob
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2505_06582_amd", "csrc")


@pytest.mark.parametrize("kernel,pattern", [("accumulate", "k_accum*.hip"), ("adjoint", "k_adjoint*.hip")])
def test_sources_of_a_stage_are_all_listed(kernel, pattern):
    listed = set(bench.TRAFFIC_SOURCES[kernel])
    files = [os.path.basename(p) for p in glob.glob(os.path.join(CSRC, pattern))]
    assert files and set(files) <= listed
    for name in files + ["k_prep.hip"]:
        text = open(os.path.join(CSRC, name)).read()
        headers = [h for h in re.findall(r'#include "([^"]+)"', text) if os.path.exists(os.path.join(CSRC, h))]
        assert set(headers) | {"gws_internal.h"} <= listed, name
