"""The benchmark's byte model of the sorting stages follows the library's choice of
sort: buckets up to 4096 of 1365 particles, radix passes beyond.
"""
import os
import re

import pytest

import bench

CSRC = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_1204_2280_amd", "csrc")


@pytest.mark.parametrize("n,sorting,moving", [(1 << 22, 68, 49), (4096 * 1365, 68, 49), (4096 * 1365 + 1, 312, 36),
                                              (1 << 24, 312, 36)])
def test_sort_bytes(n, sorting, moving):
    stage = {k: 1.0 for k in ("sorting", "moving", "tree_construction", "multipoles", "mac_prep")}
    got = bench.hbm_stages(stage, n, 0)
    assert (got["sorting"]["bytes"], got["moving"]["bytes"]) == (sorting * n, moving * n)
    assert got["tree_construction"]["bytes"] == 25 * n and got["multipoles"]["bytes"] == 16 * n


def test_the_line_is_the_librarys():
    text = open(os.path.join(CSRC, "mibh_device.h")).read()
    buckets = int(re.search(r"SORT_MAX_BUCKETS = (\d+);", text).group(1))
    mean = int(re.search(r"return n <= 1u << 21 \? \d+u : (\d+)u;", text).group(1))
    assert buckets * mean == bench.BUCKET_SORT_MAX
