"""bench.py finds the traffic of both scoring passes in the committed profile, under the names the kernels have."""

import os
import re

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("kernel", ["score_stats", "score_accum"])
def test_traffic_of_a_scoring_pass(kernel):
    # 7.8 ranked heads x 32704 keys x 256 B and the queries are 65.4 MB; a pass cannot read less, and reads little more
    got = bench.measured_traffic_bytes(kernel)
    assert got is not None and 65.4e6 <= got <= 1.25 * 65.4e6


def test_the_profile_names_kernels_that_exist():
    src = "".join(open(os.path.join(ROOT, "paper_2508_15806_amd", "csrc", f)).read() for f in ("compress.hip", "stage1.hip"))
    defined = set(re.findall(r"\b([a-z_0-9]+_kernel)\s*\(", src))
    for name in os.listdir(os.path.join(ROOT, "profiles")):
        for line in open(os.path.join(ROOT, "profiles", name)):
            if line.startswith("|"):
                for kernel in re.findall(r"\b([a-z_0-9]+_kernel)\b", line):
                    assert kernel in defined, (name, kernel)
