"""The traffic a benchmark line reports belongs to the kernel that the workload runs."""

import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize("L, spins, valu, name", [
    (2, (-2, -1, 0, 1, 2), False, "spingtp_fwd_unrolled_kernel"),
    (1, (-2, -1, 0, 1, 2), False, "spingtp_fwd_unrolled_kernel"),
    (2, (-2, -1, 0, 1, 2), True, "spingtp_fwd_direct_kernel"),
    (3, (-2, -1, 0, 1, 2), False, "spingtp_fwd_direct_kernel"),
    (0, (-2, -1, 0, 1, 2), False, "spingtp_fwd_direct_kernel"),
    (2, (-2, 0, 2), False, "spingtp_fwd_direct_kernel"),
])
def test_kernel_of_the_direct_family(L, spins, valu, name):
    assert bench.forward_kernel_name(6, L, spins, valu) == name


def test_chiral_traffic_is_of_the_kernel_that_runs():
    # the record is served for its own kernel only (and not at all once that kernel's sources changed)
    name = bench.forward_kernel_name(6, 2, (-2, -1, 0, 1, 2), False)
    with open(os.path.join(ROOT, "profiles", "traffic_spingtp_fwd_chiral_fp32.json")) as f:
        rec = json.load(f)
    assert name + "<" in rec["kernel"]
    assert bench.measured_traffic("chiral", "fp32", rec["units"], 2, name) in (None, rec["hbm_bytes_per_launch"])
    assert bench.measured_traffic("chiral", "fp32", rec["units"], 2, "spingtp_fwd_direct_kernel") is None
