"""Exchanges between the lanes of a wave through LDS, in the kernels' sources (no GPU needed)."""

import glob
import os
import re

from paper_2607_01408_amd import build


def test_wave_barriers_come_with_a_fence():
    """``__builtin_amdgcn_wave_barrier`` orders no memory, so a lane's LDS reads could be moved over the writes
    of another lane.  Every exchange goes through the helper that puts a wavefront fence before it."""
    sources = sorted(p for ext in ("h", "hip") for p in glob.glob(os.path.join(build.CSRC, "*." + ext)))
    assert sources
    helpers = []
    for path in sources:
        text = open(path).read()
        if "__builtin_amdgcn_wave_barrier" in text:
            helpers.append(os.path.basename(path))
            bare = re.findall(r'(?<!"wavefront"\);\n    )__builtin_amdgcn_wave_barrier\(\)', text)
            assert not bare, path
    assert helpers == ["lds_common.h"]  # one helper for all of them
