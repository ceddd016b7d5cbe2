"""The bytes that bench.py prices the product's kernels with, against the recorded byte counters."""
import os
import re
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


@pytest.mark.parametrize("c,suffix", [(16, ""), (8, "32")])
def test_algorithmic_bytes_are_those_that_are_moved(c, suffix):
    """256^3 sphere, two vectors: the counters see the algorithmic bytes within 1 %, and in the x and y passes
    what comes with them: one more 128-byte segment at both ends of a plane's rows for each kx and
    component (2 x 256 x 512 x 6 x 128 bytes, either precision).  Not less: lines that the kernels leave
    out are not counted as moved."""
    import bench
    from paper_0704_0037_amd import inputs
    text = open(os.path.join(ROOT, "profiles", "traffic_sphere256_fp64_2rhs.md")).read()
    ab = bench.alg_bytes(inputs.sphere_mask(256), 512, c, 2)
    for k in bench.KERNELS:
        moved = float(re.search(rf"\b{k}{suffix}_bytes=(\d+)", text)[1])
        ends = 0 if k == "zmul" else 2 * 256 * 512 * 6 * 128
        assert 0.99 * ab[k] < moved < 1.01 * ab[k] + ends, (k, moved, ab[k])


def test_lines_left_out_follow_the_launch_rule():
    import bench
    mask = np.zeros((64, 64, 64), np.uint8)
    mask[3, 10, 5] = mask[3, 20, 6] = mask[40, 63, 0] = 1  # 11 rows of plane 3, one of plane 40
    assert bench.lines_moved(mask, 128, 16, 10) == 64 * 64  # 251,658,240 bytes of planes
    assert bench.lines_moved(mask, 128, 16, 11) == 12
