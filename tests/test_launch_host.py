"""Launch shapes of the one-block kernel (DFT lengths <= 256) as the host side
chooses them, on the CPU (tests/host_runtime.py)."""

import os

import pytest

import paper_2509_24093_amd as P
from tests.host_runtime import run

pytestmark = pytest.mark.skipif(not os.path.exists(P.LIB_PATH), reason="libcgconv.so not built")


def test_a_later_smaller_plan_leaves_an_earlier_ones_lds(tmp_path):
    # L_max 5: 74752 bytes of dynamic LDS, then a plan of the same kernel with 73984
    run(tmp_path, """
big = P.cgconv_plan_create(1, 128, 5, 2)
small = P.cgconv_plan_create(256, 32, 5, 8)
for plan in (big, small):
    P.cgconv_forward(plan, ptr(0), ptr(1), ptr(2), 0)
    P.cgconv_backward(plan, ptr(0), ptr(1), ptr(2), ptr(3), ptr(4), 0)
seen = launches()
assert max(lds for _, _, lds, _ in seen) > 64 * 1024, seen
for grid, block, lds, allowed in seen:
    assert lds <= allowed, (grid, block, lds, allowed)
""")
