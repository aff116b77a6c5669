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


# (B, N, L_max, C, boundary): kernels launched by a forward, by both gradients
# and by one.  One launch is the one-block kernel, three per convolution the
# others; the first four were slower in the other form.
ROUTES = [
    ((128, 16, 2, 64, 0), (1, 1, 1)),   # many blocks that read half a line
    ((128, 256, 0, 8, 0), (1, 1, 1)),   # many blocks, no contraction
    ((128, 256, 3, 8, 0), (3, 6, 3)),   # 256 rows, a quarter of each line per block
    ((32, 256, 3, 16, 0), (3, 6, 3)),
    ((32, 33, 2, 32, 1), (1, 1, 1)),    # zero-padded: a quarter of the rows is there
    ((16, 256, 3, 16, 0), (3, 1, 3)),   # two gradients save more launches than a forward
    ((64, 16, 5, 100, 0), (3, 6, 3)),   # rows of more than 64 channels
    ((4, 128, 7, 2, 0), (3, 6, 3)),     # above the kernel's L_max
    ((1, 1, 0, 1, 1), (1, 1, 1)),
]


def test_kernels_per_call(tmp_path):
    run(tmp_path, """
for (B, N, L, C, boundary), want in %r:
    plan = P.cgconv_plan_create_boundary(B, N, L, C, boundary)
    got = []
    for call in (lambda: P.cgconv_forward(plan, ptr(0), ptr(1), ptr(2), 0),
                 lambda: P.cgconv_backward(plan, ptr(0), ptr(1), ptr(2), ptr(3), ptr(4), 0),
                 lambda: P.cgconv_backward(plan, ptr(0), ptr(1), ptr(2), ptr(3), None, 0)):
        call()
        got.append(len(launches()))
    assert tuple(got) == want, (B, N, L, C, boundary, got)
    P.cgconv_plan_destroy(plan)
""" % ROUTES)


def test_every_launch_is_within_the_kernels_limits(tmp_path):
    # the launcher refuses a shape that its kernel does not take (an exception here)
    run(tmp_path, """
for L in range(7):
    for N, boundary in ((2, 0), (4, 0), (8, 0), (16, 0), (32, 0), (64, 0), (128, 0), (256, 0), (1, 1), (13, 1), (50, 1), (128, 1)):
        for C in (1, 2, 3, 5, 8, 10, 17, 24, 40, 64, 65):
            for B in (1, 40, 300):
                plan = P.cgconv_plan_create_boundary(B, N, L, C, boundary)
                P.cgconv_forward(plan, ptr(0), ptr(1), ptr(2), 0)
                P.cgconv_forward_bf16(plan, ptr(0), ptr(1), ptr(2), 0)
                P.cgconv_backward(plan, ptr(0), ptr(1), ptr(2), ptr(3), ptr(4), 0)
                P.cgconv_backward(plan, ptr(0), ptr(1), ptr(2), None, ptr(4), 0)
                for grid, block, lds, allowed in launches():
                    assert block[0] <= 1024 and block[0] % 64 == 0 and lds <= allowed, (B, N, L, C, block, lds)
                P.cgconv_plan_destroy(plan)
""")


def test_first_pass_of_long_odd_lengths_fills_the_chip(tmp_path):
    # DFT lengths 40960, 49152, 57344 (256 rows per outer tile column) and 3584 (32
    # columns per tile): with fewer blocks they were slower than the next power of
    # two at few columns
    run(tmp_path, """
for N, L, C, blocks in ((20000, 0, 1, 256), (24500, 0, 1, 256), (28600, 0, 1, 256), (1790, 1, 16, 128)):
    plan = P.cgconv_plan_create_boundary(1, N, L, C, 1)
    P.cgconv_forward(plan, ptr(0), ptr(1), ptr(2), 0)
    grid = launches()[0][0]
    assert grid[0] * grid[1] * grid[2] >= blocks, (N, grid)
    P.cgconv_plan_destroy(plan)
""")


def test_dft_lengths_are_the_benchmarks(tmp_path):
    # unfused plans: the groups of the first two passes are the two factors of the length
    run(tmp_path, """
import bench
for N in list(range(257, 400)) + list(range(500, 32769, 487)) + [1024, 1025, 1792, 1793, 14336, 14337, 20480, 28672, 28673, 32768]:
    plan = P.cgconv_plan_create_boundary(1, N, 7, 1, 1)
    P.cgconv_forward(plan, ptr(0), ptr(1), ptr(2), 0)
    first, second = (l[0][1] for l in launches()[:2])
    assert first * second == bench.dft_length(N, "linear"), (N, first, second)
    P.cgconv_plan_destroy(plan)
""")
