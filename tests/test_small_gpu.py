"""The one-block kernel for DFT lengths <= 256 over its launch shapes: one,
two and four lane groups per point, channel groups of 2 to 16 with ragged
last groups, zero-padded lengths, and both gradients or one in a launch,
against the oracle.

Tolerance: fp32 storage and sums; the DFTs and the contraction keep the
relative error at a few 2^-24 sqrt(log2 N) (about 4e-7), bar 2e-6.
"""

import numpy as np
import pytest

from oracle.backward import backward_fft
from oracle.conv import cgconv_fft

pytestmark = pytest.mark.gpu

TOL = 2e-6

# (B, N, L, C, boundary)
SHAPES = [
    (1, 2, 0, 1, "cyclic"),      # shortest length, one part
    (1, 16, 6, 8, "cyclic"),     # four parts of one wave
    (3, 32, 4, 32, "cyclic"),    # two channels per block, four parts
    (32, 32, 4, 32, "cyclic"),   # eight channels per block, two parts; the backward fills 256 blocks
    (40, 8, 5, 7, "cyclic"),     # ragged channel group, odd C
    (300, 8, 3, 3, "cyclic"),    # more blocks than CUs: one part
    (5, 256, 3, 16, "cyclic"),   # three kernels forward, one block backward
    (2, 256, 1, 4, "cyclic"),    # longest length
    (3, 50, 2, 5, "linear"),     # zero padding, DFT length 128
    (2, 13, 6, 3, "linear"),     # zero padding, DFT length 32
    (1, 1, 4, 2, "linear"),      # a single token
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%dN%dL%dC%d%s" % s)
def test_one_block_forward_and_gradients(shape):
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    B, N, L, C, boundary = shape
    K = (L + 1) ** 2
    rng = np.random.default_rng(B * 1000 + N)
    q, k, g = (rng.normal(size=(B, N, K, C)).astype(np.float32) for _ in range(3))
    pad = 0 if boundary == "cyclic" else N  # the linear sums are the cyclic ones of the padded rows
    wide = [np.pad(a, ((0, 0), (0, pad), (0, 0), (0, 0))) for a in (q, k, g)]
    ref = cgconv_fft(wide[0], wide[1], L)[:, :N]
    rq, rk = (r[:, :N] for r in backward_fft(*wide, L))
    print(f"[gpu] one-block kernel {shape}", flush=True)
    plan = P.Plan(B, N, L, C, boundary=boundary)
    dev = [torch.from_numpy(a).cuda() for a in (q, k, g)]
    out = plan(dev[0], dev[1])
    gq, gk = plan.backward(*dev)
    only_q, none = plan.backward(*dev, need_k=False)
    none2, only_k = plan.backward(*dev, need_q=False)
    torch.cuda.synchronize()
    assert none is None and none2 is None
    for got, want in ((out, ref), (gq, rq), (gk, rk), (only_q, rq), (only_k, rk)):
        err = np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want)
        assert err <= TOL, err
    plan.close()


def test_timed_backward_of_the_one_block_kernel_is_one_call():
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    for L, gradients, calls, stages in ((4, 2, 1, ["cg_small"]), (4, 1, 1, ["cg_small"]),
                                        (7, 2, 2, ["fft_fwd", "cg", "fft_inv"])):
        plan = P.Plan(32, 32, L, 4)
        q, k, g = (torch.randn(plan.shape, device="cuda") for _ in range(3))
        P.cgconv_plan_enable_timing(plan._h, 8)
        print(f"[gpu] timed backward L={L} gradients={gradients}", flush=True)
        plan.backward(q, k, g, need_k=gradients == 2)
        times, n = P.cgconv_plan_stage_times(plan._h)
        plan.close()
        assert n == calls and list(times) == stages and all(t > 0 for t in times.values())
