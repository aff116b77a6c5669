"""The inter-channel stage where a block takes several groups of eight frequency
points (many points at L_max <= 4, ragged last group and last block), one
group per block (L_max 5, 6) and channel counts below the eight slots, against
the oracle.  Tolerance: fp32 products and sums over the components and the
channel pairs, a few 2^-24 times the square root of their number: 2e-6.
"""

import numpy as np
import pytest

from oracle.inter import cgconv_interchannel

pytestmark = pytest.mark.gpu

TOL = 2e-6


@pytest.mark.parametrize("shape", [
    (2, 16384, 1, 8, 4, 2),   # four groups per block, two channels per head
    (4, 8192, 3, 8, 2, 4),    # two groups per block
    (5, 4096, 2, 16, 4, 4),   # two groups per block, ragged
    (3, 8192, 4, 9, 3, 2),    # L_max 4, odd channels per head
    (1, 512, 0, 8, 1, 8),     # degree 0 only
    (2, 128, 5, 14, 2, 6),    # seven channels per head
    (1, 64, 6, 16, 2, 8),
], ids=lambda s: "B%dN%dL%dC%dH%do%d" % s)
def test_groups_of_points(shape):
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    B, N, L, C, heads, m_out = shape
    rng = np.random.default_rng(N + L)
    q, k = (rng.normal(size=(B, N, (L + 1) ** 2, C)).astype(np.float32) for _ in range(2))
    w = rng.normal(size=(heads, L + 1, m_out, (C // heads) ** 2)).astype(np.float32)
    print(f"[gpu] inter-channel groups {shape}", flush=True)
    plan = P.Plan(B, N, L, C)
    out = plan.forward_interchannel(*(torch.from_numpy(a).cuda() for a in (q, k, w)), heads)
    torch.cuda.synchronize()
    plan.close()
    ref = cgconv_interchannel(q, k, L, heads, w, mode="fft")
    assert np.linalg.norm(out.cpu().numpy() - ref) <= TOL * np.linalg.norm(ref)
