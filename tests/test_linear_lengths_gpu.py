"""Zero-padded plans at DFT lengths P * 2^a, P = 3, 5, 7 (lengths the powers of
two would overshoot): every outer-pass radix, the fused pipeline, the unfused
one (L_max 7, lengths above 32768) and the stages that keep spectra between
passes (channel mixing, inter-channel), against the oracle's cyclic FFT mode
on padded inputs (any padded length >= 2N - 1 gives the linear sums).  Then
the powers of two that zero-padded plans still take.

Tolerance: fp32 DFTs and sums, a few 2^-24 sqrt(log2 N); bar 2e-6.  The mixed
form multiplies bfloat16 high and low parts: 2e-5.
"""

import numpy as np
import pytest

from oracle.backward import backward_fft
from oracle.conv import cgconv_fft
from oracle.inter import cgconv_interchannel
from oracle.mix import cgconv_mixed_fft

pytestmark = pytest.mark.gpu

TOL, TOL_MIXED = 2e-6, 2e-5

LENGTHS = [P << a for a in range(5, 15) for P in (3, 5, 7) if (3584 if P == 7 else 640) <= P << a <= 57344]


def _case(B, N, L, C, seed):
    rng = np.random.default_rng(seed)
    K = (L + 1) ** 2
    arrays = [rng.normal(size=(B, N, K, C)).astype(np.float32) for _ in range(3)]
    pad = 1 << (2 * N - 1).bit_length()
    return arrays, [np.pad(a, ((0, 0), (0, pad - N), (0, 0), (0, 0))) for a in arrays]


def _err(got, want):
    return np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want)


@pytest.mark.parametrize("length", LENGTHS)
def test_forward_and_gradients_at_every_length(length):
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    N, L, C = (length + 1) // 2, 1, 3  # the largest N of this length
    (q, k, g), wide = _case(1, N, L, C, length)
    print(f"[gpu] linear length {length} N={N}", flush=True)
    dev = [torch.from_numpy(a).cuda() for a in (q, k, g)]
    plan = P.Plan(1, N, L, C, boundary="linear")
    out = plan(dev[0], dev[1])
    gq, gk = plan.backward(*dev)
    bf = plan(dev[0].bfloat16(), dev[1].bfloat16())
    torch.cuda.synchronize()
    # the workspace holds two spectra of the DFT length
    assert plan.info()[2] < 2 * 8 * (length + 512) * (L + 1) ** 2 * C + 64 * N * (L + 1) * C
    plan.close()
    rq, rk = backward_fft(*wide, L)
    ref = cgconv_fft(wide[0], wide[1], L)[:, :N]
    assert _err(out, ref) <= TOL
    assert _err(gq, rq[:, :N]) <= TOL and _err(gk, rk[:, :N]) <= TOL
    assert np.linalg.norm(bf.float().cpu().numpy() - ref) <= 1e-2 * np.linalg.norm(ref)


@pytest.mark.parametrize("N,L,C", [(320, 6, 6), (380, 3, 2), (1280, 4, 9), (1792, 5, 4), (700, 7, 2), (1300, 8, 3)])
def test_degrees_and_channels(N, L, C):
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    (q, k, g), wide = _case(2, N, L, C, N)
    print(f"[gpu] linear N={N} L={L} C={C}", flush=True)
    dev = [torch.from_numpy(a).cuda() for a in (q, k, g)]
    plan = P.Plan(2, N, L, C, boundary="linear")
    out = plan(dev[0], dev[1])
    gq, gk = plan.backward(*dev)
    torch.cuda.synchronize()
    plan.close()
    rq, rk = backward_fft(*wide, L)
    assert _err(out, cgconv_fft(wide[0], wide[1], L)[:, :N]) <= TOL
    assert _err(gq, rq[:, :N]) <= TOL and _err(gk, rk[:, :N]) <= TOL


@pytest.mark.parametrize("N", [320, 380, 1790])  # lengths 640, 768, 3584
def test_mixed_and_interchannel(N):
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    L, C, heads, m_out = 3, 8, 2, 4
    (q, k, _), wide = _case(2, N, L, C, N)
    rng = np.random.default_rng(7)
    w = rng.normal(size=(len(P.cgconv_paths(L)), C, C)).astype(np.float32)
    wi = rng.normal(size=(heads, L + 1, m_out, (C // heads) ** 2)).astype(np.float32)
    print(f"[gpu] linear mixed and inter-channel N={N}", flush=True)
    plan = P.Plan(2, N, L, C, boundary="linear")
    dev = [torch.from_numpy(a).cuda() for a in (q, k, w, wi)]
    mixed = plan.forward_mixed(*dev[:3])
    inter = plan.forward_interchannel(dev[0], dev[1], dev[3], heads)
    torch.cuda.synchronize()
    plan.close()
    assert _err(mixed, cgconv_mixed_fft(wide[0], wide[1], L, w)[:, :N]) <= TOL_MIXED
    assert _err(inter, cgconv_interchannel(wide[0], wide[1], L, heads, wi, mode="fft")[:, :N]) <= TOL


# 2048 fused, 32768 fused with outer passes of 512, 65536 unfused, 1024 unfused at L_max 8
@pytest.mark.parametrize("N,length,L,C", [(1000, 2048, 2, 3), (14337, 32768, 1, 2), (16384, 32768, 1, 2),
                                          (28673, 65536, 1, 2), (32768, 65536, 0, 3), (400, 1024, 8, 2)])
def test_power_of_two_lengths(N, length, L, C):
    torch = pytest.importorskip("torch")
    import paper_2509_24093_amd as P
    (q, k, g), wide = _case(1, N, L, C, N)
    print(f"[gpu] linear N={N} length {length} L={L}", flush=True)
    dev = [torch.from_numpy(a).cuda() for a in (q, k, g)]
    plan = P.Plan(1, N, L, C, boundary="linear")
    out = plan(dev[0], dev[1])
    gq, gk = plan.backward(*dev)
    bf = plan(dev[0].bfloat16(), dev[1].bfloat16())
    torch.cuda.synchronize()
    spectra = 2 * 8 * (L + 1) ** 2 * C  # the workspace holds two spectra of the DFT length
    assert spectra * length <= plan.info()[2] < spectra * (length + 512) + 64 * N * (L + 1) * C
    plan.close()
    rq, rk = backward_fft(*wide, L)
    ref = cgconv_fft(wide[0], wide[1], L)[:, :N]
    assert _err(out, ref) <= TOL
    assert _err(gq, rq[:, :N]) <= TOL and _err(gk, rk[:, :N]) <= TOL
    assert np.linalg.norm(bf.float().cpu().numpy() - ref) <= 1e-2 * np.linalg.norm(ref)
