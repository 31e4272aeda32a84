"""The fp32 kernels deal the streamed chunks of a 32-row block out to four or eight waves: parity
with the fp64 oracle where that split can go wrong -- fewer chunks than waves, ragged last chunks,
either wave count, and causal grids on both sides of one and two workgroups per compute unit
(whose dispatch order mirrors the second 256 places)."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc
from paper_2409_04431_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of max |reference|: the fp32 bar of the library, sums of at most 1024 products


@pytest.mark.parametrize("B,H,Hkv,N,d,causal,alibi", [
    (1, 1, 1, 31, 128, True, False),      # one ragged chunk for eight waves
    (1, 2, 2, 33, 64, False, True),       # two chunks, the second with a single row
    (1, 3, 1, 257, 128, True, True),      # a group of three query heads in the dK/dV pass
    (1, 12, 12, 352, 64, True, False),    # forward 132 workgroups (eight waves), backward 264 (four)
    (2, 12, 12, 352, 128, True, False),   # 264: the mirrored places begin inside a row of heads
    (3, 16, 16, 353, 64, True, True),     # 576: more than two workgroups per compute unit
    (3, 16, 4, 353, 64, False, False),
])
def test_fp32_split_over_waves_matches_oracle(B, H, Hkv, N, d, causal, alibi):
    g = torch.Generator().manual_seed(41 + N + H)
    q, do = (torch.randn(B, H, N, d, generator=g) for _ in range(2))
    k, v = (torch.randn(B, Hkv, N, d, generator=g) for _ in range(2))
    slopes = W.alibi_slopes(H) if alibi else None
    sl = slopes.cuda() if alibi else None
    bias = -math.log(N)
    Q, K, V, DO = (t.cuda() for t in (q, k, v, do))
    o, dq = (torch.full_like(Q, float("nan")) for _ in range(2))
    dk, dv = (torch.full_like(K, float("nan")) for _ in range(2))
    sa.sigmoid_attn_mqa_fwd(Q, K, V, o, bias, causal, sl)
    sa.sigmoid_attn_mqa_bwd(Q, K, V, DO, dq, dk, dv, bias, causal, sl)
    if Hkv == H:  # the passes alone add up in the same order
        dq1, dk1, dv1 = (torch.empty_like(Q) for _ in range(3))
        sa.sigmoid_attn_bwd_dkdv(Q, K, V, DO, dk1, dv1, bias, causal, sl)
        sa.sigmoid_attn_bwd_dq(Q, K, V, DO, dq1, bias, causal, sl)
        torch.cuda.synchronize()
        assert torch.equal(dq, dq1) and torch.equal(dk, dk1) and torch.equal(dv, dv1)
    torch.cuda.synchronize()
    f = lambda t: t.double().numpy()
    ro = orc.sigmoid_attn_mqa_fwd(f(q), f(k), f(v), bias, causal, slopes)
    refs = orc.sigmoid_attn_mqa_bwd(f(q), f(k), f(v), f(do), bias, causal, slopes)
    for name, got, ref in zip(("o", "dq", "dk", "dv"), (o, dq, dk, dv), (ro, *refs)):
        err = abs(got.double().cpu().numpy() - ref).max() / abs(ref).max()
        assert err <= TOL, f"{name}: {err:.3e}"
