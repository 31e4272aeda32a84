"""Packed fp32 batches whose longest length, heads and sequences make more blocks of 32 rows than one
launch takes work-items for (most of the blocks belong to no sequence): computed as any other, against
the dense call on each sequence."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa

pytestmark = pytest.mark.gpu


def test_packed_fp32_with_more_blocks_than_one_launch_takes():
    B, H, d, longest = 64, 32, 64, 1 << 18  # 2^24 blocks a pass, four waves each
    lengths = [0] * B
    lengths[0], lengths[37], lengths[63] = 45, 130, 64
    starts = [sum(lengths[:i]) for i in range(B + 1)]
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, do = (torch.randn(starts[-1], H, d, generator=g, device="cuda") for _ in range(4))
    o, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    cu = torch.tensor(starts, dtype=torch.int32, device="cuda")
    bias = -math.log(100)
    sa.sigmoid_attn_varlen_fwd(q, k, v, o, cu, longest, bias, True)
    sa.sigmoid_attn_varlen_bwd(q, k, v, do, dq, dk, dv, cu, longest, bias, True)
    for a, b in zip(starts, starts[1:]):
        if a == b:
            continue
        one = lambda x: x[a:b].transpose(0, 1).unsqueeze(0).contiguous()
        Q, K, V, DO = one(q), one(k), one(v), one(do)
        ref = [torch.empty_like(Q) for _ in range(4)]
        sa.sigmoid_attn_fwd(Q, K, V, ref[0], bias, True)
        sa.sigmoid_attn_bwd(Q, K, V, DO, *ref[1:], bias, True)
        for x, y in zip((o, dq, dk, dv), ref):  # the waves' sums run in another order: fp32 sums of at most 130 products
            assert (one(x) - y).abs().max() <= 1e-5 * y.abs().max()
