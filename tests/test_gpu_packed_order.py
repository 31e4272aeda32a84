"""The order in which packed sequences of different lengths are dealt out to the workgroups (longest
first, heads over the XCDs in turn): every block of every sequence is computed, whatever the numbers of
sequences and heads, equal and empty sequences among them.  The dense call on each sequence alone runs
the same arithmetic, so the results are equal bit for bit."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d,lengths", [
    (1, 64, [5]),
    (3, 64, [130, 0, 257, 257, 31]),            # 15 heads of sequences: a last group of seven
    (8, 128, [64, 300, 300, 1]),
    (12, 64, [129, 640, 200]),
    (2, 128, [1000, 40, 513, 0, 0, 999]),
    (1, 64, [(37 * i) % 150 for i in range(64)]),   # the most that are sorted
    (1, 64, [(41 * i) % 150 for i in range(65)]),   # the caller's order
    (16, 128, [2048, 100, 1500]),               # d = 128 with the 64-row forward
])
@pytest.mark.parametrize("causal", [False, True])
def test_packed_sequences_equal_dense_calls(H, d, lengths, causal):
    g = torch.Generator().manual_seed(sum(lengths) + H)
    total, longest = sum(lengths), max(lengths)
    q, k, v, do = (torch.randn(total, H, d, generator=g).bfloat16().cuda() for _ in range(4))
    o, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    starts = [sum(lengths[:i]) for i in range(len(lengths) + 1)]
    cu = torch.tensor(starts, dtype=torch.int32, device="cuda")
    bias = -math.log(longest)
    sa.sigmoid_attn_varlen_fwd(q, k, v, o, cu, longest, bias, causal)
    sa.sigmoid_attn_varlen_bwd(q, k, v, do, dq, dk, dv, cu, longest, bias, causal)
    for a, b in zip(starts, starts[1:]):
        if a == b:
            continue
        one = lambda x: x[a:b].transpose(0, 1).unsqueeze(0).contiguous()
        Q, K, V, DO = one(q), one(k), one(v), one(do)
        O, DQ, DK, DV = (torch.empty_like(Q) for _ in range(4))
        sa.sigmoid_attn_fwd(Q, K, V, O, bias, causal)
        sa.sigmoid_attn_bwd(Q, K, V, DO, DQ, DK, DV, bias, causal)
        for x, y in ((o, O), (dq, DQ), (dk, DK), (dv, DV)):
            assert torch.equal(one(x), y)
