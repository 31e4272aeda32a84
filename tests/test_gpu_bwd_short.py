"""The backward that holds a head whole (up to 256 keys at d = 64, 128 at d = 128): the two passes'
results bit for bit, the oracle's within the bf16 bar, nothing written past the rows of a sequence."""
import math

import numpy as np
import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2  # P, dS and the outputs are rounded to bf16
# On 256 compute units (places: two per unit up to 128 tokens at d = 64) of 17 heads a batch: 3 batches are shared by two
# workgroups a head, or left to the passes (d = 64, N > 128 unmasked, and N = 256); 9 take one a head, or are shared (d = 64,
# N <= 128); of 21 the 101 heads beyond a whole round are shared, or none (d = 64, N <= 128), of 33 there the 49 beyond.
HEADS = 17

SIZES = [(64, n) for n in (1, 31, 32, 33, 64, 65, 127, 128, 129, 160, 193, 255, 256)] + [(128, n) for n in (1, 33, 64, 97, 128)]


DENSE = [(B, d, N) for d, N in SIZES for B in (3, 9, 21)] + [(33, 64, 33), (33, 64, 128)]
ALIBI = [(B, d, N) for d, N in ((64, 31), (64, 128), (64, 129), (64, 250), (128, 33), (128, 128)) for B in (3, 9, 21)]
PACKED = [(64, [256, 1, 0, 33, 250]), (64, [128, 64, 127]), (64, [128, 1, 64, 33, 127]), (128, [128, 5, 0, 96]), (128, [97, 33])]


def _route(heads, d, N, causal, **more):
    """How the call's heads are handed out, as the library reports it."""
    n = sa.sattn_bwd_short(1, heads, N, d, causal, **more)
    return {0: "passes", heads: "whole", 2 * heads: "shared"}.get(n, "mixed")


def _declined(heads, d, N, causal):
    return d == 64 and N > 128 and (4 * heads <= 256 and N == 256 if causal else 2 * heads <= 256)


def test_every_way_of_handing_out_heads_is_among_the_cases():
    kernel = lambda d, N: (d, N > 128)
    seen = {(*kernel(d, N), causal, _route(HEADS * B, d, N, causal)) for B, d, N in DENSE for causal in (False, True)}
    alibi = {(*kernel(d, N), _route(HEADS * B, d, N, False, alibi=True)) for B, d, N in ALIBI}
    packed = {(*kernel(d, max(n)), causal, _route(64 * len(n), d, max(n), causal)) for d, n in PACKED for causal in (False, True)}
    for causal in (False, True):
        assert {(64, False, causal, "passes")} & seen == set() and (64, True, causal, "passes") in seen
        for way in ("whole", "shared", "mixed"):
            assert (64, False, causal, way) in seen and (128, False, causal, way) in seen
            assert (64, True, causal, way) in seen or (way == "shared" and not causal)
        assert {(64, True, causal, "mixed"), (64, False, causal, "shared"), (64, False, causal, "whole"), (128, False, causal, "whole"),
                (128, False, causal, "shared")} <= packed
    assert {(64, False, "whole"), (64, False, "shared"), (64, True, "whole"), (64, True, "mixed"), (64, True, "passes"),
            (128, False, "whole"), (128, False, "shared"), (128, False, "mixed")} <= alibi


def _both(call, like):
    out = []
    try:
        for mode in (2, 0):  # two launches, the choice
            sa.sattn_set_bwd_merged(mode)
            res = [torch.full_like(x, float("nan")) for x in like]
            call(*res)
            torch.cuda.synchronize()
            out.append(res)
    finally:
        sa.sattn_set_bwd_merged(0)
    return out


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,d,N", DENSE)
def test_dense_equals_two_launches_and_the_oracle(B, d, N, causal):
    assert (_route(B * HEADS, d, N, causal) == "passes") == _declined(B * HEADS, d, N, causal)
    g = torch.Generator().manual_seed(100 * N + d)
    q, k, v, do = (torch.randn(B, N, HEADS, d, generator=g).bfloat16() for _ in range(4))
    bias = -math.log(max(N, 2))
    dev = [x.cuda().transpose(1, 2) for x in (q, k, v, do)]  # [B, N, H, d] storage
    two, one = _both(lambda *r: sa.sigmoid_attn_bwd(*dev, *r, bias, causal), dev[:3])
    for a, b in zip(two, one):
        assert torch.equal(a, b) and not torch.isnan(b).any()
    few = [x[:1, :2].contiguous() for x in dev]
    ref = orc.sigmoid_attn_bwd(*(x.cpu() for x in few), bias, causal)
    for x, r in zip(one, ref):
        assert np.abs(x[:1, :2].float().cpu().numpy() - r).max() <= TOL * np.abs(r).max()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("alibi", [False, True])
@pytest.mark.parametrize("d,lengths", PACKED)
def test_packed_equals_two_launches_and_leaves_other_rows_alone(d, lengths, alibi, causal):
    total, B = sum(lengths), len(lengths)
    assert (_route(64 * B, d, max(lengths), causal, alibi=alibi) == "passes") == (alibi and causal)
    slopes = torch.tensor([2.0 ** (-8.0 * (h + 1) / 64) for h in range(64)], device="cuda") if alibi else None
    g = torch.Generator().manual_seed(total + d)
    q, k, v, do = (torch.randn(total + 64, 64, d, generator=g).bfloat16().cuda() for _ in range(4))
    cu = torch.tensor([sum(lengths[:i]) for i in range(B + 1)], dtype=torch.int32, device="cuda")
    bias = torch.tensor([-math.log(max(n, 2)) for n in lengths], dtype=torch.float32, device="cuda")
    two, one = _both(lambda *r: sa.sigmoid_attn_varlen_bwd(q, k, v, do, *r, cu, max(lengths), 0.0, causal, slopes,
                                                           bias_per_seq=bias), [q, k, v])
    for a, b in zip(two, one):
        assert torch.equal(a[:total], b[:total]) and not torch.isnan(b[:total]).any()
        assert torch.isnan(b[total:]).all()


@pytest.mark.parametrize("B,d,N", ALIBI)
def test_alibi_without_a_mask_equals_two_launches(B, d, N):
    assert (_route(B * HEADS, d, N, False, alibi=True) == "passes") == _declined(B * HEADS, d, N, False)
    g = torch.Generator().manual_seed(N + d)
    dev = [torch.randn(B, HEADS, N, d, generator=g).bfloat16().cuda() for _ in range(4)]
    slopes = torch.tensor([2.0 ** (-8.0 * (h + 1) / HEADS) for h in range(HEADS)], device="cuda")
    two, one = _both(lambda *r: sa.sigmoid_attn_bwd(*dev, *r, -math.log(max(N, 2)), False, slopes), dev[:3])
    for a, b in zip(two, one):
        assert torch.equal(a, b) and not torch.isnan(b).any()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,lengths", [(64, [128] * 5), (64, [128, 1, 0, 33]), (128, [97] * 3), (128, [64, 128])])
def test_bias_gradient_equals_two_launches(d, lengths, causal):
    H, total, B, longest = 3, sum(lengths), len(lengths), max(lengths)
    assert _route(B * H, d, longest, causal, bias_grad=True) == "shared"
    g = torch.Generator().manual_seed(total)
    q, k, v, do = (torch.randn(total, H, d, generator=g).bfloat16().cuda() for _ in range(4))
    cu = torch.tensor([sum(lengths[:i]) for i in range(B + 1)], dtype=torch.int32, device="cuda")
    rows, db = torch.empty(H, total, device="cuda"), torch.empty(B, H, device="cuda")
    two, one = _both(lambda *r: sa.sigmoid_attn_varlen_bwd_bias_grad(q, k, v, do, *r[:4], cu, longest, -math.log(longest), causal,
                                                                     None, db=r[4]), [q, k, v, rows, db])
    for a, b in zip(two, one):
        assert torch.equal(a, b) and not torch.isnan(b).any()
    if len(set(lengths)) == 1:  # the dense call
        dense = [x.view(B, longest, H, d).transpose(1, 2) for x in (q, k, v, do)]
        like = [*(x for x in dense[:3]), torch.empty(B, H, longest, device="cuda"), db]
        two, one = _both(lambda *r: sa.sigmoid_attn_bwd_bias_grad(*dense, *r[:4], -math.log(longest), causal, None, db=r[4]), like)
        for a, b in zip(two, one):
            assert torch.equal(a, b) and not torch.isnan(b).any()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,d,N", [(21, 64, 250), (3, 64, 100), (9, 128, 97), (21, 64, 33)])
def test_clock_probe_stamps_are_in_order(B, d, N, causal):
    x = [torch.randn(B, HEADS, N, d, device="cuda").bfloat16() for _ in range(4)]
    grads = [torch.empty_like(x[0]) for _ in range(3)]
    calls = [(lambda: sa.sigmoid_attn_bwd(*x, *grads, -6.0, causal), sa.sattn_bwd_short(B, HEADS, N, d, causal))]
    if sa.sattn_fwd_short(B, HEADS, N, d, causal):
        calls.append((lambda: sa.sigmoid_attn_fwd(*x[:3], grads[0], -6.0, causal), B * HEADS))
    for call, n_wg in calls:
        assert n_wg > 0
        buf = torch.zeros(8 * (n_wg + 8), dtype=torch.int64, device="cuda")
        try:
            sa.sattn_set_clock_probe(buf)
            call()
            torch.cuda.synchronize()
        finally:
            sa.sattn_set_clock_probe(None)
        rec = buf.cpu().view(-1, 8)
        assert bool((rec[n_wg:] == 0).all())
        rec = rec[:n_wg]
        marks = rec[:, 2:6]
        assert bool((marks[:, 0] > 0).all()) and bool((marks[:, 1:] >= marks[:, :-1]).all()) and bool((marks[:, 3] <= rec[:, 1]).all())
        assert bool((rec[:, 6] >= 1).all()) and bool((rec[:, 6] <= rec[:, 7]).all()) and bool((rec[:, 7] == (N + 63) // 64).all())
