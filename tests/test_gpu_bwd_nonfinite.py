"""The bf16 backward on inputs that are not finite, in sequences whose length is no multiple of a tile: an infinite
query element makes infinite logits, which weigh nothing or one, as 1 / (1 + exp(-x)) has it, so that its row of
dS is zero.  Rows past the end of a sequence must not add a NaN to what the oracle has as finite, and the
kernel that holds a head whole answers as the two passes do."""
import math

import numpy as np
import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2  # P, dS and the outputs are rounded to bf16
H = 17
WHOLE = [(9, 64, 129), (9, 64, 250), (21, 64, 33), (9, 128, 33), (9, 128, 97)]  # batch, d, N: all or most heads (256
                                                                                # compute units) take one workgroup

# Two workgroups a head: all heads, or (64, 250 tokens) the 101 beyond one round of 256
SHARED = [(3, 64, 33), (3, 64, 100), (21, 64, 250), (3, 128, 33), (3, 128, 97)]


def _inputs(B, d, N):
    g = torch.Generator().manual_seed(1000 * B + 10 * N + d)
    return [torch.randn(B, H, N, d, generator=g).bfloat16() for _ in range(4)]


def _run(x, causal):
    """dQ, dK, dV of the choice and of two launches."""
    dev, both = [t.cuda() for t in x], []
    try:
        for mode in (0, 2):
            sa.sattn_set_bwd_merged(mode)
            both.append([torch.full_like(dev[0], 7.0) for _ in range(3)])
            sa.sigmoid_attn_bwd(*dev, *both[-1], -math.log(x[0].shape[2]), causal)
    finally:
        sa.sattn_set_bwd_merged(0)
    return both


def _compare(choice, two, causal):
    """Bit for bit.  A masked pair's zero times the infinite element is a NaN in dK of both, in the kernel that holds a
    head whole for the keys of a 32-row chunk, in the passes for those of a longer block."""
    for i, (a, b) in enumerate(zip(choice, two)):
        if causal and i == 1:
            a = torch.where(b.isnan(), b, a)
        assert bool((a.isnan() == b.isnan()).all()), "dQ dK dV".split()[i]
        assert bool((a[~a.isnan()] == b[~b.isnan()]).all()), "dQ dK dV".split()[i]


def _as_oracle(got, ref):
    """Equal where the oracle has an infinity or a NaN, within the bf16 bar elsewhere."""
    got, finite = got.float().cpu().numpy(), np.isfinite(ref)
    assert np.array_equal(got[~finite], ref[~finite].astype(np.float32), equal_nan=True)
    assert np.abs(got[finite] - ref[finite]).max(initial=0.0) <= TOL * np.abs(ref[finite]).max(initial=0.0)


def _oracle(x, b, causal):
    with np.errstate(all="ignore"):
        return orc.sigmoid_attn_bwd(*(t[b:b + 1, :2].contiguous() for t in x), -math.log(x[0].shape[2]), causal)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("row", [0, 20, -1])
@pytest.mark.parametrize("B,d,N", WHOLE)
def test_infinite_query_element_where_one_workgroup_holds_a_head(B, d, N, row, causal):
    x = _inputs(B, d, N)
    x[0][:, :, row, 3] = math.inf
    choice, two = _run(x, causal)
    assert bool(choice[0].isfinite().all())
    _compare(choice, two, causal)
    _as_oracle(choice[0][:1, :2], _oracle(x, 0, causal)[0])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("row", [0, -1])
@pytest.mark.parametrize("B,d,N", SHARED)
def test_infinite_query_element_where_two_workgroups_share_a_head(B, d, N, row, causal):
    x = _inputs(B, d, N)
    x[0][:, :, row, 3] = math.inf
    choice, two = _run(x, causal)
    assert bool(choice[0].isfinite().all())
    _compare(choice, two, causal)
    _as_oracle(choice[0][-1:, :2], _oracle(x, B - 1, causal)[0])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,N", [(64, 33), (64, 100), (128, 70)])
def test_infinite_query_element_and_the_bias_gradient(d, N, causal):
    x = _inputs(2, d, N)
    x[0][:, :, N // 2, 3] = math.inf
    q, k, v, do = (t.cuda() for t in x)
    both = []
    try:
        for mode in (0, 2):
            sa.sattn_set_bwd_merged(mode)
            grads, rows, db = [torch.zeros_like(q) for _ in range(3)], torch.full((2, H, N), 7.0, device="cuda"), torch.zeros(2, H, device="cuda")
            sa.sigmoid_attn_bwd_bias_grad(q, k, v, do, *grads, rows, -math.log(N), causal, None, db=db)
            both.append((grads[0], rows, db))
    finally:
        sa.sattn_set_bwd_merged(0)
    for a, b in zip(*both):
        assert bool(a.isfinite().all()) and torch.equal(a, b)
    assert bool((both[0][1][:, :, N // 2] == 0).all())


@pytest.mark.parametrize("tensor", [1, 2, 3], ids=["k", "v", "dout"])
@pytest.mark.parametrize("row", [0, -1])
@pytest.mark.parametrize("B,d,N", WHOLE + SHARED)
def test_infinite_key_value_or_output_gradient_element(B, d, N, row, tensor):
    """Positive rows throughout, so that the oracle's sums are infinities of one sign and not differences of two."""
    x = [t.abs() for t in _inputs(B, d, N)]
    x[tensor][:, :, row, 3] = math.inf
    dev = [t.cuda() for t in x]
    grads = [torch.full_like(dev[0], 7.0) for _ in range(3)]
    sa.sigmoid_attn_bwd(*dev, *grads, -math.log(N), False)
    for b in (0, B - 1):
        for g, ref in zip(grads, _oracle(x, b, False)):
            _as_oracle(g[b:b + 1, :2], ref)
