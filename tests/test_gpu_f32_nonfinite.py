"""The fp32 path on inputs that are not finite: a NaN reaches every output that depends on it, a logit
of minus infinity weighs nothing and one of plus infinity weighs one, as 1 / (1 + exp(-x)) has it."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa

pytestmark = pytest.mark.gpu

N, ROW = 70, 40  # three chunks of 32 keys, the row in the second


def _run(q, k, v, do, bias, causal):
    o, dq, dk, dv = (torch.zeros_like(q) for _ in range(4))
    rows = torch.zeros(q.shape[:3], device="cuda")
    sa.sigmoid_attn_fwd(q, k, v, o, bias, causal)
    sa.sigmoid_attn_bwd_bias_grad(q, k, v, do, dq, dk, dv, rows, bias, causal)
    return o, dq, dk, dv, rows


def _inputs(d):
    g = torch.Generator().manual_seed(d)
    return [torch.randn(1, 2, N, d, generator=g).cuda() for _ in range(4)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_nan_in_a_query_reaches_what_depends_on_it(d, causal):
    q, k, v, do = _inputs(d)
    q[:, :, ROW, 3] = float("nan")
    o, dq, dk, dv, rows = _run(q, k, v, do, -math.log(N), causal)
    keys = slice(0, ROW + 1) if causal else slice(None)
    assert o[:, :, ROW].isnan().all() and dq[:, :, ROW].isnan().all() and rows[:, :, ROW].isnan().all()
    assert dk[:, :, keys].isnan().all() and dv[:, :, keys].isnan().all()
    others = [i for i in range(N) if i != ROW]
    assert o[:, :, others].isfinite().all() and dq[:, :, others].isfinite().all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_nan_in_a_key_reaches_every_query_that_sees_it(d, causal):
    q, k, v, do = _inputs(d)
    k[:, :, ROW, 3] = float("nan")
    o, dq, dk, dv, rows = _run(q, k, v, do, -math.log(N), causal)
    seen = slice(ROW, None) if causal else slice(None)
    for x in (o, dq, rows):
        assert x[:, :, seen].isnan().all()
    assert dk[:, :, ROW].isnan().all() and dv[:, :, ROW].isnan().all()
    assert o[:, :, :ROW].isfinite().all() or not causal


@pytest.mark.parametrize("d", [64, 128])
def test_infinite_logits_weigh_nothing_or_one(d):
    q, k, v, do = _inputs(d)
    for x in _run(q, k, v, do, float("-inf"), False):
        assert (x == 0).all()
    o, dq, dk, dv, rows = _run(q, k, v, do, float("inf"), False)
    assert (dq == 0).all() and (dk == 0).all() and (rows == 0).all()
    # sums of N products with one in fp32
    assert (o.double() - v.double().sum(2, keepdim=True)).abs().max() <= N * 2.0 ** -24 * v.double().abs().sum(2).max()
    q[:, :, ROW], k[:] = -1e30, 1e30  # the products overflow: logits of minus infinity
    o, *_ = _run(q, k, v, do, 0.0, False)
    assert (o[:, :, ROW] == 0).all()
