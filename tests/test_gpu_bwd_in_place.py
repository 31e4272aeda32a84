"""dQ written over Q or dO: the dK/dV pass, which reads all their rows, is through before, also where the
two passes would share a grid.  Bit-equal to the call with a buffer of its own."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["q", "dout"])
@pytest.mark.parametrize("dtype,B,H,Hkv,N,d,causal", [
    (torch.float32, 2, 4, 4, 333, 64, True),
    (torch.float32, 1, 4, 2, 257, 128, False),
    (torch.bfloat16, 4, 12, 12, 700, 64, False),    # one grid with a buffer of its own
    (torch.bfloat16, 1, 8, 8, 1024, 128, True),     # the same
])
def test_dq_over_an_input_of_the_backward(dtype, over, B, H, Hkv, N, d, causal):
    g = torch.Generator(device="cuda").manual_seed(N)
    q, do = (torch.randn(B, H, N, d, generator=g, device="cuda").to(dtype) for _ in range(2))
    k, v = (torch.randn(B, Hkv, N, d, generator=g, device="cuda").to(dtype) for _ in range(2))
    bwd = sa.sigmoid_attn_bwd if Hkv == H else sa.sigmoid_attn_mqa_bwd
    ref = [torch.empty_like(x) for x in (q, k, v)]
    bwd(q, k, v, do, *ref, -math.log(N), causal)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = q if over == "q" else do
    bwd(q, k, v, do, dq, dk, dv, -math.log(N), causal)
    for x, y in zip((dq, dk, dv), ref):
        assert torch.equal(x, y)


@pytest.mark.parametrize("over", ["q", "dout"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_dq_over_an_input_of_the_packed_backward(dtype, over):
    H, d, lengths = 4, 64, (129, 400, 33)
    starts = [sum(lengths[:i]) for i in range(len(lengths) + 1)]
    g = torch.Generator(device="cuda").manual_seed(8)
    q, k, v, do = (torch.randn(starts[-1], H, d, generator=g, device="cuda").to(dtype) for _ in range(4))
    cu = torch.tensor(starts, dtype=torch.int32, device="cuda")
    ref = [torch.empty_like(x) for x in (q, k, v)]
    sa.sigmoid_attn_varlen_bwd(q, k, v, do, *ref, cu, 400, -5.0)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = q if over == "q" else do
    sa.sigmoid_attn_varlen_bwd(q, k, v, do, dq, dk, dv, cu, 400, -5.0)
    for x, y in zip((dq, dk, dv), ref):
        assert torch.equal(x, y)
