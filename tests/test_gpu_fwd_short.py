"""The forward that holds a head whole (up to 256 keys at d = 64, 128 at d = 128): bit-equal to the kernels that
stream the keys, the oracle's result within the bf16 bar, nothing written past the rows of a sequence."""
import math

import numpy as np
import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc

pytestmark = pytest.mark.gpu
TOL = 2e-2  # P and the output are rounded to bf16
SIZES = [(64, n) for n in (1, 31, 32, 33, 64, 65, 127, 128, 129, 160, 193, 255, 256)] + [(128, n) for n in (1, 33, 64, 97, 128)]


def _both(call, like):
    out = []
    try:
        for waves in (4, 0):  # four waves that stream the keys, the choice
            sa.sattn_set_fwd_waves(waves)
            o = torch.full_like(like, float("nan"))
            call(o)
            torch.cuda.synchronize()
            out.append(o)
    finally:
        sa.sattn_set_fwd_waves(0)
    return out


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,N", SIZES)
@pytest.mark.parametrize("B", [2, 9])  # 17 heads each: on either side of the rule's line at d = 64, N > 128
def test_dense_equals_the_streaming_kernel_and_the_oracle(B, d, N, causal):
    g = torch.Generator().manual_seed(100 * N + d)
    q, k, v = (torch.randn(B, N, 17, d, generator=g).bfloat16().cuda().transpose(1, 2) for _ in range(3))
    bias = -math.log(max(N, 2))
    other, o = _both(lambda o: sa.sigmoid_attn_fwd(q, k, v, o, bias, causal), q)
    assert torch.equal(other, o) and not torch.isnan(o).any()
    ref = orc.sigmoid_attn_fwd(*(x[:1, :2].contiguous().cpu() for x in (q, k, v)), bias, causal)
    assert np.abs(o[:1, :2].float().cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,lengths", [(64, [256, 1, 0, 33, 250]), (64, [128, 64, 127]), (128, [128, 5, 0, 96])])
def test_packed_equals_the_streaming_kernel_and_leaves_other_rows_alone(d, lengths, causal):
    total = sum(lengths)
    g = torch.Generator().manual_seed(total + d)
    q, k, v = (torch.randn(total + 64, 64, d, generator=g).bfloat16().cuda() for _ in range(3))
    cu = torch.tensor([sum(lengths[:i]) for i in range(len(lengths) + 1)], dtype=torch.int32, device="cuda")
    bias = torch.tensor([-math.log(max(n, 2)) for n in lengths], dtype=torch.float32, device="cuda")
    other, o = _both(lambda o: sa.sigmoid_attn_varlen_fwd(q, k, v, o, cu, max(lengths), 0.0, causal, None, bias_per_seq=bias), q)
    assert torch.equal(other[:total], o[:total]) and not torch.isnan(o[:total]).any()
    assert torch.isnan(o[total:]).all()
