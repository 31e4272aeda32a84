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
@pytest.mark.parametrize("B", [2, 9, 18])  # 17 heads each: on either side of the rule's lines at d = 64, N > 128, and
def test_dense_equals_the_streaming_kernel_and_the_oracle(B, d, N, causal):  # (causal, up to 48 tokens) at d = 128
    streams = (d == 64 and N > 128 and (B == 2 or (B == 18 and N > 192 and not causal))) or (d == 128 and causal and N <= 48 and B < 18)
    assert sa.sattn_fwd_short(B, 17, N, d, causal) == (0 if streams else 8 if N > 128 else 4)
    g = torch.Generator().manual_seed(100 * N + d)
    q, k, v = (torch.randn(B, N, 17, d, generator=g).bfloat16().cuda().transpose(1, 2) for _ in range(3))
    bias = -math.log(max(N, 2))
    other, o = _both(lambda o: sa.sigmoid_attn_fwd(q, k, v, o, bias, causal), q)
    assert torch.equal(other, o) and not torch.isnan(o).any()
    ref = orc.sigmoid_attn_fwd(*(x[:1, :2].contiguous().cpu() for x in (q, k, v)), bias, causal)
    assert np.abs(o[:1, :2].float().cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,lengths", [(64, [256, 1, 0, 33, 250]), (64, [256, 1, 0, 250]), (64, [128, 64, 127]), (128, [128, 5, 0, 96])])
def test_packed_equals_the_streaming_kernel_and_leaves_other_rows_alone(d, lengths, causal):
    total = sum(lengths)
    assert bool(sa.sattn_fwd_short(len(lengths), 64, max(lengths), d, causal)) == (causal or len(lengths) != 5)
    g = torch.Generator().manual_seed(total + d)
    q, k, v = (torch.randn(total + 64, 64, d, generator=g).bfloat16().cuda() for _ in range(3))
    cu = torch.tensor([sum(lengths[:i]) for i in range(len(lengths) + 1)], dtype=torch.int32, device="cuda")
    bias = torch.tensor([-math.log(max(n, 2)) for n in lengths], dtype=torch.float32, device="cuda")
    other, o = _both(lambda o: sa.sigmoid_attn_varlen_fwd(q, k, v, o, cu, max(lengths), 0.0, causal, None, bias_per_seq=bias), q)
    assert torch.equal(other[:total], o[:total]) and not torch.isnan(o[:total]).any()
    assert torch.isnan(o[total:]).all()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("tensor", [0, 1, 2], ids=["q", "k", "v"])
@pytest.mark.parametrize("row", [0, -1])
@pytest.mark.parametrize("B,d,N", [(9, 64, 129), (9, 64, 250), (2, 64, 33), (2, 64, 100), (18, 128, 33), (2, 128, 97)])
def test_infinite_elements(B, d, N, row, tensor, causal):
    """Rows past the end repeat a row or are zeros and must not make a NaN of what is finite: the oracle's infinities and
    NaNs without a mask, and in either case the streaming kernel's numbers where it has one (the zero weight of a masked
    pair or of its repeated last row times an infinite element of V is a NaN there)."""
    assert sa.sattn_fwd_short(B, 17, N, d, causal) > 0
    g = torch.Generator().manual_seed(N + d)
    x = [torch.randn(B, 17, N, d, generator=g).bfloat16() for _ in range(3)]
    if tensor:  # positive rows: sums are infinities of one sign and not differences of two
        x = [t.abs() for t in x]
    x[tensor][:, :, row, 3] = math.inf
    dev = [t.cuda() for t in x]
    other, o = _both(lambda o: sa.sigmoid_attn_fwd(*dev, o, -math.log(N), causal), dev[0])
    known = ~other.isnan()
    assert torch.equal(other[known], o[known])
    with np.errstate(all="ignore"):
        ref = orc.sigmoid_attn_fwd(*(t[:1, :2].contiguous() for t in x), -math.log(N), causal)
    got, finite = o[:1, :2].float().cpu().numpy(), np.isfinite(ref)
    if not causal:
        assert np.array_equal(got[~finite], ref[~finite].astype(np.float32), equal_nan=True)
    finite &= ~np.isnan(got) if causal else True
    assert np.abs(got[finite] - ref[finite]).max(initial=0.0) <= TOL * np.abs(ref[finite]).max(initial=0.0)
