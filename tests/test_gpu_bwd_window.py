"""The dK/dV pass at d = 64, whose steps run the second products first and fetch their operands through a
window of four fragments: parity with the fp64 oracle around the edges of its 32-row chunks, 64-row tiles
and 128-row blocks."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc
from paper_2409_04431_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 2e-2  # of max |reference|: the bf16 bar of the library (P, dS and the results are rounded to bf16, 2^-9 each)


@pytest.mark.parametrize("N", [1, 31, 33, 64, 65, 96, 127, 129, 191, 192, 257, 320, 449, 512])
@pytest.mark.parametrize("causal,alibi", [(False, False), (True, False), (False, True), (True, True)])
def test_dkdv_at_d64_matches_oracle(N, causal, alibi):
    B, H, d = 1, 2, 64
    g = torch.Generator().manual_seed(1000 * causal + 500 * alibi + N)
    q, k, v, do = (torch.randn(B, H, N, d, generator=g).bfloat16() for _ in range(4))
    slopes = W.alibi_slopes(H) if alibi else None
    bias = -math.log(N)
    dk, dv = (torch.full((B, H, N, d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sa.sigmoid_attn_bwd_dkdv(q.cuda(), k.cuda(), v.cuda(), do.cuda(), dk, dv, bias, causal, slopes.cuda() if alibi else None)
    torch.cuda.synchronize()
    _, rk, rv = orc.sigmoid_attn_bwd(q, k, v, do, bias, causal, slopes)
    for x, r in ((dk, rk), (dv, rv)):
        err = abs(x.double().cpu().numpy() - r).max() / max(abs(r).max(), 1e-12)
        assert err <= TOL, f"{err:.3e}"
