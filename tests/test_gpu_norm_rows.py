"""The norm over concatenated heads at the row widths where tokens begin to share a wave and where a wave
takes another chunk per lane, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d", [(1, 64), (2, 64), (1, 128), (3, 64), (2, 128), (4, 64), (5, 64), (8, 64), (9, 64), (16, 64), (17, 128)])
@pytest.mark.parametrize("kind", ["layer", "rms"])
def test_norm_rows(H, d, kind):
    B, N = 3, 37  # 111 tokens: the last workgroup of 4, 8 or 16 is not full
    g = torch.Generator().manual_seed(H * d)
    x, dy = (torch.randn(B, H, N, d, generator=g).bfloat16() for _ in range(2))
    X, DY = x.cuda(), dy.cuda()
    y, dx = (torch.full_like(X, float("nan")) for _ in range(2))
    st = torch.full((B, N, 2), float("nan"), device="cuda")
    sa.sattn_headconcat_norm_fwd(X, y, st, kind=kind)
    sa.sattn_headconcat_norm_bwd(X, DY, st, dx, kind=kind)
    ry, _, _ = orc.headconcat_norm_fwd(x.double().numpy(), kind)
    rdx = orc.headconcat_norm_bwd(x.double().numpy(), dy.double().numpy(), kind)
    for got, ref in ((y, ry), (dx, rdx)):  # one bf16 rounding, 2^-9 of the largest value of a binade
        assert np.abs(got.double().cpu().numpy() - ref).max() <= 4e-3 * np.abs(ref).max()
