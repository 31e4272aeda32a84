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


def test_shared_heads_at_d64_split_once_more_or_with_room_for_less():
    # 3 x 17 key blocks: 8 workgroups a group make 408, more than one and fewer than two per compute unit
    B, H, N, d = 3, 16, 2100, 64
    if sa.sattn_device_info()[0] != 256:
        pytest.skip("sizes chosen for 256 compute units")
    g = torch.Generator(device="cuda").manual_seed(4)
    q, do = (torch.randn(B, H, N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn(B, 1, N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    need = sa.sigmoid_attn_mqa_bwd_workspace_bytes(B, H, 1, N, d)
    assert need == 2 * 16 * B * N * d * 4
    out = []
    for room in (need, need // 2):
        ws = torch.full((room,), 255, dtype=torch.uint8, device="cuda")
        out.append([torch.full_like(x, float("nan")) for x in (q, k, v)])
        sa.sigmoid_attn_mqa_bwd_split(q, k, v, do, *out[-1], -math.log(N), workspace=ws)
    ref = [torch.empty_like(x) for x in (q, k, v)]
    sa.sigmoid_attn_mqa_bwd(q, k, v, do, *ref, -math.log(N))
    with pytest.raises(sa.SattnError):
        sa.sigmoid_attn_mqa_bwd_split(q, k, v, do, *out[0], -math.log(N), workspace=ws[: need // 2 - 16])
    for got in out:
        assert torch.equal(got[0], ref[0])
        for x, r in zip(got[1:], ref[1:]):  # two bf16 roundings of sums in another order
            assert ((x.double() - r.double()).abs().amax(-1) / r.double().abs().amax(-1)).max() <= 2 ** -7


@pytest.mark.parametrize("B,Hkv,N,causal", [
    (33, 16, 100, True),    # 528 blocks: more than two per compute unit, so only the further split would take a workspace
    (17, 16, 65, False),    # 272: the same without the mask
])
def test_shared_heads_at_d64_without_room_run_unsplit_where_only_the_further_split_asks_for_it(B, Hkv, N, causal):
    if sa.sattn_device_info()[0] != 256:
        pytest.skip("sizes chosen for 256 compute units")
    H, d = 2 * Hkv, 64
    g = torch.Generator(device="cuda").manual_seed(6)
    q, do = (torch.randn(B, H, N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn(B, Hkv, N, d, generator=g, device="cuda").bfloat16() for _ in range(2))
    need = sa.sigmoid_attn_mqa_bwd_workspace_bytes(B, H, Hkv, N, d, causal=causal)
    assert need == 2 * 2 * B * Hkv * N * d * 4
    ref = [torch.empty_like(x) for x in (q, k, v)]
    sa.sigmoid_attn_mqa_bwd(q, k, v, do, *ref, -math.log(N), causal)
    for ws in (torch.empty(0, dtype=torch.uint8, device="cuda"), torch.empty(need - 16, dtype=torch.uint8, device="cuda"),
               torch.empty(need + 4, dtype=torch.uint8, device="cuda")[4:]):  # none, too little, misaligned
        got = [torch.full_like(x, float("nan")) for x in (q, k, v)]
        sa.sigmoid_attn_mqa_bwd_split(q, k, v, do, *got, -math.log(N), causal, workspace=ws)
        for x, r in zip(got, ref):
            assert torch.equal(x, r)
