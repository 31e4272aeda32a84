"""The forward kernel for few queries (32 rows per workgroup, the keys split over its waves and over
workgroups): parity with the fp64 oracle at the edges of its range."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa
from oracle import sattn_oracle as orc
from paper_2409_04431_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 2e-2  # of max |reference|: the bf16 bar of the library (P and O are rounded to bf16, 2^-9 each)


@pytest.mark.parametrize("B,H,Nq,Nk,d,causal,alibi,split", [
    (1, 1, 1, 2, 128, False, False, 1),        # one chunk for eight waves, two keys
    (2, 2, 1, 225, 64, False, True, 1),        # eight chunks, the last with one key
    (1, 3, 1, 1023, 128, False, True, 4),      # 32 chunks: the fewest that are split, ragged
    (1, 2, 33, 33 + 64 * 32, 64, True, True, 8),    # a second block of one row, masked chunks, split
    (1, 2, 100, 420, 128, True, False, 1),     # four blocks, the last of four rows
    (1, 16, 512, 2048, 128, True, False, 1),   # 256 blocks and four keys per query: the last that take this kernel
    (1, 16, 513, 2081, 128, True, False, 0),   # 272 blocks: the first that do not
    (1, 2, 257, 993, 64, True, False, 0),      # less than four keys per query
])
def test_few_queries_match_oracle(B, H, Nq, Nk, d, causal, alibi, split):
    g = torch.Generator().manual_seed(17 + Nq + Nk)
    q = torch.randn(B, H, Nq, d, generator=g).bfloat16()
    k, v = (torch.randn(B, H, Nk, d, generator=g).bfloat16() for _ in range(2))
    slopes = W.alibi_slopes(H) if alibi else None
    sl = slopes.cuda() if alibi else None
    bias = -math.log(Nk)
    Q, K, V = q.cuda(), k.cuda(), v.cuda()
    need = sa.sigmoid_attn_cross_aligned_fwd_workspace_bytes(B, H, Nq, Nk, d)
    cus, _ = sa.sattn_device_info()
    if cus == 256:
        assert need == (split * B * H * Nq * d * 4 if split > 1 else 0)
    o, o1 = (torch.full_like(Q, float("nan")) for _ in range(2))
    sa.sigmoid_attn_cross_aligned_fwd(Q, K, V, o, bias, causal, sl)
    ws = torch.full((max(need, 4) // 4,), float("nan"), dtype=torch.float32, device="cuda")
    sa.sigmoid_attn_cross_aligned_fwd_split(Q, K, V, o1, bias, causal, sl, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(o, o1)
    slo = slopes.double().numpy() if alibi else None
    ref = orc.sigmoid_attn_cross_fwd(q.double().numpy(), k.double().numpy(), v.double().numpy(), bias, causal, slo)
    err = abs(o.double().cpu().numpy() - ref).max() / abs(ref).max()
    assert err <= TOL, f"{err:.3e}"
    if need:
        with pytest.raises(sa.SattnError):
            sa.sigmoid_attn_cross_aligned_fwd_split(Q, K, V, o1, bias, causal, sl, workspace=ws[:-1])


def test_errors_name_the_function_that_was_called():
    q, k = (torch.zeros(1, 2, n, 64, device="cuda", dtype=torch.bfloat16) for n in (16, 90))
    small = [x[..., :32].contiguous() for x in (q, k)]
    for call, name in ((lambda: sa.sigmoid_attn_cross_fwd(small[0], small[1], small[1], small[0].clone(), 0.0), "sigmoid_attn_cross_fwd"),
                       (lambda: sa.sigmoid_attn_cross_aligned_fwd(q, k, k, q.clone(), 0.0, True), "sigmoid_attn_cross_aligned_fwd"),
                       (lambda: sa.sigmoid_attn_cross_aligned_fwd_split(q, k, k, q.clone(), 0.0, True),
                        "sigmoid_attn_cross_aligned_fwd_split")):
        with pytest.raises(sa.SattnError, match=rf"^{name} failed"):
            call()


@pytest.mark.parametrize("B,H,Nq,Nk,d,causal,alibi,takes", [
    (1, 2, 1, 1300, 128, False, False, True),     # few blocks, more keys than a wave walks alone
    (3, 12, 1, 1201, 64, False, True, True),      # 36 blocks, up to a quarter of the units
    (2, 16, 40, 2600, 64, True, False, True),     # two blocks a head, the second of eight rows
    (9, 8, 32, 1056, 128, True, True, False),     # 72 blocks, one a head: the kernel of 128 rows
    (9, 8, 1, 1000, 128, False, False, True),     # the same with fewer than 32 chunks of keys
])
def test_c_entry_points_without_a_workspace_match_oracle(B, H, Nq, Nk, d, causal, alibi, takes):
    """sigmoid_attn_cross_aligned_fwd (and sigmoid_attn_cross_fwd) as C callers have them: the keys of a block are
    not split over workgroups, and where that would not pay the other forward kernels run."""
    if sa.sattn_device_info()[0] != 256:
        pytest.skip("sizes chosen for 256 compute units")
    lib = sa.load_library()
    g = torch.Generator().manual_seed(23 + Nk)
    q = torch.randn(B, H, Nq, d, generator=g).bfloat16()
    k, v = (torch.randn(B, H, Nk, d, generator=g).bfloat16() for _ in range(2))
    slopes = W.alibi_slopes(H) if alibi else None
    sl = slopes.cuda() if alibi else None
    bias = -math.log(Nk)
    Q, K, V = q.cuda(), k.cuda(), v.cuda()
    stream = torch.cuda.current_stream().cuda_stream
    none = [None] * 4  # contiguous

    def aligned():
        o = torch.full_like(Q, float("nan"))
        assert lib.sigmoid_attn_cross_aligned_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), o.data_ptr(), B, H, Nq, Nk, d, 0, bias,
                                                  int(causal), sl.data_ptr() if alibi else None, *none, stream) == 0
        torch.cuda.synchronize()
        return o

    o = aligned()
    ref = orc.sigmoid_attn_cross_fwd(q.double().numpy(), k.double().numpy(), v.double().numpy(), bias, causal,
                                     slopes.double().numpy() if alibi else None)
    err = abs(o.double().cpu().numpy() - ref).max() / abs(ref).max()
    assert err <= TOL, f"{err:.3e}"
    if not causal and not alibi:
        o1 = torch.full_like(Q, float("nan"))
        assert lib.sigmoid_attn_cross_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), o1.data_ptr(), B, H, Nq, Nk, d, 0, bias, *none,
                                          stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(o, o1)
    if not takes:
        try:
            sa.sattn_set_fwd_waves(4)  # keeps the call to the kernels of 128 rows, whose bits are the same in every shape
            wide = aligned()
        finally:
            sa.sattn_set_fwd_waves(0)
        assert torch.equal(o, wide)


def test_clock_probe_records_the_workgroups_of_few_queries():
    B, H, Nk, d = 1, 4, 1100, 64
    q = torch.randn(B, H, 1, d, device="cuda").bfloat16()
    k, v = (torch.randn(B, H, Nk, d, device="cuda").bfloat16() for _ in range(2))
    splits = max(1, sa.sigmoid_attn_cross_aligned_fwd_workspace_bytes(B, H, 1, Nk, d) // (B * H * d * 4))
    buf = torch.zeros(8 * 64, dtype=torch.int64, device="cuda")
    try:
        sa.sattn_set_clock_probe(buf)
        sa.sigmoid_attn_cross_fwd(q, k, v, torch.empty_like(q), -7.0)
        torch.cuda.synchronize()
    finally:
        sa.sattn_set_clock_probe(None)
    rec = buf.cpu().view(-1, 8)
    assert (rec[:B * H * splits, 0] > 0).all() and (rec[B * H * splits:] == 0).all()
    marks = rec[:B * H * splits, 2:6]
    assert (marks[:, 1:] >= marks[:, :-1]).all() and (marks[:, 3] <= rec[:B * H * splits, 1]).all()
