"""Both passes of the backward in one grid where the bias gradient is asked for and for packed sequences:
bit-equal to the two launches."""
import math

import pytest
import torch

import paper_2409_04431_amd as sa


def test_one_grid_where_the_paired_launches_leave_places_empty():
    # 256 compute units (what the library assumes without a device); workgroups per pass and unit
    assert sa.sattn_bwd_merged(3, 16, 2048, True) and sa.sattn_bwd_merged(5, 16, 2048, True)      # 3, 5
    assert not sa.sattn_bwd_merged(4, 16, 2048, True) and not sa.sattn_bwd_merged(64, 12, 2048, True)  # 4, 48
    assert not sa.sattn_bwd_merged(3, 16, 2176, True)     # 17 blocks per head: not dealt out in pairs
    assert not sa.sattn_bwd_merged(3, 16, 2048, False)
    # equal workgroups: only where one grid takes fewer rounds
    assert sa.sattn_bwd_merged(3, 16, 1024) and not sa.sattn_bwd_merged(4, 16, 1024) and not sa.sattn_bwd_merged(39, 12, 64, True)


def test_the_choice_is_reported_for_the_head_dimension_and_for_packed_sequences():
    # workgroups per pass and unit: 2, 6, 6.25
    assert not sa.sattn_bwd_merged(4, 16, 1024) and sa.sattn_bwd_merged(4, 16, 1024, d=64)
    assert sa.sattn_bwd_merged(12, 16, 1024, d=64) and not sa.sattn_bwd_merged(25, 64, 128, d=64)
    # packed: up to 6, at d = 64 up to 9
    assert sa.sattn_bwd_merged(12, 16, 1024, packed=True) and not sa.sattn_bwd_merged(25, 64, 128, packed=True)
    assert sa.sattn_bwd_merged(18, 16, 1024, d=64, packed=True) and not sa.sattn_bwd_merged(37, 64, 128, d=64, packed=True)
    lib = sa.load_library()
    assert lib.sattn_bwd_one_grid(0, 1, 16, 64, 0, 0) == -2 and lib.sattn_bwd_one_grid(1, 1, 16, 32, 0, 0) == -3


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal,alibi", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("lengths", [[1], [300, 300], [129, 640, 0, 33]])
def test_bias_gradient_in_one_grid_equals_two_launches(d, causal, alibi, lengths):
    H, total, longest = 2, sum(lengths), max(lengths)
    g = torch.Generator().manual_seed(total + d)
    q, k, v, do = (torch.randn(total, H, d, generator=g).bfloat16().cuda() for _ in range(4))
    cu = torch.tensor([sum(lengths[:i]) for i in range(len(lengths) + 1)], dtype=torch.int32, device="cuda")
    slopes = torch.tensor([0.5, 0.03], device="cuda") if alibi else None
    dense = len(set(lengths)) == 1
    view = (lambda x: x.view(len(lengths), longest, H, d).transpose(1, 2)) if dense else None
    out = []
    try:
        for mode in (1, 2):
            sa.sattn_set_bwd_merged(mode)
            res = [torch.full_like(q, float("nan")) for _ in range(3)]
            rows = torch.full((H, total), float("nan"), device="cuda")
            db = torch.full((len(lengths), H), float("nan"), device="cuda")
            sa.sigmoid_attn_varlen_bwd_bias_grad(q, k, v, do, *res, rows, cu, longest, -math.log(longest + 1), causal, slopes, db=db)
            out.append(res + [rows, db])
            if dense:
                res = [torch.full_like(q, float("nan")) for _ in range(3)]
                rows = torch.full((len(lengths), H, longest), float("nan"), device="cuda")
                sa.sigmoid_attn_bwd_bias_grad(*(view(x) for x in (q, k, v, do)), *(view(x) for x in res), rows,
                                              -math.log(longest + 1), causal, slopes)
                out[-1] += res + [rows]
    finally:
        sa.sattn_set_bwd_merged(0)
    for x, y in zip(*out):
        assert torch.equal(x, y) and not torch.isnan(x).any()
