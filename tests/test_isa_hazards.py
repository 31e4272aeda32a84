"""The hand-placed MFMAs must keep the data-hazard distances the compiler cannot enforce for
inline asm.  Checked on the gfx950 assembly of the library sources (no GPU needed)."""
import re

import pytest

from paper_2409_04431_amd import isa_check

_HEAD = "kernel_x:\n"
_MFMA = "\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], a[4:7], v[0:15]\n\t;;#ASMEND\n"


def test_scanner_flags_valu_write_right_before_asm_mfma():
    txt = _HEAD + "\tv_accvgpr_read_b32 v21, a9\n" + _MFMA + "\ts_endpgm\n"
    msgs = isa_check.check_text(txt)
    assert len(msgs) == 1 and "rule A" in msgs[0]
    ok = _HEAD + "\tv_accvgpr_read_b32 v21, a9\n\ts_nop 1\n" + _MFMA + "\ts_endpgm\n"
    assert isa_check.check_text(ok) == []
    ok2 = _HEAD + "\tv_accvgpr_read_b32 v21, a9\n\tv_add_u32_e32 v40, v41, v42\n\ts_add_i32 s0, s0, 1\n" + _MFMA + "\ts_endpgm\n"
    assert isa_check.check_text(ok2) == []


def test_scanner_flags_early_read_of_asm_mfma_result():
    txt = _HEAD + _MFMA + "\tv_add_f32_e32 v30, v31, v32\n\tv_accvgpr_write_b32 a100, v15\n\ts_endpgm\n"
    msgs = isa_check.check_text(txt)
    assert len(msgs) == 1 and "rule B" in msgs[0]
    ok = _HEAD + _MFMA + "\ts_nop 15\n\tv_accvgpr_write_b32 a100, v15\n\ts_endpgm\n"
    assert isa_check.check_text(ok) == []
    # an independent MFMA in between occupies the matrix pipe for its 8 passes
    other = "\tv_mfma_f32_32x32x16_bf16 v[64:79], v[20:23], a[4:7], v[64:79]\n"
    ok2 = _HEAD + _MFMA + other + other + "\tv_accvgpr_write_b32 a100, v15\n\ts_endpgm\n"
    assert isa_check.check_text(ok2) == []


def test_scanner_ignores_compiler_emitted_mfma():
    txt = _HEAD + "\tv_accvgpr_read_b32 v21, a9\n\tv_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], a[4:7], v[0:15]\n\ts_endpgm\n"
    assert isa_check.check_text(txt) == []


def test_scanner_flags_m0_write_outside_asm_next_to_lds_dma():
    dma = "\t;;#ASMSTART\n\ts_mov_b32 m0, s5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v3, s[8:9]\n\t;;#ASMEND\n"
    more = "\t;;#ASMSTART\n\tglobal_load_lds_dwordx4 v4, s[8:9] offset:1024\n\t;;#ASMEND\n"
    assert isa_check.check_text(_HEAD + dma + "\tv_add_u32_e32 v40, v41, v42\n" + more + "\ts_endpgm\n") == []
    msgs = isa_check.check_text(_HEAD + dma + "\ts_mov_b32 m0, -1\n" + more + "\ts_endpgm\n")
    assert len(msgs) == 1 and "rule C" in msgs[0]
    # without such loads in the function the compiler may use M0 as it likes
    assert isa_check.check_text(_HEAD + "\ts_mov_b32 m0, -1\n\ts_endpgm\n") == []


_FILL = "".join(f"\tv_add_f32_e32 v{40 + i}, v31, v32\n" for i in range(12))  # wait states of other work


def test_scanner_follows_the_back_edge_of_a_loop():
    # the loop's last MFMA is read by the first instruction of the next trip
    loop = ".LBB0_1:\n{first}" + _FILL + "\ts_cmp_lg_u32 s0, s1\n{last}\ts_cbranch_scc1 .LBB0_1\n" + _FILL + "\ts_endpgm\n"
    msgs = isa_check.check_text(_HEAD + loop.format(first="\tv_exp_f32_e32 v33, v3\n", last=_MFMA))
    assert len(msgs) == 1 and "rule B" in msgs[0]
    assert isa_check.check_text(_HEAD + loop.format(first=_FILL + "\tv_exp_f32_e32 v33, v3\n", last=_MFMA)) == []
    # the loop's last vector instruction writes what the next trip's first MFMA reads
    msgs = isa_check.check_text(_HEAD + loop.format(first=_MFMA, last="\tv_mov_b32_e32 v21, v9\n"))
    assert len(msgs) == 1 and "rule A" in msgs[0]
    assert isa_check.check_text(_HEAD + loop.format(first=_MFMA, last="\tv_mov_b32_e32 v21, v9\n\ts_nop 1\n")) == []


def test_scanner_follows_taken_branches_and_reads_past_an_early_end():
    body = _MFMA + "\ts_cbranch_scc1 .LBB0_2\n" + _FILL + "\ts_endpgm\n.LBB0_2:\n{read}" + "\ts_endpgm\n"
    msgs = isa_check.check_text(_HEAD + body.format(read="\tv_exp_f32_e32 v33, v3\n"))
    assert len(msgs) == 1 and "rule B" in msgs[0]
    assert isa_check.check_text(_HEAD + body.format(read=_FILL + "\tv_exp_f32_e32 v33, v3\n")) == []
    # what follows an unconditional branch in the listing is not what runs after it
    jump = _MFMA + "\ts_branch .LBB0_4\n.LBB0_3:\n\tv_exp_f32_e32 v33, v3\n.LBB0_4:\n" + _FILL + "\ts_endpgm\n"
    assert isa_check.check_text(_HEAD + jump) == []


def test_sigmoid_backward_kernels_at_d64_leave_room_for_a_second_workgroup():
    """Two workgroups of 256 threads share a compute unit up to 256 registers, which the pinned kernels at
    d = 64 (template arguments: 64, [pass,] causal, ALiBi, softmax, ...) stay below by themselves."""
    regs = isa_check.kernel_registers(isa_check.compile_to_asm())
    ours = {k: n for k, n in regs.items()
            if re.search(r"attn_bwd_kernelILi64ELi\dELb\dELb\dELb0E|attn_bwd_merged_kernelILi64ELb\dELb\dELb0E", k)}
    assert len(ours) == 32 and max(ours.values()) <= 256, {k: n for k, n in ours.items() if n > 256}


def test_library_kernels_have_no_mfma_hazard():
    asm = isa_check.compile_to_asm()
    n_asm_mfma = sum(1 for _, insts in isa_check.parse_functions(asm) for i in insts if i.is_mfma and i.in_asm)
    assert n_asm_mfma > 1000  # the pinned forward and backward steps are in there
    assert isa_check.check_text(asm) == []
