"""The address emulator behind the build-time check of the hand-scheduled kernels (paper_2504_20039_amd/isa_emu.py), on small
hand-written instruction sequences whose results are worked out by hand."""
import numpy as np
import pytest

from paper_2504_20039_amd import check_isa
from paper_2504_20039_amd.isa_emu import Emu, Poison


def run(text, kernarg=b"\0" * 64, wg=3, tid_base=64):
    seen = []
    e = Emu(text.strip().splitlines(), kernarg, wg, tid_base, lambda emu, op, o, t: seen.append((op, t)))
    e.run()
    return e, seen


def test_scalar_arithmetic_carries_and_selects():
    e, _ = run("""
        s_mov_b32 s4, 0xfffffff0
        s_add_u32 s5, s4, 0x20
        s_addc_u32 s6, 0, 0
        s_mul_i32 s7, s2, 100
        s_cmp_lt_i32 s7, 301
        s_cselect_b32 s8, 11, 22
        s_lshl_b64 s[10:11], s[4:5], 4
        s_addk_i32 s7, 0xff00
        s_min_i32 s9, s7, -1
        s_endpgm
    """)
    assert e.s["s5"] == 0x10 and e.s["s6"] == 1                 # the carry of the 32-bit addition
    assert e.s["s8"] == 11                                        # 3 * 100 < 301
    assert e.get64("s[10:11]") == ((0xfffffff0 | (0x10 << 32)) << 4) & (2**64 - 1)
    assert e.s["s7"] == 300 - 256 and e.s["s9"] == 0xFFFFFFFF   # a signed 16-bit constant; the signed minimum


def test_a_counted_loop_and_lane_arithmetic():
    e, seen = run("""
        s_mov_b32 s4, 0
        v_mbcnt_lo_u32_b32 v1, -1, 0
        v_mbcnt_hi_u32_b32 v1, -1, v1
        v_lshrrev_b32_e32 v2, 3, v0
        v_mov_b32_e32 v3, 0
    .LBB0_1:
        v_mad_u32_u24 v3, v2, 3, v3
        s_add_i32 s4, s4, 1
        s_cmp_lg_u32 s4, 5
        s_waitcnt vmcnt(2)
        s_cbranch_scc1 .LBB0_1
        v_readlane_b32 s6, v3, 63
        v_writelane_b32 v4, s6, 2
        v_readfirstlane_b32 s7, v1
        s_endpgm
    """)
    assert np.array_equal(e.v[1], np.arange(64))                  # the lane index
    assert np.array_equal(e.v[3], 15 * ((np.arange(64) + 64) >> 3))
    assert e.s["s6"] == 15 * 15 and e.v[4][2] == 225 and e.s["s7"] == 0
    assert sum(op == "s_waitcnt" for op, _ in seen) == 5


def test_loaded_data_is_unknown_and_a_branch_on_it_stops_the_run():
    text = """
        buffer_load_dword v5, v0, s[8:11], 0 offen
        v_readfirstlane_b32 s4, v5
        s_cmp_eq_u32 s4, 0
        s_cbranch_scc1 .LBB0_2
    .LBB0_2:
        s_endpgm
    """
    with pytest.raises(Poison):
        run(text)


def test_an_instruction_it_does_not_know_raises():
    with pytest.raises(RuntimeError):
        run("s_sendmsg sendmsg(MSG_INTERRUPT)\ns_endpgm")


@pytest.mark.parametrize("mask", (0xFFFF, 2**64 - 1))
def test_exec_is_known_again_after_a_branch_on_data(mask):
    lo, hi = mask & 0xFFFFFFFF, mask >> 32
    text = f"""
        s_mov_b32 s4, {lo:#x}
        s_mov_b32 s5, {hi:#x}
        s_mov_b64 exec, s[4:5]
        buffer_load_dword v5, v0, s[8:11], 0 offen
        v_cmp_nlt_f32_e32 vcc, v5, v6
        s_and_saveexec_b64 s[6:7], vcc
        s_xor_b64 s[6:7], exec, s[6:7]
        v_mov_b32_e32 v7, 1
        RESTORE
        s_endpgm
    """
    e, _ = run(text.replace("RESTORE", "s_or_b64 exec, exec, s[6:7]"))
    assert e.get64("exec") == mask
    # a pair that was written in between no longer stands for the lanes that were left out
    e, _ = run(text.replace("RESTORE", "s_and_b64 s[6:7], vcc, s[4:5]\n s_or_b64 exec, exec, s[6:7]"))
    assert e.get64("exec") is None


def test_spilled_registers_are_reported():
    def report(name, spilled):
        return f"a.h:1:1: remark: Function Name: {name} [-R]\na.h:1:1: remark:     VGPRs: 256 [-R]\na.h:1:1: remark:     VGPRs Spill: {spilled} [-R]\n"
    clean = report("_Z19k_lm_head_f32_splitILi4ELi5ELi1E", 0) + report("_Z14k_lm_head_slabILi4ELi8ELi3ELb1ELb0E", 5)
    check_isa.check_spills(clean)
    for bad in (report("_Z19k_lm_head_f32_splitILi4ELi5ELi1E", 1), report("_Z14k_lm_head_slabILi4ELi8ELi3ELb0E", 5)):
        with pytest.raises(RuntimeError):
            check_isa.check_spills(clean + bad)
