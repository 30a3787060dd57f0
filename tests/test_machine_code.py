"""The built library's machine code keeps the rules that the compiler does not see to in inline assembly
(paper_2503_01586_amd/check_machine_code.py), and the scan finds what breaks them."""
import pytest

from paper_2503_01586_amd import check_machine_code as mc


def code(*lines):
    """Instructions 4 bytes apart; a branch is written with the number of the line it goes to."""
    out = []
    for i, line in enumerate(lines):
        op, _, text = line.partition(" ")
        word = 0
        if op.startswith(("s_branch", "s_cbranch")):
            word = (int(text) - i - 1) & 0xffff
        out.append(mc.Instruction(op, text, 4 * i, "%08X" % word))
    return out


def findings(scan, *lines, kernel="k"):
    return [f.address // 4 for f in scan.run(kernel, *mc.blocks_of(code(*lines)))]


def test_scalar_registers_that_a_vector_instruction_wrote():
    scan = mc.VectorWrittenScalars()
    write, load, other = "v_readfirstlane_b32 s3, v1", "global_load_lds_dwordx4 v5, s[2:3]", "v_mov_b32_e32 v9, v8"
    assert findings(scan, write, load, "s_endpgm ") == [1]
    assert findings(scan, write, "s_nop 3", load, "s_endpgm ") == [2]
    assert findings(scan, write, "s_nop 4", load, "s_endpgm ") == []
    assert findings(scan, write, "s_nop 3", other, load, "s_endpgm ") == []
    assert findings(scan, write, "s_cmp_eq_u32 s3, 0", load, "s_endpgm ") == [2]        # read, not written anew
    assert findings(scan, write, "s_mov_b32 s3, s9", load, "s_endpgm ") == []
    assert findings(scan, write, "s_nop 4", "global_load_dword v1, v2, s[4:5]", load, "s_endpgm ") == []
    assert findings(scan, "v_cmp_lt_u32_e64 s[2:3], v1, v2", load, "s_endpgm ") == [1]
    assert findings(scan, "v_add_co_u32_e32 v1, vcc, v1, v2", "buffer_load_dword v1, v2, s[4:7], vcc_lo offen", "s_endpgm ") == [1]
    # the shorter of two ways to the load, and the way around a loop
    assert findings(scan, write, "s_cbranch_scc1 3", "s_nop 4", load, "s_endpgm ") == [3]
    assert findings(scan, "s_nop 0", load, other, write, "s_cbranch_scc1 1", "s_endpgm ") == [1]


def test_direct_loads_behind_a_write_of_m0():
    scan = mc.LdsLoadsBehindM0()
    write, load = "s_mov_b32 m0, s29", "global_load_lds_dwordx4 v1, s[50:51]"
    assert findings(scan, write, load, "s_endpgm ") == [1]
    assert findings(scan, write, "buffer_load_dword v1, s[4:7], 0 offen lds", "s_endpgm ") == [1]
    assert findings(scan, write, "s_nop 0", load, "s_endpgm ") == []
    assert findings(scan, write, "s_mov_b32 s4, s29", load, "s_endpgm ") == []
    assert findings(scan, write, "global_load_dword v1, v2, s[4:5]", load, load, "s_endpgm ") == []


def test_registers_of_the_query_in_flight():
    q, q2 = "global_load_dwordx4 v[8:11], v[2:3], off", "global_load_dwordx4 v[12:15], v[4:5], off"
    tile, product = "global_load_lds_dwordx4 v1, s[2:3]", "v_mfma_f32_16x16x32_bf16 v[20:23], v[16:19], v[8:11], 0"
    found = lambda *lines: findings(mc.QueryInFlight(), *lines, kernel="attn_mfma_kernel")
    assert found(q, q2, "s_waitcnt vmcnt(0)", product, "s_endpgm ") == []
    assert found(q, q2, tile, "s_waitcnt vmcnt(1)", product, "v_mov_b32_e32 v8, v9", "s_endpgm ") == []
    # a copy, arithmetic, or another use of the register, ahead of the wait
    assert found(q, q2, "v_accvgpr_write_b32 a1, v15", "s_waitcnt vmcnt(0)", product, "s_endpgm ") == [2]
    assert found(q, q2, "v_pk_mul_f16 v30, v31, v9", "s_waitcnt vmcnt(0)", product, "s_endpgm ") == [2]
    assert found(q, q2, "v_mov_b32_e32 v12, 0", "s_waitcnt vmcnt(0)", product, "s_endpgm ") == [2]
    # a wait that leaves them under way, the address of a later load, the way out of an empty split
    assert found(q, q2, tile, "s_waitcnt vmcnt(2)", "v_mov_b32_e32 v12, 0", product, "s_endpgm ") == [4]
    assert found(q, "global_load_dwordx4 v[12:15], v[8:9], off", "s_waitcnt vmcnt(0)", product, "s_endpgm ") == [1]
    assert found(q, q2, "s_cbranch_scc1 6", "s_waitcnt vmcnt(0)", product, "s_endpgm ", "v_mov_b32_e32 v8, 0",
                 "s_waitcnt vmcnt(0)", "s_endpgm ") == [6]
    # loaded in one of two places: what stands ahead of the second is not on the first one's way
    assert found("s_cbranch_scc1 3", q, q2, "s_cbranch_scc0 6", "v_mov_b32_e32 v8, 0", q, "s_waitcnt vmcnt(0)", product, "s_endpgm ") == []


@pytest.fixture(scope="module")
def library():
    return mc.check()


def test_library_is_scanned(library):
    kernels, _ = library
    assert kernels >= 300


@pytest.mark.parametrize("rule", [s.rule for s in mc.SCANS])
def test_no_findings(library, rule):
    found = [f for f in library[1] if f.rule == rule]
    assert not found, "%d findings, the first: %s" % (len(found), found[0])
