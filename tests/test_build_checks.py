"""The build's scans of the generated assembly, on small pieces of code with and without the mistake they look for."""
import pytest

from paper_2509_16518_amd import build


def scan(tmp_path, lines, check=build.check_untracked_loads):
    path = tmp_path / "piece.s"
    path.write_text("piece:\n" + "".join("\t%s\n" % x if not x.endswith(":") else x + "\n" for x in lines) + ".Lfunc_end0:\n")
    return check(str(path))


LOAD = "global_load_dword v5, v1, s[2:3] ; fg_id"
GATHER = "global_load_lds_dwordx4 v7, s[4:5]"
USE = "v_add_u32_e32 v6, v5, v5"
END = "s_endpgm"

LOOP = [LOAD, ".LBB0_1:", GATHER, GATHER, "s_waitcnt vmcnt(2)", USE, LOAD.replace("v1", "v2"), "v_mov_b32_e32 v9, v8",
        "s_cbranch_scc1 .LBB0_1", "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v5, 0", END]

CLEAN = {
    "waited for": [LOAD, "s_waitcnt vmcnt(0)", USE, END],
    "covered by a count": [LOAD, GATHER, GATHER, "s_waitcnt vmcnt(2)", USE, END],
    "waited for with other counters": [LOAD, "s_waitcnt vmcnt(0) lgkmcnt(0)", USE, END],
    "other registers": [LOAD, "v_mov_b32_e32 v6, v4", "ds_read_b128 v[8:11], v0", "s_waitcnt vmcnt(0)", USE, END],
    "around a loop": LOOP,
    "both paths": [LOAD, "s_cbranch_vccz .LBB0_2", "s_waitcnt vmcnt(0)", "s_branch .LBB0_3", ".LBB0_2:", "s_waitcnt vmcnt(0)",
                   ".LBB0_3:", USE, END],
    "a condition that is constant": [LOAD, "s_mov_b64 s[8:9], -1", "s_and_b64 vcc, exec, s[8:9]", "s_cbranch_vccnz .LBB0_3", USE,
                                     ".LBB0_3:", "s_waitcnt vmcnt(0)", END],
    "the way out, not the way round": [".LBB0_1:", "s_waitcnt vmcnt(0)", USE, "s_mov_b64 s[8:9], -1", LOAD, "s_cbranch_scc1 .LBB0_2",
                                       "s_waitcnt vmcnt(0)", "s_cselect_b64 s[8:9], -1, 0", ".LBB0_2:", "s_and_b64 vcc, exec, s[8:9]",
                                       "s_cbranch_vccnz .LBB0_3", "v_mov_b32_e32 v9, v5", "s_branch .LBB0_1", ".LBB0_3:",
                                       "s_waitcnt vmcnt(0)", END],
}


@pytest.mark.parametrize("name", sorted(CLEAN))
def test_untracked_loads_that_are_waited_for(tmp_path, name):
    assert scan(tmp_path, CLEAN[name]) == sum("fg_id" in x for x in CLEAN[name])


FAULTY = {
    "read at once": [LOAD, USE, END],
    "reused before it lands": [LOAD, "v_mov_b32_e32 v5, v0", "s_waitcnt vmcnt(0)", END],
    "reused as part of a wider register": [LOAD, "ds_read_b128 v[2:5], v0", "s_waitcnt vmcnt(0)", END],
    "spilled": [LOAD, "scratch_store_dword off, v5, off", "s_waitcnt vmcnt(0)", END],
    "used as an address": [LOAD, "global_load_lds_dwordx4 v5, s[4:5]", "s_waitcnt vmcnt(0)", END],
    "count too large": [LOAD, GATHER, "s_waitcnt vmcnt(2)", USE, END],
    "only another counter": [LOAD, "s_waitcnt lgkmcnt(0)", USE, END],
    "one path only": [LOAD, "s_cbranch_vccz .LBB0_2", "s_waitcnt vmcnt(0)", ".LBB0_2:", USE, END],
    "fewer operations on one path": [LOAD, "s_cbranch_scc0 .LBB0_2", GATHER, ".LBB0_2:", "s_waitcnt vmcnt(1)", USE, END],
    "around a loop": [x.replace("v_mov_b32_e32 v9, v8", "v_mov_b32_e32 v9, v5") for x in LOOP],
    "an unknown condition": [x.replace("s_mov_b64 s[8:9], -1", "s_mov_b64 s[8:9], s[10:11]")
                             for x in CLEAN["the way out, not the way round"]],
    "a condition that changed": [LOAD, "s_mov_b64 s[8:9], -1", "s_mov_b32 s8, 0", "s_and_b64 vcc, exec, s[8:9]",
                                 "s_cbranch_vccnz .LBB0_3", USE, ".LBB0_3:", "s_waitcnt vmcnt(0)", END],
}


@pytest.mark.parametrize("name", sorted(FAULTY))
def test_untracked_loads_that_are_not(tmp_path, name):
    with pytest.raises(RuntimeError):
        scan(tmp_path, FAULTY[name])


def test_spills_of_forward_kernels(tmp_path):
    def listing(kernel, spills):
        return ["    .name:           %s" % kernel, "    .vgpr_spill_count: %d" % spills]
    scan(tmp_path, listing("_ZN2fg17fgattn_fwd_kernelILi64E", 1), build.check_spills)
    scan(tmp_path, listing("_ZN3fgm13select_kernel", 9), build.check_spills)
    with pytest.raises(RuntimeError):
        scan(tmp_path, listing("_ZN2fg17fgattn_fwd_kernelILi64E", 2), build.check_spills)


MODE = "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3"
WEIGHT = [";#ASMSTART", "v_cvt_f64_f32 v[4:5], v1", "v_mul_f64 v[4:5], v[4:5], s[2:3]", ";#ASMEND"]
PLAIN = "v_mul_f64 v[4:5], v[4:5], s[2:3]"


def test_rounding_mode_that_holds(tmp_path):
    assert scan(tmp_path, [MODE] + WEIGHT + ["v_add_u32_e32 v1, v2, v3"] + WEIGHT + [END], build.check_rounding_mode) == 1
    assert scan(tmp_path, [PLAIN, "v_cvt_f64_f32_e32 v[4:5], v1", END], build.check_rounding_mode) == 0
    assert scan(tmp_path, [MODE] + WEIGHT + [END, ".Lfunc_end7:", PLAIN, END], build.check_rounding_mode) == 1


@pytest.mark.parametrize("lines", [[MODE, PLAIN, END], [MODE] + WEIGHT + ["v_cvt_f64_u32_e32 v[4:5], v1", END], [MODE] + WEIGHT + [MODE, END],
                                   [MODE] + WEIGHT + ["s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 0", END], WEIGHT + [END],
                                   ["s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3"] + WEIGHT + [END], [PLAIN, MODE] + WEIGHT + [END]])
def test_rounding_mode_that_does_not(tmp_path, lines):
    with pytest.raises(RuntimeError):
        scan(tmp_path, lines, build.check_rounding_mode)
