"""Host-only tests of the build's checks on generated assembly (paper_2603_15619_amd/build.py):
each check is run on small hand-written assembly texts, one that must pass and ones that carry
exactly the mistake the check exists for."""
import pytest

from paper_2603_15619_amd import build as B

GOOD_ACC = """\
_Z6kernelv:
\tv_accvgpr_write_b32 a3, v1
\t;;#ASMSTART
\t; MODA_ACC_REGISTERS_ACQUIRED
\t;;#ASMEND
.LBB0_1:
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 a[64:79], a[32:35], v[0:3], a[64:79]
\t;;#ASMEND
\tv_add_f32_e32 v1, v2, v3
\ts_cbranch_scc1 .LBB0_1
\t;;#ASMSTART
\t; MODA_ACC_REGISTERS_RELEASED
\t;;#ASMEND
\tv_accvgpr_read_b32 v5, a7
\ts_endpgm
.Lfunc_end0:
"""


def check(tmp_path, text):
    f = tmp_path / "k.s"
    f.write_text(text)
    for name, body in B._kernel_bodies(str(f)):
        B._check_kernel(str(f), name, body)


def test_named_register_region_accepts_clean_code(tmp_path):
    check(tmp_path, GOOD_ACC)


def test_compiler_use_inside_owned_region_is_rejected(tmp_path):
    bad = GOOD_ACC.replace("\tv_add_f32_e32 v1, v2, v3\n", "\tv_accvgpr_write_b32 a9, v1\n")
    with pytest.raises(RuntimeError, match="compiler-allocated accumulation register"):
        check(tmp_path, bad)


def test_named_use_after_release_is_rejected(tmp_path):
    bad = GOOD_ACC.replace("\tv_accvgpr_read_b32 v5, a7\n",
                           "\t;;#ASMSTART\n\tv_accvgpr_read_b32 v5, a7\n\t;;#ASMEND\n")
    with pytest.raises(RuntimeError, match="outside the owned region"):
        check(tmp_path, bad)


def test_missing_marker_is_rejected(tmp_path):
    bad = GOOD_ACC.replace("\t; MODA_ACC_REGISTERS_RELEASED\n", "\t; nothing\n")
    with pytest.raises(RuntimeError, match="expected exactly one"):
        check(tmp_path, bad)


# a hand-written matrix instruction, `%s` behind it, then a loop around the code that uses its result
RESULT = """\
_Z6kernelv:
.LBB0_1:
\tv_add_f32_e32 v40, v3, v41
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 v[0:15], a[32:35], a[0:3], 0
\t;;#ASMEND
%s
\ts_cbranch_scc1 .LBB0_1
\tv_mul_f32_e32 v50, v15, v51
\ts_endpgm
.Lfunc_end0:
"""
MORE = "\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 v[0:15], a[36:39], a[4:7], v[0:15]\n\t;;#ASMEND\n"
OTHER = "\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 a[64:79], a[40:43], v[%d:%d], a[64:79]\n\t;;#ASMEND\n"


def check_distance(tmp_path, text):
    f = tmp_path / "r.s"
    f.write_text(RESULT % text)
    for name, body in B._kernel_bodies(str(f)):
        B._check_result_distance(str(f), name, body)


@pytest.mark.parametrize("between", ["\ts_nop 10", "\ts_nop 7\n\ts_nop 2", "\tv_mov_b32_e32 v60, 0\n" * 11, MORE + "\ts_nop 10",
                                     OTHER % (20, 23) + "\ts_nop 2"])
def test_matrix_results_used_late_enough(tmp_path, between):
    check_distance(tmp_path, between)


@pytest.mark.parametrize("between", ["", "\ts_nop 9", "\tv_mov_b32_e32 v60, 0\n" * 10, "\ts_nop 10\n" + MORE, "\tv_mov_b32_e32 v7, 0\n\ts_nop 15",
                                     OTHER % (20, 23) + "\ts_nop 1", "\ts_nop 5\n" + OTHER % (12, 15) + "\ts_nop 15"])
def test_matrix_results_used_too_early_are_rejected(tmp_path, between):
    """By the next instruction, around the loop, by an overwriting move, or as another product's factor."""
    with pytest.raises(RuntimeError, match="issue slots after it instead of 12"):
        check_distance(tmp_path, between)


SCRATCH = """\
_Z9my_kernelv:
\tscratch_store_dword off, v1, off
.LBB0_1:                                ; =>This Inner Loop Header: Depth=1
\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]
%s
\ts_cbranch_scc1 .LBB0_1
; %%bb.2:
\tscratch_load_dword v1, off, off
.LBB0_3:                                ; =>This Inner Loop Header: Depth=1
\tscratch_load_dword v2, off, off
\ts_cbranch_scc1 .LBB0_3
\ts_endpgm
.Lfunc_end0:
"""


def test_scratch_outside_key_loops_is_accepted(tmp_path):
    f = tmp_path / "s.s"
    f.write_text(SCRATCH % "\tv_add_f32_e32 v1, v2, v3")
    B.scan_scratch_in_key_loops(str(f), "my_kernel")


def test_scratch_inside_a_key_loop_is_rejected(tmp_path):
    f = tmp_path / "s.s"
    f.write_text(SCRATCH % "\tscratch_load_dword v3, off, off offset:4")
    with pytest.raises(RuntimeError, match="inside a key loop"):
        B.scan_scratch_in_key_loops(str(f), "my_kernel")
    with pytest.raises(RuntimeError, match="no kernel named"):
        B.scan_scratch_in_key_loops(str(f), "other_kernel")


NESTED = """\
_Z9my_kernelv:
.LBB0_1:                                ; =>This Loop Header: Depth=1
                                        ;     Child Loop BB0_2 Depth 2
                                        ;     Child Loop BB0_4 Depth 2
%s
.LBB0_2:                                ;   Parent Loop BB0_1 Depth=1
                                        ; =>  This Inner Loop Header: Depth=2
\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]
\ts_cbranch_scc1 .LBB0_2
; %%bb.3:                                ;   in Loop: Header=BB0_1 Depth=1
%s
.LBB0_4:                                ;   Parent Loop BB0_1 Depth=1
                                        ; =>  This Inner Loop Header: Depth=2
%s
\ts_cbranch_scc1 .LBB0_4
; %%bb.5:                                ;   in Loop: Header=BB0_1 Depth=1
\ts_cbranch_scc1 .LBB0_1
; %%bb.6:
%s
.LBB0_7:                                ; =>This Inner Loop Header: Depth=1
%s
\ts_cbranch_scc1 .LBB0_7
\ts_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("place", range(5))
def test_scratch_around_a_nested_key_loop(tmp_path, place):
    """In the outer loop before (0) or behind (1) the loop of matrix instructions, or in another loop
    inside it (2), scratch is rejected; behind the loops (3) or in a later loop (4) it is not."""
    lines = ["\tv_add_f32_e32 v1, v2, v3"] * 5
    f = tmp_path / "n.s"
    f.write_text(NESTED % tuple(lines))
    B.scan_scratch_in_key_loops(str(f))
    lines[place] = "\tscratch_load_dword v3, off, off offset:4"
    f.write_text(NESTED % tuple(lines))
    if place < 3:
        with pytest.raises(RuntimeError, match="inside a key loop"):
            B.scan_scratch_in_key_loops(str(f), "my_kernel")
    else:
        B.scan_scratch_in_key_loops(str(f), "my_kernel")


def test_scratch_in_a_loop_of_a_kernel_without_matrix_instructions_is_rejected(tmp_path):
    text = (NESTED % tuple(["\tv_add_f32_e32 v1, v2, v3"] * 4 + ["\tscratch_load_dword v3, off, off"]))
    f = tmp_path / "v.s"
    f.write_text("\n".join(x for x in text.split("\n") if "v_mfma" not in x))
    with pytest.raises(RuntimeError, match="inside a key loop"):
        B.scan_scratch_in_key_loops(str(f))


def test_every_source_is_checked(monkeypatch, tmp_path):
    """The build hands every kernel source to the check, and a refusal ends the build."""
    seen = []

    def refuse_last(src):
        seen.append(src)
        if len(seen) == len(B.sources()):
            raise RuntimeError("refused")

    monkeypatch.setattr(B, "OBJ", str(tmp_path))
    monkeypatch.setattr(B, "check_named_acc_registers", lambda src: None)
    monkeypatch.setattr(B, "check_no_scratch_in_loops", refuse_last)
    monkeypatch.setattr(B, "_compile", lambda src: src)
    with pytest.raises(RuntimeError, match="refused"):
        B.build_libmoda()
    assert sorted(seen) == B.sources()
