"""The wait-state lints of the build (paper_2411_01288_amd/build.py: lint_asm_hazards, lint_asm_mfma) on small listings."""
import pytest

from paper_2411_01288_amd import build
from paper_2411_01288_amd.build import lint_asm_hazards, lint_asm_mfma

STORE = "\tbuffer_store_dwordx4 v[4:7], v2, s[0:3], s16 offen\n"


@pytest.mark.parametrize("text,hits", [
    (STORE + "\tv_accvgpr_read_b32 v4, a20\n", 1),                       # data register overwritten at once
    (STORE + "\tv_mov_b32_e32 v9, v1\n\tv_accvgpr_read_b32 v7, a20\n", 1),  # one wait state behind the store
    (STORE + "\ts_nop 1\n\tv_accvgpr_read_b32 v4, a20\n", 0),
    (STORE + "\tv_mov_b32_e32 v9, v1\n\ts_add_i32 s1, s2, s3\n\tv_accvgpr_read_b32 v4, a20\n", 0),
    (STORE + "\tv_mov_b32_e32 v2, v4\n", 0),                             # the address, and a read of the data
    ("\tbuffer_store_dwordx2 v[4:5], v2, s[0:3], s16 offen\n\tv_mov_b32_e32 v4, 0\n", 0),
    ("\tglobal_store_dwordx4 v2, v[4:7], s[0:1]\n\tv_mov_b32_e32 v5, 0\n", 1),
    ("\tv_readfirstlane_b32 s16, v1\n\ts_nop 3\n" + STORE, 1),           # scalar offset read too early
    ("\tv_readfirstlane_b32 s16, v1\n\ts_nop 4\n" + STORE, 0),
    ("\tv_readfirstlane_b32 s9, v1\n\tbuffer_load_dwordx4 v1, s[4:7], s9 offen lds\n", 1),
])
def test_lint_finds_the_hazards_the_compiler_leaves(text, hits):
    assert len(lint_asm_hazards(text)) == hits


def mfma(d, c):
    return f"\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 v[{d}:{d + 3}], v[20:23], v[24:27], {c}\n\t;;#ASMEND\n"


SUM, FRESH, OTHER = mfma(4, "v[4:7]"), mfma(4, "0"), "\tv_mov_b32_e32 v30, v1\n"


@pytest.mark.parametrize("text,hits", [
    (FRESH + "\tv_add_f32_e32 v1, v1, v4\n", 1),                                      # result read at once
    (FRESH + "\ts_nop 10\n\tv_add_f32_e32 v1, v1, v7\n", 1),                          # after eleven wait states
    (FRESH + "\ts_nop 11\n\tv_add_f32_e32 v1, v1, v7\n", 0),
    (FRESH + OTHER * 11 + "\tds_write_b32 v1, v4\n", 1),
    (FRESH + OTHER * 12 + "\tv_mov_b32_e32 v4, 0\n", 0),
    (FRESH + "\ts_nop 5\n\tv_mov_b32_e32 v5, 0\n", 1),                                # overwritten
    (SUM + "\ts_nop 1\n" + SUM, 0),                                                   # added to again
    (SUM + SUM, 1),
    (SUM + "\ts_nop 5\n\tv_mfma_f32_16x16x32_bf16 v[8:11], v[4:7], v[24:27], 0\n", 1),   # an operand of the compiler's own
    ("\tv_mov_b32_e32 v24, v1\n" + FRESH, 1),                                         # operand written just before
    ("\tv_mov_b32_e32 v24, v1\n\ts_nop 0\n" + FRESH, 1),
    ("\tv_mov_b32_e32 v24, v1\n\ts_nop 1\n" + FRESH, 0),
    ("\tv_mov_b32_e32 v5, v1\n\ts_nop 0\n" + SUM, 1),
    (".LBB0_1:\n\tv_add_f32_e32 v1, v1, v4\n\ts_nop 7\n\ts_nop 7\n" + FRESH + "\ts_cbranch_scc1 .LBB0_1\n", 1),   # around a loop
    ("\ts_branch .LBB0_2\n\tv_mov_b32_e32 v24, v1\n.LBB0_2:\n" + FRESH + "\ts_branch .LBB0_3\n\tv_mov_b32_e32 v4, v1\n.LBB0_3:\n\ts_nop 11\n", 1),
    ("\tv_mfma_f32_16x16x32_bf16 v[4:7], v[20:23], v[24:27], 0\n\tv_mov_b32_e32 v4, 0\n", 0),   # the compiler's own are its to pad
])
def test_lint_finds_hazards_of_matrix_instructions_in_assembly(text, hits):
    assert len(lint_asm_mfma(text)) == hits


def test_kernels_with_registers_in_assembly_are_checked(monkeypatch):
    """A spill and a hazard in either source of the contraction kernels refuse the build."""
    assert set(build.NO_SCRATCH) == {"gemm_bf16.hip", "f32_path.hip"}
    for src, kernel in build.NO_SCRATCH.items():
        text = f"remark: Function Name: _Z{kernel}ILi4E\nremark:     ScratchSize [bytes/lane]: 68\n"
        monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: build.subprocess.CompletedProcess(cmd, 0, FRESH + "\tv_mov_b32_e32 v4, 0\n", text))
        with pytest.raises(RuntimeError, match="spill"):
            build._compile(src)
        with pytest.raises(RuntimeError, match="hazards"):
            build.lint_staging_hazards(src)


def test_both_builds_make_all_that_the_binding_loads(monkeypatch):
    for name, library in (("build_library", build.LIB), ("build_sanitized_library", build.SAN_LIB)):
        made = set()
        monkeypatch.setattr(build.subprocess, "check_call", lambda cmd, **kw: made.add(cmd[cmd.index("-o") + 1]))
        monkeypatch.setattr(build, "_compile", lambda src: src)
        monkeypatch.setattr(build, "lint_staging_hazards", lambda *a: None)
        getattr(build, name)()
        assert {library, build.MARSHAL} <= made
