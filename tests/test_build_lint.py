"""The wait-state lint of the build (paper_2411_01288_amd/build.py: lint_asm_hazards) on small listings."""
import pytest

from paper_2411_01288_amd import build
from paper_2411_01288_amd.build import lint_asm_hazards

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


def test_both_builds_make_all_that_the_binding_loads(monkeypatch):
    for name, library in (("build_library", build.LIB), ("build_sanitized_library", build.SAN_LIB)):
        made = set()
        monkeypatch.setattr(build.subprocess, "check_call", lambda cmd, **kw: made.add(cmd[cmd.index("-o") + 1]))
        monkeypatch.setattr(build, "_compile", lambda src: src)
        monkeypatch.setattr(build, "lint_staging_hazards", lambda *a: None)
        getattr(build, name)()
        assert {library, build.MARSHAL} <= made
