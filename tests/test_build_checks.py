"""What the build refuses in the kernels' listings, and what it does without a C compiler (host only)."""
import importlib.machinery
import os

import pytest

from paper_2603_29010_amd import build
from paper_2603_29010_amd.build import early_use_of_transpose_reads, overwritten_store

READ_A = ["ds_read_b64_tr_b16 v[10:11], v2", "ds_read_b64_tr_b16 v[12:13], v2 offset:1024"]
READ_B = ["ds_read_b128 v[20:23], v3", "ds_read_b128 v[24:27], v3 offset:2048"]
MUL = ["v_mfma_f32_16x16x32_bf16 v[0:3], v[20:23], v[10:13], v[0:3]"]


def scan(*parts):
    return early_use_of_transpose_reads(["_ZN3ucl6kernelE:"] + [line for part in parts for line in part])


def test_a_wait_has_to_cover_the_transpose_read():
    assert scan(READ_A, MUL) == (4, MUL[0])
    assert scan(READ_A, READ_B, ["s_waitcnt lgkmcnt(2)"], MUL) is None
    # the same wait with the ordinary loads moved ahead of the transpose reads, or behind the wait: it covers nothing
    assert scan(READ_B, READ_A, ["s_waitcnt lgkmcnt(2)"], MUL) is not None
    assert scan(READ_A, ["s_waitcnt lgkmcnt(2)"], READ_B, MUL) is not None
    assert scan(READ_B, READ_A, ["s_waitcnt lgkmcnt(0)"], MUL) is None
    assert scan(READ_A, READ_B, ["s_waitcnt vmcnt(0)"], MUL) is not None
    assert scan(READ_A, READ_B, ["s_waitcnt vmcnt(0) lgkmcnt(0)"], MUL) is None
    assert scan(READ_A, ["v_add_u32_e32 v12, 1, v4"], ["s_waitcnt lgkmcnt(0)"]) is not None        # overwritten in flight


def test_the_data_of_a_wide_store_stay_for_two_wait_states():
    store, write = "buffer_store_dwordx4 v[172:175], v215, s[28:31], s59 offen", "v_mov_b32_e32 v172, v192"
    assert overwritten_store([store, write]) == (2, write)
    assert overwritten_store(["global_store_dwordx4 v[2:3], v[4:7], off", "v_add_u32_e32 v6, 1, v9"]) == (2, "v_add_u32_e32 v6, 1, v9")
    for between in ("s_nop 0", "v_mov_b32_e32 v215, v192", "v_mov_b32_e32 v171, v192", "s_waitcnt vmcnt(0)"):
        assert overwritten_store([store, between, write]) == (3, write)
        assert overwritten_store([store, between, between, write]) is None
    assert overwritten_store([store, "s_nop 1", write]) is None
    assert overwritten_store([store, "s_nop 0", "v_swap_b32 v1, v174"]) is not None
    assert overwritten_store([store.replace("x4 v[172:175]", "x2 v[172:173]"), write]) is None


def test_the_data_of_a_wide_store_across_branches():
    store, write = "buffer_store_dwordx4 v[172:175], v215, s[28:31], 0 offen", "v_mov_b32_e32 v172, v192"
    # a loop's head, behind its back edge; the fall-through of a conditional branch; either side of one
    assert overwritten_store([".LBB0_1:", write, "s_nop 3", store, "s_cbranch_scc1 .LBB0_1", "s_endpgm"]) == (2, write)
    assert overwritten_store([store, "s_cbranch_scc1 .LBB0_2", write, ".LBB0_2:", "s_endpgm"]) == (3, write)
    assert overwritten_store([".LBB0_1:", write, "s_nop 3", store, "s_nop 0", "s_cbranch_scc1 .LBB0_1", "s_endpgm"]) is None
    # what stands behind an unconditional branch is not what runs
    assert overwritten_store([store, "s_branch .LBB0_2", ".LBB0_1:", write, ".LBB0_2:", "s_endpgm"]) is None
    assert overwritten_store([store, "s_endpgm", "_Z4nextv:", write]) is None


def test_the_extension_module_is_named_for_its_interpreter():
    suffix = os.path.basename(build.CALLS)[len("_calls"):]
    assert suffix == importlib.machinery.EXTENSION_SUFFIXES[0] and suffix != ".so"


@pytest.mark.parametrize("cc", ["/nonexistent/cc", "false"])
def test_without_a_compiler_the_build_goes_on(tmp_path, monkeypatch, cc):
    module, untagged = tmp_path / "_calls.tag.so", tmp_path / "_calls.so"
    module.write_bytes(b"of an earlier source")
    untagged.write_bytes(b"of an earlier build")
    monkeypatch.setattr(build, "CALLS", str(module))
    monkeypatch.setattr(build, "CC", cc)
    with pytest.warns(UserWarning, match="ctypes"):
        build._build_calls(True)
    assert not module.exists() and not untagged.exists()
