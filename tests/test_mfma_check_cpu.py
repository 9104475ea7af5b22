"""The build's check of the wait states around the GEMM's inline-assembly MFMAs: listings with a
planted hazard are refused, the same without it are not, and the built library has none."""
import os

import pytest

from paper_2609_39223_amd import build, mfma_check

MFMA = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"


def _hazards(*lines):
    """Lines of assembly at 4-byte steps from 0x100; "@n" in a branch is line n."""
    text = "0000000000000100 <f>:\n"
    for i, l in enumerate(lines):
        tail = ""
        if "@" in l:
            l, n = l.split("@")
            tail = " <f+0x%x>" % (4 * int(n))
        text += "\t%s   // %012X: 00000000%s\n" % (l, 0x100 + 4 * i, tail)
    return mfma_check.hazards(mfma_check.parse(text)["f"])


def test_vector_write_before_an_mfma():
    for r in ("v0", "v7", "a3"):
        w = "v_accvgpr_write_b32 a3, 0" if r == "a3" else "v_mov_b32_e32 %s, v9" % r
        assert _hazards(w, MFMA) and _hazards(w, "s_nop 0", MFMA)
        assert not _hazards(w, "s_nop 1", MFMA)
    assert not _hazards("v_mov_b32_e32 v8, v0", MFMA)
    assert not _hazards("ds_read_b128 v[0:3], v9", MFMA)


@pytest.mark.parametrize("use", ["v_accvgpr_read_b32 v9, a2", "v_accvgpr_write_b32 a0, 0",
                                 "ds_write_b64 v9, a[2:3]",
                                 "v_mfma_f32_16x16x32_bf16 a[4:7], v[0:3], v[4:7], a[0:3]",
                                 "v_mfma_f32_16x16x32_bf16 a[4:7], a[0:3], v[4:7], a[4:7]"])
def test_use_of_a_result(use):
    assert _hazards(MFMA, use) and _hazards(MFMA, "s_nop 15", "s_nop 0", use)
    assert not _hazards(MFMA, "s_nop 15", "s_nop 1", use)
    assert not _hazards(MFMA, MFMA) and not _hazards(MFMA, "s_nop 15", "s_nop 15", use)


def test_along_branches():
    # the write is at the end of the loop, the MFMA at its start
    loop = ["s_nop 1", MFMA, "s_nop 0", "v_mov_b32_e32 v5, v9", "s_cbranch_scc1 65531 @1", "s_endpgm"]
    assert _hazards(*loop)
    assert not _hazards(*(loop[:3] + ["v_mov_b32_e32 v9, v5"] + loop[4:]))
    # one of two ways to the read skips the wait
    skip = [MFMA, "s_cbranch_scc1 2 @4", "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v9, a0", "s_endpgm"]
    assert _hazards(*skip)
    assert not _hazards(*([MFMA, "s_cbranch_scc1 2 @2"] + skip[2:]))


def test_built_library():
    if not (os.path.exists(build.LIB) and os.path.exists(build.OBJDUMP)):
        pytest.skip("nothing built here, or no disassembler")
    assert mfma_check.check_library(build.LIB, build.OBJDUMP) >= 20
