"""The forms of the NT GEMM that decode a packed B store the decoded rows into LDS between their
MFMAs without waiting for the direct-to-LDS copies under way (the compiler puts such a wait before
an ordinary LDS store; it stopped the MFMAs four times a step)."""
import os

import pytest

from paper_2609_39223_amd import build, mfma_check


def test_decoded_rows_are_stored_without_waiting_for_the_copies():
    if not (os.path.exists(build.LIB) and os.path.exists(build.OBJDUMP)):
        pytest.skip("nothing built here, or no disassembler")
    stores = {}
    for name, code in mfma_check.kernels(build.LIB, build.OBJDUMP):
        for i, c in enumerate(code):
            near = code[max(0, i - 60):i], code[i + 1:i + 61]
            if c.name != "ds_write_b128" or not all(any(x.mfma for x in n) for n in near):
                continue                         # not between MFMAs
            stores[name] = stores.get(name, 0) + 1
            before = [x.text for x in code[max(0, i - 2):i] if x.name == "s_waitcnt"]
            assert not any("vmcnt(0)" in t for t in before), (name, "%x" % c.address)
    # a stage's eight 16-byte chunks, two steps a loop; dense NVFP4, MXFP4, Q4_K, per expert two
    assert len(stores) == 5 and min(stores.values()) >= 16, stores
