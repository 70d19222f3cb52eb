"""The assembly of the bit-packed sweeps: the additions that take a mask from
scalar registers as carry-in are inline assembly, before which the compiler
keeps no wait states.  Each block of them opens with its own two, so that a
vector instruction that writes those registers (a spilled mask read back) may
stand right before it."""
import os
import re
import subprocess

import pytest

from paper_2606_25203_amd import build


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "bits.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--offload-device-only", os.path.join(build.CSRC, "bits.hip"),
                    "-o", out], check=True, capture_output=True)
    text = open(out).read()
    return text, re.findall(r";APP\n(.*?);NO_APP", text, flags=re.S) or re.findall(r";;#ASMSTART\n(.*?);;#ASMEND", text, flags=re.S)


def test_blocks_open_with_wait_states(blocks):
    text, found = blocks
    adds = [[x.split() for x in b.strip().splitlines() if x.strip()] for b in found if "v_addc_co_u32" in b]
    assert sum(len(b) - 1 for b in adds) == text.count("v_addc_co_u32"), "an addition outside the blocks"
    assert len(adds) > 100
    for b in adds:
        assert b[0][0] == "s_nop" and int(b[0][1]) >= 1, b
        assert all(i[0] == "v_addc_co_u32_e64" for i in b[1:])
