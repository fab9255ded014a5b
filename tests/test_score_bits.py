"""Lists of the cells (Section 3.1) take two bits of each score from the conversion of 32 numbers to six bits, an instruction that writes its result before it
has read all of its operands, which the compiler does not know. Read from its assembly: the registers are different ones. (That the operands are stored in the order
in which those bits come is asserted where both are written, when cells.hip is compiled.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_13089_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_result_has_registers_of_its_own():
    path = os.path.join(os.path.dirname(build.__file__), "csrc", "cells.hip")
    text = subprocess.run(["hipcc", *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "--cuda-device-only", "-S", "-o", "-", path],
                          capture_output=True, text=True, check=True).stdout
    found = re.findall(r"v_cvt_scalef32_2xpk16_fp6_f32 v\[(\d+):(\d+)\], v\[(\d+):(\d+)\], v\[(\d+):(\d+)\]", text)
    assert found and len(found) == text.count("v_cvt_scalef32_2xpk16_fp6_f32")
    for registers in found:
        to, a, b = [range(int(lo), int(hi) + 1) for lo, hi in zip(registers[::2], registers[1::2])]
        assert len(to) == 6 and len(a) == len(b) == 16
        assert not set(to) & (set(a) | set(b))


@pytest.mark.parametrize("line,fine", [("v[0:5], v[6:21], v[22:37], 1.0", True), ("v[6:11], v[6:21], v[22:37], 1.0", False), ("v[36:41], v[6:21], v[22:37], 1.0", False),
                                       ("v[0:5], a[6:21], v[22:37], 1.0", False)])
def test_the_build_refuses_shared_registers(line, fine):
    name = "v_cvt_scalef32_2xpk16_fp6_f32"
    if fine:
        build.check_early_results(name, f"\t{name} {line}\n")
    else:
        with pytest.raises(RuntimeError):
            build.check_early_results(name, f"\t{name} {line}\n")
