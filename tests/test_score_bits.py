"""Lists of the cells (Section 3.1) take two bits of each score from the conversion of 32 numbers to six bits, an instruction that writes its result before it
has read all of its operands, which the compiler does not know. Read from its assembly: the registers are different ones. And the order in which
those bits come, which the operands are stored by, is the one that the source states."""
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


def test_bits_stand_where_the_operands_say():
    """Number i of the first and of the second operand are the six bits from 12 i and 12 i + 6 on; paired_row of cells.hip turned round."""
    masks = (0x30c30c30, 0x0c30c30c, 0xc30c30c3)
    place = {}   # (word, pair of bits from the top) -> (tile, result)
    for tile in (0, 1):
        for i in range(16):
            bit = 12 * i + 6 * tile + 4   # upper exponent bit, then the sign
            word, at = divmod(bit, 96)
            assert at % 2 == 0 and masks[at // 32] >> (at % 32) & 3 == 3
            place[word, 15 - at % 32 // 2] = (tile, i)
    assert len(place) == 32
    for at in range(64):
        word, z = at >> 5 & 1, at & 15
        p = 15 - z
        turn = {2: p // 3, 1: 5 + p // 3, 0: 10 + p // 3}[p % 3]
        assert place[word, z] == (turn & 1, 8 * word + turn // 2)
