"""Requests that load straight into LDS (global_load_lds) are counted by vmcnt, and a barrier does not wait for them: a wave has to, before other waves
may read what it requested. The source says so itself, whatever the present compiler adds."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_13089_amd", "csrc")
SOURCES = [p for p in sorted(glob.glob(os.path.join(CSRC, "*"))) if "global_load_lds(" in open(p).read()]


def test_there_are_such_requests():
    assert SOURCES


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_every_request_is_waited_for_before_a_barrier(path):
    text = re.sub(r"//[^\n]*", "", open(path).read())
    for request in re.finditer(r"global_load_lds\(", text):
        after = re.search(r"vmcnt\(0\)|__syncthreads\(\)|s_barrier|__global__", text[request.end():])
        assert after is not None and after.group() == "vmcnt(0)", f"{os.path.basename(path)}: a request goes through {after and after.group()} unwaited"
