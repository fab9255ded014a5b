"""The E-step kernels for vectors of 16 hide their loads behind four waves per SIMD; index recovery has cost them one before, and the kernels of few vectors
a quarter of their registers in scratch memory. Read from the compiler's resource report."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_13089_amd import build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")


@pytest.mark.parametrize("source,kernels", [("assign_mfma.hip", {"assign_mfma_kernelILi16ELi2ELi4ELi2ELb0E": 0, "assign_mfma_kernelILi16ELi2ELi4ELi2ELb1E": 0}),
                                            ("assign_mfma_f16.hip", {"assign_mfma_f16_kernelILi16ELi4ELi4ELi4ELb1E": 0, "assign_few_f16_kernelILi16ELi1ELb0E": 16,
                                                                     "assign_few_f16_kernelILi16ELi2ELb0E": 16, "assign_few_f16_kernelILi16ELi2ELb1E": 16})])
def test_four_waves_per_simd_at_16(source, kernels):
    """kernels: name -> bytes of scratch memory a lane may use (a few values that are read once)"""
    path = os.path.join(os.path.dirname(build.__file__), "csrc", source)
    report = subprocess.run(["hipcc", *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
                             "-o", os.devnull, path], capture_output=True, text=True, check=True).stderr
    parts = re.split(r"Function Name: ", report)[1:]
    for name, scratch in kernels.items():
        found = [p for p in parts if name in p.split(maxsplit=1)[0]]
        assert len(found) == 1, name
        assert int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", found[0])[1]) >= 4, name
        assert int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", found[0])[1]) <= scratch, name
