"""Registers of kernels whose workgroup is a quarter or more of a CU's wave slots: one
register block more and a CU holds one workgroup where it held two."""
import re
import shutil
import subprocess

import pytest

from paper_2411_09156_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_two_workgroups_of_1024_threads_fit():
    """A CU has 32 wave slots: 512 registers per lane and SIMD, eight waves of 64."""
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
    out = subprocess.run(["hipcc", *flags, "-I", f"{build.ROOT}/include", "-I", f"{build.HERE}/csrc",
                          "--cuda-device-only", "-S", "-o", "-", f"{build.HERE}/csrc/gesr_render.hip"], check=True,
                         capture_output=True, text=True).stdout
    meta = re.findall(r"\.max_flat_workgroup_size: (\d+)\n(?:.*\n)*?\s+\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)",
                      out)
    big = {name: int(vgprs) for size, name, vgprs in meta if size == "1024"}
    assert len(big) == 3, big  # the 32x32 forward, with and without counts, and adjoint
    assert max(big.values()) <= 64, big
