"""The neighbour lists' insertion (place_f64 in gesr_device.h) as the compiler emits it.

b = max(below, min(b, c)) writes b before it reads `below`.  In a new list all entries are
equal, and the compiler knows it: `below` must still have registers of its own."""
import re
import shutil
import subprocess

import pytest

from paper_2411_09156_amd import build

KERNEL = """
#include "gesr_device.h"
__global__ void k(const double* c, double* out) {
    double b[2] = {1e300, 1e300};
    gesr::place_f64(b[1], b[0], c[threadIdx.x]);
    out[threadIdx.x] = b[1];
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_equal_entries_keep_their_registers(tmp_path):
    src = tmp_path / "place.hip"
    src.write_text(KERNEL)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
    asm = subprocess.run(["hipcc", *flags, "-I", f"{build.ROOT}/include", "-I", f"{build.HERE}/csrc",
                          "--cuda-device-only", "-S", "-o", "-", str(src)], check=True, capture_output=True,
                         text=True).stdout
    (low,) = re.findall(r"v_min_f64\S* (\S+), (\S+), (\S+)", asm)
    (high,) = re.findall(r"v_max_f64\S* (\S+), (\S+), (\S+)", asm)
    assert low[0].rstrip(",") == high[0].rstrip(",")
    assert high[1].rstrip(",") != high[2].rstrip(","), (low, high)
