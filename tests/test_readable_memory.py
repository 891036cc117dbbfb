"""The rule that decides whether a kernel reads a caller's P where it lies or
a copy of it (csrc/sap_mem.h), on the CPU: a small program over every kind of
memory and both sides of the device comparison.  What the rule refuses goes
through a copy, which works for another device's memory and is an error for
pageable host memory."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
ROCM = Path("/opt/rocm/include")

PROGRAM = r"""
#include <cstdio>
#include "sap_mem.h"
static int x;
static bool reads(hipMemoryType type, int of, int device, void *dev = &x, void *host = &x) {
    hipPointerAttribute_t at{};
    at.type = type;
    at.device = of;
    at.devicePointer = dev;
    at.hostPointer = host;
    return sap::kernel_can_read(at, device);
}
int main() {
    printf("device_same %d\n", reads(hipMemoryTypeDevice, 1, 1));
    printf("device_other %d\n", reads(hipMemoryTypeDevice, 1, 0) || reads(hipMemoryTypeDevice, 0, 1));
    printf("managed %d\n", reads(hipMemoryTypeManaged, 0, 0) && reads(hipMemoryTypeManaged, 1, 0));
    printf("pinned %d\n", reads(hipMemoryTypeHost, 0, 0) && reads(hipMemoryTypeHost, 1, 0));
    printf("pinned_elsewhere %d\n", reads(hipMemoryTypeHost, 0, 0, &x + 1, &x));
    printf("pinned_unmapped %d\n", reads(hipMemoryTypeHost, 0, 0, nullptr, nullptr));
    printf("pageable %d\n", reads(hipMemoryTypeUnregistered, 0, 0, nullptr, &x));
    printf("array %d\n", reads(hipMemoryTypeArray, 0, 0));
}
"""


@pytest.mark.skipif(not shutil.which("g++") or not ROCM.exists(), reason="needs g++ and the HIP headers")
def test_which_memory_a_kernel_reads(tmp_path):
    src, exe = tmp_path / "reads.cpp", tmp_path / "reads"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}",
                    f"-I{ROOT / 'paper_1807_03425_amd' / 'csrc'}", "-o", str(exe), str(src)], check=True)
    got = dict(l.split() for l in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines())
    assert got == dict(device_same="1", device_other="0", managed="1", pinned="1", pinned_elsewhere="0",
                       pinned_unmapped="0", pageable="0", array="0")
