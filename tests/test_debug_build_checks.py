"""Every kind of access of the transform passes is bounds-checked in the debug build, on the CPU.

A check that is missing shows nowhere: a valid run counts no violation with or without it, and a buffer
access that leaves its rows is dropped by the hardware.  So the accesses are compiled one by one
(debug_checks_probe.hip) with -DRECON_DEBUG, and each kernel's listing must name the violation counter."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def kernels(listing):
    """Kernel name: text of its listing."""
    out = {}
    for m in re.finditer(r"^(\w*(?:probe_|k_plane_)\w*):.*?^\.Lfunc_end", listing, re.M | re.S):
        out[m.group(1)] = m.group(0)
    return out


@pytest.mark.timeout(300)
def test_each_access_counts_what_lies_outside(tmp_path):
    if not (shutil.which(HIPCC) or os.path.exists(HIPCC)):
        pytest.skip("ROCm compiler not found")
    asm = tmp_path / "probe.s"
    base = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "--offload-device-only", "-S",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I" + os.path.join(ROOT, "paper_1504_02591_amd", "csrc"),
            os.path.join(ROOT, "tests", "debug_checks_probe.hip"), "-o", str(asm)]
    subprocess.run(base + ["-DRECON_DEBUG"], check=True, capture_output=True, timeout=280)
    found = kernels(asm.read_text())
    assert len(found) == 14, sorted(found)
    missing = sorted(k for k, text in found.items() if "recon_debug_count" not in text)
    assert not missing
