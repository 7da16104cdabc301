"""Host code of the library's calls over a stand-in HIP runtime, under AddressSanitizer and UBSan (no GPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_02852_amd", "csrc")


@pytest.mark.skipif(not os.path.isdir("/opt/rocm/include/hip"), reason="HIP headers not available")
def test_host_paths(tmp_path):
    exe = str(tmp_path / "host_paths_check")
    srcs = [os.path.join(CSRC, f + ".cpp") for f in ("runtime", "qnae", "batch", "grad", "prologue", "sample")]
    srcs += [os.path.join(CSRC, "tune.cpp"), os.path.join(ROOT, "tests", "native", "host_paths_check.cpp")]
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-o", exe, *srcs],
                   check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "host paths ok" in r.stdout, r.stdout + r.stderr
