"""Host and device decisions on sizes that no test can allocate, in a CPU program."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
def test_table_sizes_past_32_bits(tmp_path):
    exe = str(tmp_path / "limits_check")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xarch_host", "-fsanitize=undefined",
                    "-o", exe, os.path.join(ROOT, "tests", "native", "limits_check.cpp")], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "limits ok" in r.stdout, r.stdout + r.stderr


def test_kernels_take_no_32_bit_table_product():
    """The one-workgroup kernels decide with rows_fit where the tables are."""
    for name, room in (("resident.hip", "kTabMax"), ("resident_grad.hip", "kGradTab")):
        text = open(os.path.join(ROOT, "paper_2401_02852_amd", "csrc", name)).read()
        assert f"a.lut_len, {room})" in text and f"* a.lut_len <= {room}" not in text
