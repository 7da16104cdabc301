"""Order of memory operations in the built sweep kernels (no GPU)."""
import os
import re
import subprocess

import pytest

from test_native_checks import _gfx950_code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="ROCm LLVM tools not available")
def test_costs_and_state_of_a_tile_are_in_flight_together(tmp_path):
    """The boundary and final sweeps on 12- and 13-bit tiles ask for 16 costs and 16
    amplitudes (eight loads of two) a thread before they wait for any of them."""
    from paper_2401_02852_amd import _binding
    path = _binding.library_path()
    if not os.path.exists(path):
        pytest.skip("libqnae.so not built")
    seen = 0
    for i, co in enumerate(_gfx950_code_objects(path)):
        f = tmp_path / f"co{i}.o"
        f.write_bytes(co)
        asm = subprocess.run([OBJDUMP, "-d", str(f)], capture_output=True, text=True, check=True).stdout
        # sweep_kernel<TB, costs (h or t), KIND, ...>; the batched form has the same body behind a search
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*sweep_kernelILi1[23]E[ht]Li[23]E\S*)>:\n(.*?)(?=\n\n|\Z)",
                                     asm, re.M | re.S):
            ahead = body[:re.search(r"s_waitcnt vmcnt", body).start()]
            assert len(re.findall(r"\bglobal_load_", ahead)) >= 24, name
            seen += 1
    assert seen >= 2 * 2 * 2 * 4  # tiles, cost types, kinds, mirrored or not and layouts
