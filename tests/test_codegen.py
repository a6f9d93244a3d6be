"""What the compiler made of the kernels: no registers addressed by index, anywhere in the library."""
import os
import shutil
import subprocess

import pytest

import paper_2509_22418_amd as pp

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_kernel_addresses_its_registers_by_index(tmp_path):
    """A loop over accumulators that is not unrolled in full becomes s_set_gpr_idx around every access (the fp32-multiply attention backward at head dim 128: 8448 of
    them, 1.1 to 1.2 times the time)."""
    pp.load_library()          # builds it if it has never been built
    lib = shutil.copy(pp.lib_path(), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    text = "".join(subprocess.run([OBJDUMP, "-d", str(o)], check=True, capture_output=True, text=True).stdout for o in sorted(tmp_path.glob("*gfx950*")))
    assert "v_mfma" in text and "s_endpgm" in text
    assert text.count("s_set_gpr_idx") == 0
