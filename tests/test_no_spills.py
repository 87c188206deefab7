"""No kernel of the library keeps vector registers in scratch memory: the
spill counts that the compiler recorded in the built objects' kernel metadata.
(A spill costs the loop that it is in, and one was seen stored under the
wrong lane mask after a divergent loop, with wrong results.)"""
import os
import re
import subprocess

import pytest

from paper_2308_10169_amd import build as B

LLVM = os.path.join(B.ROCM, "llvm", "bin")


@pytest.mark.parametrize("name", ["kernels", "bf", "mlp", "fitness", "philox"])
def test_no_vector_register_spills(name, tmp_path):
    obj = os.path.join(B.BUILD, name + ".o")
    if not os.path.exists(obj):
        pytest.skip("library not built here")
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", obj,
                    str(tmp_path / "copy.o")], check=True)
    subprocess.run([os.path.join(LLVM, "clang-offload-bundler"), "--unbundle", "--type=o",
                    f"--targets=hipv4-amdgcn-amd-amdhsa--{B.ARCH}", f"--input={fat}", f"--output={code}"], check=True)
    notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", code], check=True, capture_output=True,
                           text=True).stdout
    kernels = re.findall(r"\.symbol: +(\S+).*?\.vgpr_spill_count: +(\d+)", notes, re.S)
    assert kernels
    assert [k for k, n in kernels if int(n)] == []
