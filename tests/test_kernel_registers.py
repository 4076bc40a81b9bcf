"""No kernel of the library spills vector registers or keeps anything in
scratch memory: read from the metadata of the built code objects.  CPU only."""
import os
import re
import shutil
import subprocess

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_04189_amd")
LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")), reason="ROCm's LLVM tools not installed")
def test_no_kernel_spills(tmp_path):
    lib = shutil.copy(os.path.join(PKG, "libpcx.so"), tmp_path)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    kernels, bad = 0, []
    for f in sorted(p for p in os.listdir(tmp_path) if "gfx950" in p):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", f], cwd=tmp_path, check=True,
                               capture_output=True, text=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            val = lambda key: re.search(r"\." + key + r":\s+(\S+)", k)[1]
            kernels += 1
            if int(val("vgpr_spill_count")) or int(val("private_segment_fixed_size")):
                bad.append((val("symbol"), val("vgpr_spill_count"), val("private_segment_fixed_size")))
    assert kernels > 100
    assert not bad, bad
