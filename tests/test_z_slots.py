"""Host-side check of the z solve's LDS slots: the waves of its workgroups
are not synchronized, so each must read and write its own lines' slots only,
the padding of the lines in memory included.  Compiles and runs
tests/hostcheck/z_slot_check.cpp against the library's own header.  CPU only."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_z_waves_keep_to_their_own_lines(tmp_path):
    exe = tmp_path / "z_slot_check"
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I",
                           os.path.join(ROOT, "paper_2502_04189_amd", "csrc"),
                           os.path.join(HERE, "hostcheck", "z_slot_check.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
