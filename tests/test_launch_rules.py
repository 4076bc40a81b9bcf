"""Host-side checks of the rules that choose strides, tiles and chunks of
planes, and of what the create calls do without pinned memory, by compiling and running tests/hostcheck/*_check.cpp against the
library's own headers and, where a rule is not in one, the library itself
(host code only: no device call).  CPU only."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2502_04189_amd")
LIB = ["-L" + PKG, "-l:libpcx.so", "-Wl,-rpath," + PKG]
LINK = {"shapes": LIB, "no_pinned": LIB, "fft_lds": LIB}
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("rule", ["z_stride", "shapes", "no_pinned", "march_chunk", "momentum_chunk", "fft_lds", "tune_items", "vec_wgs"])
def test_rule(tmp_path, rule):
    exe = tmp_path / rule
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I",
                           os.path.join(ROOT, "paper_2502_04189_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                           os.path.join(HERE, "hostcheck", rule + "_check.cpp"), "-o", str(exe)] + LINK.get(rule, []))
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
