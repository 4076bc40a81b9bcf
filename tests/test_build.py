"""The library's build ends with an error, not with a library whose solves
fail when they run, where a source is missing or an object has lost a kernel
table; and every table has a kernel for each length and number of levels the
host code chooses.  CPU only."""
import ctypes
import os
import re
import shutil

import pytest

from paper_2502_04189_amd import build as B

CSRC = B.CSRC


def test_missing_source_stops_the_build(tmp_path, monkeypatch):
    monkeypatch.setattr(B, "CSRC", str(tmp_path))
    monkeypatch.setattr(B, "BUILD", str(tmp_path / "_build"))
    monkeypatch.setattr(B, "LIB", str(tmp_path / "libpcx.so"))
    monkeypatch.setattr(B, "_compile", lambda src: src)
    for s in B.SOURCES:
        if s != "pcx_z.hip":
            (tmp_path / s).write_text("")
    with pytest.raises(RuntimeError, match="pcx_z.hip"):
        B.build()
    assert not os.path.exists(B.LIB)


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_link_without_a_kernel_table_fails(tmp_path, monkeypatch):
    objs = [os.path.join(B.BUILD, os.path.splitext(s)[0] + ".o") for s in B.SOURCES]
    if not all(map(os.path.exists, objs)):
        pytest.skip("objects of a build not kept")
    monkeypatch.setattr(B, "LIB", str(tmp_path / "libpcx.so"))
    with pytest.raises(RuntimeError, match="z_kernel"):
        B.link([o for o in objs if not o.endswith("pcx_z.o")])
    assert not os.path.exists(B.LIB)


def test_every_table_has_its_kernels():
    lib = ctypes.CDLL(B.LIB)
    tables = {re.match(r"_ZN3pcx\d+(\w+?)Eii", s)[1]: getattr(lib, s) for s in B.REQUIRED}
    for f in tables.values():
        f.restype, f.argtypes = ctypes.c_void_p, [ctypes.c_int, ctypes.c_int]
    plans = [int(n) for n in re.findall(r"case (\d+): return", open(os.path.join(CSRC, "pcx_fplan.hpp")).read())]
    assert len(plans) == 33
    f64, f32 = 0, 1
    for prec in (f64, f32):
        for n in plans:
            for name, f in tables.items():
                if name == "z_kernel" or (name.startswith("fft_x") and n > 512) or (name == "fft_xinv_accum_kernel" and prec == f64):
                    continue
                assert f(prec, n), (name, prec, n)
            assert not any(tables[t](prec, n + 1) for t in tables if t != "z_kernel" and n > 128 and n + 1 not in plans)
        for levels in (2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16):
            assert tables["z_kernel"](prec, levels), (prec, levels)
