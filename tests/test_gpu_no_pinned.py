"""Where no pinned host memory can be had, reports, the substep's minimum
density and the projection's residual are copied from device memory instead:
the same numbers and fields, bit for bit.  A child process loads a small
library with a hipHostMalloc that can be told to fail, in front of the
runtime's, and runs each call both ways."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
int pinned_fail = 0, pinned_failed = 0;
int hipHostMalloc(void **p, size_t n, unsigned f)
{
    static int (*next)(void **, size_t, unsigned);
    if (pinned_fail) { ++pinned_failed; return 2; /* hipErrorOutOfMemory */ }
    if (!next) next = (int (*)(void **, size_t, unsigned))dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), "hipHostMalloc");
    return next(p, n, f);
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import torch
torch.zeros(1, device="cuda")
from paper_2502_04189_amd import pcx, workloads as W
from tests.gpu_util import to_dev
fail, failed = (ctypes.c_int.in_dll(shim, n) for n in ("pinned_fail", "pinned_failed"))
c = W.random_case(3, 64, 48, 24, 0, 0, 1, stretch=1.1)
rho, ps, u, v, w = [to_dev(a) for a in c.fields()]
phi = (rho - rho.min()) / (rho.max() - rho.min())
zero = lambda: torch.zeros_like(rho)

def run():
    out = []
    for prec in ("fp64", "fp32_refined"):
        p = pcx.Plan(c.grid, prec)
        out += p.step(c.dt, c.rho0, rho, ps, u, v, w)
        p.close()
    f = pcx.Flow(c.grid, 1.0, 50.0, 1e-3, 1e-2, sigma=0.01, gamma=0.1)
    o = [zero() for _ in range(5)]
    out += [f.substep(1, 1e-4, phi, u, v, w, ps, ps, 0.0, [zero() for _ in range(4)], o)] + o
    out += f.predict(1, 1e-4, phi, u, v, w, ps, ps, 0.0, [zero() for _ in range(4)], zero())
    f.close()
    vc = pcx.VarCoef(c.grid)
    out += vc.project(c.dt, c.rho0, rho, u, v, w, tol=1e-10)
    vc.close()
    torch.cuda.synchronize()
    return out

want = run()
assert failed.value == 0
fail.value = 1
got = run()
fail.value = 0
assert failed.value == 4, failed.value
assert len(got) == len(want)
for a, b in zip(got, want):
    assert torch.equal(a, b) if torch.is_tensor(a) else a == b, (a, b)
print("same")
"""


def test_copies_in_place_of_pinned_memory(tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    src, so = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"])
    r = subprocess.run([sys.executable, "-c", CHILD, str(so)], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("same"), r.stdout[-2000:] + r.stderr[-2000:]
