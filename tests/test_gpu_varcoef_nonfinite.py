"""The projection reports a residual norm that is not finite
(PCX_ERR_NONFINITE): a NaN or an infinity in a velocity or in the density,
and velocities whose divergence norm overflows, end the call with that
status at the first norm they reach, and the handle then solves a finite
problem as a new one does."""
import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_04189_amd import pcx as P
    P.lib()
    return P


@pytest.mark.parametrize("field,value,iters", [
    ("u", np.nan, 0), ("w", np.inf, 0), ("v", 1e200, 0), ("rho", np.nan, 1), ("rho", -np.nan, 1)])
def test_nonfinite_input_is_reported(pcx, field, value, iters):
    import torch
    c = W.random_case(77, 48, 18, 10, 0, 1, 1, stretch=1.1)
    rho, _, u, v, w = [to_dev(a) for a in c.fields()]
    vc = pcx.VarCoef(c.grid)
    print(f"{field} {value}", flush=True)
    want = vc.project(c.dt, c.rho0, rho, u, v, w, tol=1e-10)
    assert want[6] == pcx.PCX_OK
    bad = {"rho": rho, "u": u, "v": v, "w": w}
    bad[field] = bad[field].clone()
    bad[field][4, 7, 20] = value
    got = vc.project(c.dt, c.rho0, bad["rho"], bad["u"], bad["v"], bad["w"], tol=1e-10, check=False)
    torch.cuda.synchronize()
    assert got[6] == pcx.PCX_ERR_NONFINITE, got[4:]
    assert got[4] == iters and not np.isfinite(got[5]), got[4:]
    again = vc.project(c.dt, c.rho0, rho, u, v, w, tol=1e-10)
    assert again[4:] == want[4:]
    for a, b in zip(again[:4], want[:4]):
        assert torch.equal(a, b)
    vc.close()
