"""The wall and open transforms at every length with a fixed plan: refined
steps of closed boxes (the FP32 cosine passes, stored and accumulated), and
the open solve (sine transforms) with each x half length and each y length
beside a short other side, against the oracle.  tests/test_gpu_lengths.py
pairs short lengths with long ones, which leaves most of these out."""
import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests.gpu_util import to_dev
from tests.test_gpu_lengths import PAIRS, XHALF, YLEN, _bounds, _run, pcx  # noqa: F401

pytestmark = pytest.mark.gpu


# The residual and the bounds are those of test_refined_lengths; enough planes
# for more than 64 x tiles (of at most 4096 points and 16 to 128 rows) and 16 y
# tiles, below which a lone closed domain takes the general passes.
@pytest.mark.parametrize("m,ny", [p for p in PAIRS if p[1] % 2 == 0])
def test_refined_closed_lengths(pcx, orc, m, ny):  # noqa: F811
    rows = min(128, max(16, 4096 // m))
    case, e, rep, ref = _run(pcx, orc, m, ny, (1, 1, 1), max(7, -(-66 * rows // ny)), "fp32_refined")
    assert rep["converged"] == 1 and rep["max_div_rel"] <= 1e-10
    tol = _bounds(case, rep["f_inf"], ref)
    assert all(e[n] <= 1e-10 + tol[n] for n in e), (e, tol)


@pytest.mark.parametrize("m,ny", [(m, 16) for m in XHALF] + [(16, ny) for ny in YLEN if ny != 16])
def test_open_solve_each_length(pcx, orc, m, ny):  # noqa: F811
    """L p = f with open x and y.  The transforms are off by at most 4 eps
    log2(nx ny) of the 2-norm (a factor 2 for the oracle's sums), the solve
    divides by at least the smallest eigenvalue: |dp| <= 4 eps log2(nx ny)
    sqrt(n) max|f| / lambda_min, beside the parity bound 1e-12."""
    nx, nz = 2 * m, 3
    g = W.GridSpec(nx, ny, nz, nx / 32.0, ny / 32.0, W.zf_uniform(nz, 0.1), 2, 2, 1)
    print(f"open {nx}x{ny}x{nz}", flush=True)
    f = np.random.default_rng(7 * m + ny).standard_normal(g.shape)
    plan = pcx.Plan(g, "fp64")
    got = plan.poisson_solve(to_dev(f)).cpu().numpy()
    plan.close()
    ref = orc.poisson_bc(orc.Grid.from_workload(g), f)
    lam = ((np.pi / g.lx) ** 2 + (np.pi / g.ly) ** 2) * 4 / np.pi ** 2
    tol = 1e-12 + 4 * np.finfo(np.float64).eps * np.log2(nx * ny) * np.sqrt(g.cells) * np.abs(f).max() / lam / np.abs(ref).max()
    err = float(np.abs(got - ref).max() / np.abs(ref).max())
    print(f"  error {err:.2e} of {tol:.2e}", flush=True)
    assert err <= tol
