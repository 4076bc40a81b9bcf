"""The x and y passes at every transform length with a fixed plan, against
the oracle: periodic and wall transforms, tiles that run over plane and mode
boundaries and end in the middle of one, both forms and the open (sine
transform) solve."""
import sys

import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests.gpu_util import errors, run_plan, to_dev

pytestmark = pytest.mark.gpu

# half lengths of x and lengths of y, short ones paired with long ones
XHALF = (16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 243, 256, 288, 324, 384, 432, 486,
         512)
YLEN = XHALF + (576, 648, 729, 768, 864, 972, 1024)
PAIRS = [(XHALF[min(i, len(XHALF) - 1)], YLEN[len(YLEN) - 1 - i]) for i in range(len(YLEN))]


@pytest.fixture(scope="module")
def pcx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_04189_amd import pcx as P
    P.lib()
    return P


def _bounds(case, f_inf, ref):
    """Relative bounds on u, v, w and p.  The transforms of f and of p are
    each off by at most 2 eps log2(nx ny) of the 2-norm (a factor 2 for the
    oracle's own), and the solve divides by at least the smallest non-zero
    eigenvalue: |dp| <= 4 eps log2(nx ny) sqrt(n) max|f| / lambda_min; the
    velocity follows as 2 dt / (rho0 h_min) |dp|, beside the parity bound
    1e-12."""
    g = case.grid
    eps = np.finfo(np.float64).eps
    lam = min(np.pi / g.lx if g.bcx else 2 * np.pi / g.lx, np.pi / g.ly if g.bcy else 2 * np.pi / g.ly,
              np.pi / g.lz if g.bcz else 2 * np.pi / g.lz) ** 2 * 4 / np.pi ** 2
    dp = 4 * eps * np.log2(g.nx * g.ny) * np.sqrt(g.cells) * f_inf / lam
    du = 2 * case.dt / (case.rho0 * min(g.dx, g.dy, float(np.diff(g.zf).min()))) * dp
    return {n: 1e-12 + (dp if n == "p" else du) / np.abs(r).max() for n, r in zip("uvwp", ref)}


def _run(pcx, orc, m, ny, bc, nz, prec):
    case = W.random_case(m + ny, 2 * m, ny, nz, *bc, stretch=1.1 if bc[2] else 0.0)
    print(f"{case.name} {prec}", flush=True)
    sys.stdout.flush()
    ref = orc.step(orc.Grid.from_workload(case.grid), case.dt, case.rho0, *case.fields())[:4]
    plan = pcx.Plan(case.grid, prec)
    got, rep = run_plan(plan, case)
    plan.close()
    e = errors(got, ref)
    print(f"  errors {e} residual {rep['rel_residual']:.2e}", flush=True)
    return case, e, rep, ref


# The residual |f - L p| / |f| is the sharp check (a wrong mode shows in full,
# whatever its eigenvalue); 1e-12 as in the parity tests.
@pytest.mark.parametrize("m,ny", PAIRS)
def test_fp64_lengths(pcx, orc, m, ny):
    for bc, nz in (((0, 0, 1), 3), ((1, 1, 0), 5)):
        if bc[1] == 0 and ny % 2:
            continue
        case, e, rep, ref = _run(pcx, orc, m, ny, bc, nz, "fp64")
        assert rep["max_div_rel"] <= 1e-12
        tol = _bounds(case, rep["f_inf"], ref)
        assert all(e[n] <= tol[n] for n in e), (e, tol)


@pytest.mark.parametrize("m,ny", PAIRS)
def test_refined_lengths(pcx, orc, m, ny):
    case, e, rep, ref = _run(pcx, orc, m, ny, (1, 1, 1) if ny % 2 else (0, 0, 0), 3, "fp32_refined")
    assert rep["converged"] == 1 and rep["max_div_rel"] <= 1e-10
    tol = _bounds(case, rep["f_inf"], ref)
    assert all(e[n] <= 1e-10 + tol[n] for n in e), (e, tol)


@pytest.mark.parametrize("m,ny", [p for p in PAIRS if p[0] * p[1] <= 81 * 128])
def test_open_solve_lengths(pcx, orc, m, ny):
    """L p = f with open x and y: the oracle's explicit sine sums (O(n^2))."""
    nx, nz = 2 * m, 3
    g = W.GridSpec(nx, ny, nz, nx / 32.0, ny / 32.0, W.zf_uniform(nz, 0.1), 2, 2, 1)
    print(f"open {nx}x{ny}x{nz}", flush=True)
    f = np.random.default_rng(m + ny).standard_normal(g.shape)
    plan = pcx.Plan(g, "fp64")
    got = plan.poisson_solve(to_dev(f)).cpu().numpy()
    plan.close()
    ref = orc.poisson_bc(orc.Grid.from_workload(g), f)
    err = float(np.abs(got - ref).max() / np.abs(ref).max())
    print(f"  error {err:.2e}", flush=True)
    assert err <= 1e-12
