"""Refined steps of lone closed domains with few tiles (general passes in x,
in y or in both) and with just enough for the fixed-plan ones, against the
oracle, and shallow periodic ones, whose z-lines are not padded."""
import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests.gpu_util import errors, run_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_04189_amd import pcx as P
    P.lib()
    return P


# 1e-10 is the refined form's own bar; cubic cells and sides within 1 : 32 of
# one another keep the smallest eigenvalue's amplification of rounding below it
@pytest.mark.parametrize("dims,bc", [
    ((64, 64, 3), (1, 1, 1)), ((64, 64, 9), (1, 1, 1)), ((64, 64, 128), (1, 1, 1)), ((64, 64, 129), (1, 1, 1)),
    ((32, 48, 16), (1, 1, 0)), ((256, 32, 10), (1, 0, 1)), ((32, 256, 10), (0, 1, 1)), ((162, 81, 5), (1, 1, 1)),
    ((64, 64, 2), (0, 0, 1)), ((96, 54, 10), (0, 0, 0))])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32_refined", 1e-10)])
def test_few_tiles_vs_oracle(pcx, orc, dims, bc, prec, tol):
    case = W.random_case(sum(dims), *dims, *bc)
    print(f"{case.name} {prec}", flush=True)
    ref = orc.step(orc.Grid.from_workload(case.grid), case.dt, case.rho0, *case.fields())[:4]
    plan = pcx.Plan(case.grid, prec)
    got, rep = run_plan(plan, case)
    plan.close()
    e = errors(got, ref)
    print(f"  errors {e} residual {rep['rel_residual']:.2e}", flush=True)
    assert rep["max_div_rel"] <= tol and all(np.isfinite(g).all() for g in got)
    assert max(e.values()) <= tol
