"""The z solve at line lengths that fill its lanes' levels exactly, fall short
of them by one to many (the rows past the end) or are not a whole number of
128-byte lines, periodic and wall, both forms, against the oracle."""
import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests.gpu_util import to_dev
from tests.test_gpu_lengths import _bounds, _run, pcx  # noqa: F401

pytestmark = pytest.mark.gpu

NZ = (2, 3, 4, 5, 7, 9, 15, 17, 24, 33, 49, 64, 75, 96, 100, 127, 130, 250, 257, 449, 512, 513, 700, 1024)


@pytest.mark.parametrize("nz", NZ)
@pytest.mark.parametrize("prec,tol0", [("fp64", 1e-12), ("fp32_refined", 1e-10)])
def test_line_lengths(pcx, orc, nz, prec, tol0):  # noqa: F811
    for bc in ((0, 0, 1), (0, 1, 0)):
        case, e, rep, ref = _run(pcx, orc, 8, 18, bc, nz, prec)
        assert rep["max_div_rel"] <= tol0
        tol = _bounds(case, rep["f_inf"], ref)
        assert all(e[n] <= tol0 + tol[n] for n in e), (e, tol)


@pytest.mark.parametrize("nz", [3, 9, 65, 130, 250])
def test_open_lines(pcx, orc, nz):  # noqa: F811
    """Dirichlet z: the last row's coefficients differ, the rows past it do not
    touch it.  p = 0 on both ends bounds |p| by |f| h-independently: 1e-12."""
    g = W.GridSpec(16, 18, nz, 0.5, 0.5, W.zf_tanh(nz, 0.5, 1.3), 0, 1, 2)
    f = np.random.default_rng(nz).standard_normal(g.shape)
    print(f"open z {nz}", flush=True)
    plan = pcx.Plan(g, "fp64")
    got = plan.poisson_solve(to_dev(f)).cpu().numpy()
    plan.close()
    ref = orc.poisson_bc(orc.Grid.from_workload(g), f)
    assert float(np.abs(got - ref).max() / np.abs(ref).max()) <= 1e-12
