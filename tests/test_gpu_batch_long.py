"""Batches of domains with sides above 128: the grouped launches of the longer
fixed plans (one kernel a length, items of several domains, columns of
64-byte segments in pairs per XCD) beside those of the short ones, against
single-domain plans bit for bit in FP64 and the oracle in the refined form."""
import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests import manufactured as M
from tests.test_gpu_batch import _domains, _outs, pcx  # noqa: F401
from tests.test_gpu_lengths import _bounds

pytestmark = pytest.mark.gpu

SPECS = [((288, 144, 9), (0, 0, 1)), ((288, 32, 17), (1, 0, 1)), ((32, 648, 5), (0, 0, 1)), ((48, 648, 10), (0, 1, 0)),
         ((64, 1024, 4), (0, 0, 1)), ((36, 972, 7), (0, 0, 0)), ((1024, 36, 6), (0, 0, 1)), ((324, 162, 12), (1, 1, 1)),
         ((512, 243, 5), (0, 1, 1)), ((64, 64, 33), (0, 0, 1)), ((1152, 48, 5), (0, 0, 1)), ((48, 1296, 4), (0, 0, 1))]


def _cases():
    return [W.random_case(300 + i, *d, *bc) for i, (d, bc) in enumerate(SPECS)]


def test_fp64_long_sides_match_plans_bitwise(pcx):  # noqa: F811
    import torch
    cases = _cases()
    print("batch fp64: " + ", ".join(c.name for c in cases), flush=True)
    doms = _domains(cases)
    b = pcx.Batch(doms, "fp64")
    for launch in range(2):
        b.launch()
    torch.cuda.synchronize()
    for c, d in zip(cases, doms):
        plan = pcx.Plan(c.grid, "fp64")
        uo, vo, wo, p, _ = plan.step(c.dt, c.rho0, d["rho"], d["pstar"], d["u"], d["v"], d["w"])
        for x, y in zip((uo, vo, wo, p), (d["u_out"], d["v_out"], d["w_out"], d["p_out"])):
            assert torch.equal(x, y), c.name
        plan.close()
    b.close()


def test_refined_long_sides_vs_oracle(pcx, orc):  # noqa: F811
    import torch
    cases = _cases()
    print("batch refined: " + ", ".join(c.name for c in cases), flush=True)
    doms = _domains(cases)
    b = pcx.Batch(doms, "fp32_refined")
    b.launch()
    torch.cuda.synchronize()
    reps, st = b.reports()
    for c, d, r in zip(cases, doms, reps):
        ref = orc.step(orc.Grid.from_workload(c.grid), c.dt, c.rho0, *c.fields())[:4]
        e = {n: M.relerr(x, y) for n, x, y in zip("uvwp", _outs(d), ref)}
        tol = _bounds(c, r["f_inf"], ref)
        print(f"{c.name}: errors {e} div {r['max_div_rel']:.2e}", flush=True)
        assert all(np.isfinite(x).all() for x in _outs(d))
        assert r["max_div_rel"] <= 1e-10 and all(e[n] <= 1e-10 + tol[n] for n in e), (c.name, e, tol)
    # a batch runs three solves; the stop test may ask an elongated domain for more
    assert st == (pcx.PCX_OK if all(r["converged"] for r in reps) else pcx.PCX_ERR_NOT_CONVERGED)
    b.close()
