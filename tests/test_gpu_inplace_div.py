"""The in-place step: its velocity equals the out-of-place step's bit for bit,
and the separate divergence pass reports max |D u_out| of the velocity it
stored, on rows shorter and longer than a wave, chunk remainders and every
kind of wall."""
import sys

import numpy as np
import pytest

from paper_2502_04189_amd import workloads as W
from tests.gpu_util import check_div, run_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pcx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_04189_amd import pcx as P
    P.lib()
    return P


@pytest.mark.parametrize("dims,bc", [((2, 3, 2), (1, 1, 0)), ((6, 9, 5), (1, 1, 1)), ((96, 27, 70), (1, 1, 0)),
                                     ((144, 32, 37), (0, 0, 1)), ((64, 96, 130), (0, 1, 1))])
def test_inplace_divergence(pcx, orc, dims, bc):
    case = W.random_case(17 + sum(dims), *dims, *bc, stretch=1.2 if bc[2] else 0.0)
    print(f"in place {case.name}", flush=True)
    sys.stdout.flush()
    plan = pcx.Plan(case.grid, "fp64")
    ref, _ = run_plan(plan, case)
    got, rep = run_plan(plan, case, inplace=True)
    plan.close()
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)
    # outputs on wall faces are written 0, so check_div's D sees what the pass saw
    check_div(orc, case, got, rep, case.name)
