"""The variable-coefficient operator against its oracle where its tiles end:
the smallest grids, columns and rows past a tile, chunks of one plane and
of several with a remainder, more tiles than workgroups, every wall.

Tolerance: a face flux takes 8 roundings, the cell's sum of six of them and
their factors 6 more, so the error is below 6 (8 + 6) 2^-53 = 9.4e-15 of the
largest term; with random p the largest |out| is at least a tenth of that
term: 1e-13."""
import sys

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


@pytest.mark.parametrize("dims,bc,stretch", [((2, 4, 2), (0, 0, 0), 0.0), ((2, 3, 2), (1, 1, 1), 0.0),
                                             ((72, 12, 5), (0, 0, 1), 1.2), ((72, 18, 40), (1, 0, 0), 0.0),
                                             ((216, 54, 31), (0, 1, 1), 1.3), ((1152, 972, 3), (0, 0, 1), 0.0),
                                             ((1152, 972, 3), (1, 1, 0), 0.0)])
def test_operator_tiles(pcx, orc, dims, bc, stretch):
    print(f"varcoef tiles {dims} bc {bc}", flush=True)
    sys.stdout.flush()
    c = W.random_case(41, *dims, *bc, stretch=stretch)
    p = np.random.default_rng(5).normal(size=c.grid.shape)
    ref = orc.varcoef_apply(orc.Grid.from_workload(c.grid), c.rho, p)
    vc = pcx.VarCoef(c.grid)
    got = vc.apply(to_dev(c.rho), to_dev(p)).cpu().numpy()
    vc.close()
    assert np.abs(got - ref).max() <= 1e-13 * np.abs(ref).max()
