"""The marching flux pass through the phase and momentum right-hand sides
against the oracle: the smallest grids it takes, partial tiles in x and y
(rows in fours, tiles in eights), chunks of one plane and of several with a
remainder, wrap across each periodic direction, and the interior cells whose
normals the tiles along the walls read.

Tolerance: 1e-11 of the right-hand side's max norm.  The face fluxes differ
from the oracle's by a few ulps (device log and exp), and the right-hand side
is their difference over a cell width, about 100 times smaller: a few 1e-14,
with two decades for the steep profile's own conditioning."""
import sys

import numpy as np
import pytest

from tests.gpu_util import to_dev
from tests.test_gpu_flow import PARAMS, _case

pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.fixture(scope="module")
def pcx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_04189_amd import pcx as P
    P.lib()
    return P


@pytest.mark.parametrize("dims,bc,stretch", [((72, 6, 3), (0, 0, 0), 0.0), ((72, 12, 37), (0, 0, 0), 0.0),
                                             ((144, 12, 9), (1, 0, 1), 1.2), ((216, 18, 13), (1, 1, 1), 1.3),
                                             ((72, 24, 70), (0, 1, 0), 0.0), ((216, 54, 31), (0, 0, 0), 0.0)])
def test_flux_march(pcx, orc, dims, bc, stretch):
    gs, eps, phi, u, v, w, _, _ = _case(31 + sum(dims), *dims, bc, stretch)
    print(f"flux march {dims} bc {bc}", flush=True)
    sys.stdout.flush()
    g = orc.Grid.from_workload(gs)
    fl = orc.flow_params(eps=eps, **PARAMS)
    ref = [orc.acdi_rhs(g, fl, phi, u, v, w)] + list(orc.momentum_rhs(g, fl, phi, u, v, w))
    F = pcx.Flow(gs, eps=eps, **PARAMS)
    dev = [to_dev(a) for a in (phi, u, v, w)]
    got = [F.phase_rhs(*dev)] + list(F.momentum_rhs(*dev))
    got = [t.cpu().numpy() for t in got]
    F.close()
    for a, b in zip(got, ref):
        assert np.abs(a - b).max() <= TOL * np.abs(b).max()
