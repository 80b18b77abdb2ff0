"""Inflow conditions that the general 2D step kernel applies to its own boundary
nodes (vortex and 1D-like fields) against the oracle, on grids where most
nodes lie on a face and where a wave holds several rows or part of one."""
import numpy as np
import pytest

import oracle
import paper_0905_3409_amd as pkg
from gpu_util import TOL64, gpu_advance, rel, rel_psi
from paper_0905_3409_amd import inputs
from test_gpu_inflow import _coords, _moving_data, _nearly_consistent, gpu_inflow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,period", [(inputs.PSEUDO1D, 0.0), (inputs.VORTEX, 1.7)])
@pytest.mark.parametrize("bc", [pkg.BC_INFLOW, pkg.BC_INFLOW_NEUMANN])
@pytest.mark.parametrize("psi", [pkg.PSI_SUPERCONSISTENT, pkg.PSI_HEUN])
@pytest.mark.parametrize("ncell", [(2, 2), (9, 2), (2, 9), (63, 4), (255, 2), (130, 33)])
def test_step_kernels_own_boundary_nodes(kind, period, bc, psi, ncell):
    lo, hi = (-0.1, 0.05), (1.05, 0.95)  # off the unit box the vortex crosses the faces too
    params = np.zeros(0)
    coords = _coords(ncell, lo, hi)
    data = _nearly_consistent(_moving_data(coords, k=[2.1, 1.3], w=1.9), coords, ncell, kind,
                              params, period)
    phi0, psi0, _ = data(0.0)
    args = (2, ncell, lo, hi, kind, params, period, phi0, psi0, 0.0, 0.01, 3)
    print(f"case kind={kind} bc={bc} psi={psi} {ncell}", flush=True)
    if bc == pkg.BC_INFLOW:
        g = gpu_inflow(*args, data, psi=psi)
        o = oracle.advance_inflow(*args, data, psi_update=psi)
    else:
        g = gpu_advance(*args, dtype="float64", bc=bc, psi=psi)
        o = oracle.advance(*args, bc=oracle.BC_INFLOW_NEUMANN, psi_update=psi)
    hmin = min((hi[a] - lo[a]) / ncell[a] for a in range(2))
    assert rel(g[0], o[0]) <= TOL64
    assert rel_psi(g[1], o[1], o[0], hmin) <= TOL64
