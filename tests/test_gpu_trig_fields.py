"""The vortex (FP64) and the 3D deformation field, whose stages shift the
node's sines and cosines by angle addition: stage offsets inside and beyond
the series' range against the oracle, and advances long enough to read the
per-axis table against the same steps in calls too short for it, bit for bit."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from gpu_util import TOL64, fp32_tolerances, gpu_advance, oracle_advance, rel, rel_psi
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

# field, cells, largest speed per axis
FIELDS = {"vortex": (inputs.VORTEX, (37, 29), 1.0), "leveque": (inputs.LEVEQUE3D, (13, 9, 11), 2.0)}


def _state(ncell, seed):
    rng = np.random.default_rng(seed)
    phi, psi = inputs.gaussian_bump(inputs.node_grid(ncell), [0.45] * len(ncell))
    return phi + 0.01 * rng.normal(size=phi.shape), psi + 0.01 * rng.normal(size=psi.shape)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("angle", [0.02, 0.19, 0.21, 0.26, 0.9])  # largest |pi d| of a stage
@pytest.mark.parametrize("field", sorted(FIELDS))
def test_stage_offsets_in_and_beyond_the_series(field, angle, dtype):
    kind, ncell, vmax = FIELDS[field]
    dim, steps = len(ncell), 3
    phi0, psi0 = _state(ncell, 7)
    args = (dim, ncell, (0.0,) * dim, (1.0,) * dim, kind, np.zeros(0), 2.5, phi0, psi0, 0.1,
            angle / (np.pi * vmax), steps)
    print(f"case {field} {angle} {dtype}", flush=True)
    g = gpu_advance(*args, dtype=dtype)
    o = oracle_advance(*args)
    hmin = 1.0 / max(ncell)
    if dtype == "float64":
        assert rel(g[0], o[0]) <= TOL64 and rel_psi(g[1], o[1], o[0], hmin) <= TOL64
    else:
        tp, tg = fp32_tolerances(o[0], o[1], hmin, steps)
        assert rel(g[0], o[0]) <= tp and rel(g[1], o[1]) <= tg


@pytest.mark.parametrize("field,ncell,dtype", [("vortex", (260, 255), "float64"),
                                               ("leveque", (40, 43, 39), "float64"),
                                               ("leveque", (40, 43, 39), "float32")])
def test_with_and_without_the_table(field, ncell, dtype):
    import torch
    kind = FIELDS[field][0]
    steps = 34  # from 2^21 node-steps on the table is built
    nodes = int(np.prod([n + 1 for n in ncell]))
    assert nodes * steps >= 2 ** 21 > nodes * (steps // 2)
    g = pkg.Grid(ncell, dtype=dtype)
    g.set_velocity(kind, np.zeros(0), 2.5)
    a = g.from_numpy(*_state(ncell, 3))
    b = a.clone()
    dt = 0.004
    print(f"case {field} {dtype}", flush=True)
    g.advance(a, 0.0, dt, steps)
    g.advance(b, 0.0, dt, steps // 2)
    g.advance(b, (steps // 2) * dt, dt, steps // 2)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
