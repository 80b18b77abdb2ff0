"""The 3D interpolant with central cross derivatives on the smallest grids
(two and three cells: every cell is a first or last one), where the one-sided
differences change the stencil's weights, against the oracle; the padding of
the state holds NaN, which no result may see."""
import numpy as np
import pytest

import oracle
import paper_0905_3409_amd as pkg
from gpu_util import TOL64, fp32_tolerances, oracle_advance, rel, rel_psi
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

FIELDS = {
    "affine": (inputs.AFFINE, inputs.affine_params([0.05, 0.0, -0.1], [0.5, 0.5, 0.5],
                                                   [[0.2, -1.0, 0.5], [1.0, 0.1, -0.3],
                                                    [0.2, 0.6, -0.3]])),
    "vecpot": (inputs.VECPOT_SIN, np.array([0.05, -0.01, 0.02, 1, 3, 2, -0.02, 0.04, 0.01, 4, 2, 1])),
    "leveque": (inputs.LEVEQUE3D, np.zeros(0)),
}


def _state(ncell, dtype):
    import torch
    rng = np.random.default_rng(sum(ncell))
    n = int(np.prod([c + 1 for c in ncell]))
    g = pkg.Grid(ncell, dtype=dtype)
    st = g.from_numpy(rng.normal(size=n), rng.normal(size=3 * n))
    pad = torch.full_like(st, float("nan"))
    shape = tuple(reversed(g.nodes[1:])) + (g.pitch,)
    for a in range(4):
        pad[a].view(shape)[..., : g.nodes[0]] = st[a].view(shape)[..., : g.nodes[0]]
    return g, pad


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("ncell", [(2, 2, 2), (3, 2, 5), (2, 3, 2), (63, 2, 3), (64, 3, 2)])
@pytest.mark.parametrize("field", sorted(FIELDS))
def test_advance_on_the_smallest_grids(field, ncell, dtype):
    import torch
    kind, params = FIELDS[field]
    g, st = _state(ncell, dtype)
    phi0, psi0 = g.to_numpy(st)
    g.set_velocity(kind, params, 2.5)
    print(f"case {field} {ncell} {dtype}", flush=True)
    g.advance(st, 0.1, 0.04, 2)
    torch.cuda.synchronize()
    phi, psi = g.to_numpy(st)
    o = oracle_advance(3, ncell, (0.0,) * 3, (1.0,) * 3, kind, params, 2.5, phi0, psi0, 0.1, 0.04, 2)
    hmin = 1.0 / max(ncell)
    if dtype == "float64":
        assert rel(phi, o[0]) <= TOL64 and rel_psi(psi, o[1], o[0], hmin) <= TOL64
    else:
        tp, tg = fp32_tolerances(o[0], o[1], hmin, 2)
        assert rel(phi, o[0]) <= tp and rel(psi, o[1]) <= tg


@pytest.mark.parametrize("ncell", [(2, 2, 2), (3, 5, 2), (64, 2, 3)])
def test_points_on_the_smallest_grids(ncell):
    import torch
    g, st = _state(ncell, "float64")
    phi, psi = g.to_numpy(st)
    pts = np.random.default_rng(3).uniform(0.0, 1.0, (500, 3))
    print(f"case points {ncell}", flush=True)
    val, nrm, cur = (t.double().cpu().numpy() for t in g.eval_points(st, pts))
    torch.cuda.synchronize()
    o = oracle.eval_points(3, ncell, np.zeros(3), np.ones(3), phi, psi, pts)
    gn = np.linalg.norm(o["grad"], axis=1)
    ok = gn > 0.1 * gn.max()
    assert rel(val, o["val"]) <= TOL64
    assert np.abs(nrm.T - o["normal"])[ok].max() <= 100 * TOL64
    assert rel(cur[ok], o["kappa"][ok]) <= 1e-10
