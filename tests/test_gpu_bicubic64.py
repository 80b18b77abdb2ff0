"""The FP64 bicubic with folded cross derivatives on the smallest grids (two and
three cells, where every cell is a first or last one) against the oracle, and
exact shifts whose feet land on the grid's last node, in 2D and 3D, with NaN in
the padding."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from gpu_util import TOL64, oracle_advance, rel, rel_psi
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

STREAM = np.array([0.05, 1, 3, -0.03, 4, 2, 0.02, 2, 2])


def _grid(ncell, kind, params, dtype="float64", hi=None):
    import torch
    rng = np.random.default_rng(sum(ncell))
    g = pkg.Grid(ncell, hi=hi, dtype=dtype)
    g.set_velocity(kind, params, 0.0)
    n = g.num_nodes
    st = g.from_numpy(rng.normal(size=n), rng.normal(size=len(ncell) * n))
    pad = torch.full_like(st, float("nan"))
    for a in range(st.shape[0]):
        g._grid_view(pad[a]).copy_(g._grid_view(st[a]))
    return g, pad


@pytest.mark.parametrize("kind,params", [(inputs.STREAM_SIN, STREAM),
                                         (inputs.VORTEX, np.zeros(0)),
                                         (inputs.PSEUDO1D, np.zeros(0))])
@pytest.mark.parametrize("ncell", [(2, 2), (3, 2), (2, 5), (63, 2), (300, 300)])
def test_smallest_grids(ncell, kind, params):
    import torch
    g, st = _grid(ncell, kind, params)
    phi0, psi0 = g.to_numpy(st)
    print(f"case {ncell} kind {kind}", flush=True)
    steps, dt = 3, 0.3 / max(ncell)
    g.advance(st, 0.1, dt, steps)
    torch.cuda.synchronize()
    phi, psi = g.to_numpy(st)
    o = oracle_advance(2, ncell, (0.0, 0.0), (1.0, 1.0), kind, params, 0.0, phi0, psi0, 0.1, dt,
                       steps)
    assert rel(phi, o[0]) <= TOL64
    assert rel_psi(psi, o[1], o[0], 1.0 / max(ncell)) <= TOL64


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("shift", [(1, 0), (-1, 0), (0, -2), (-3, 1), (1, 0, 0), (-1, 0, 0),
                                   (0, -2, 0), (0, 0, -1), (-1, -1, -1)])
def test_exact_shifts_to_the_last_node(shift, dtype):
    import torch
    dim = len(shift)
    ncell = (16, 8, 8)[:dim]
    h, dt = 1.0 / 16, 1.0 / 32
    vel = [s * h / dt for s in shift]
    params = inputs.affine_params(vel, [0.0] * dim, np.zeros((dim, dim)))
    g, st = _grid(ncell, inputs.AFFINE, params, dtype, hi=[n * h for n in ncell])
    phi0, psi0 = g.to_numpy(st)
    print(f"case {shift} {dtype}", flush=True)
    g.advance(st, 0.0, dt, 1)
    torch.cuda.synchronize()
    phi, psi = g.to_numpy(st)
    shape = tuple(reversed(g.nodes))
    P0, P = phi0.reshape(shape), phi.reshape(shape)
    S0, S = psi0.reshape((dim,) + shape), psi.reshape((dim,) + shape)
    # node i takes the data of node i - shift, where that is in the grid
    dst = tuple(slice(max(s, 0), n + 1 + min(s, 0)) for n, s in zip(ncell, shift))[::-1]
    src = tuple(slice(max(-s, 0), n + 1 + min(-s, 0)) for n, s in zip(ncell, shift))[::-1]
    np.testing.assert_array_equal(P[dst], P0[src])
    for a in range(dim):
        np.testing.assert_array_equal(S[a][dst], S0[a][src])
