"""Points on the nodes of a grid, the last ones of every axis among them, return the
nodes' data: phi bit for bit, and the normal of psi."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell", [(16, 12), (2, 3), (9, 8, 7), (2, 2, 2), (5, 11, 64)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("mixed", [pkg.MIXED_CENTRAL, pkg.MIXED_CELL, pkg.MIXED_ZERO])
def test_points_on_nodes(ncell, dtype, mixed):
    import torch
    print(f"case {ncell} {dtype} {mixed}", flush=True)
    dim = len(ncell)
    # cells of size 1: the nodes' coordinates are exact
    g = pkg.Grid(ncell, (0.0,) * dim, tuple(float(n) for n in ncell), dtype=dtype, mixed=mixed)
    rng = np.random.default_rng(dim)
    st = g.from_numpy(rng.normal(size=g.num_nodes), rng.normal(size=dim * g.num_nodes))
    val, nrm, _ = g.eval_points(st, np.stack(inputs.node_grid(ncell, g.lo, g.hi), 1))
    torch.cuda.synchronize()
    psi = torch.stack([g._grid_view(st[1 + a]).reshape(-1) for a in range(dim)])
    assert torch.equal(val, g._grid_view(st[0]).reshape(-1))
    # the sum of squares, the root and the quotient: at most 4 roundings
    ref = psi.double() / torch.sqrt((psi.double() ** 2).sum(0))
    assert float((nrm.double() - ref).abs().max()) <= 4 * torch.finfo(st.dtype).eps / 2


@pytest.mark.parametrize("ncell", [(6, 5), (5, 4, 6)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_data_that_are_not_finite_show_at_every_point_of_their_cells(ncell, dtype, bad):
    import torch
    print(f"case {ncell} {dtype} {bad}", flush=True)
    dim = len(ncell)
    g = pkg.Grid(ncell, (0.0,) * dim, tuple(float(n) for n in ncell), dtype=dtype)
    rng = np.random.default_rng(dim)
    phi = rng.normal(size=g.num_nodes)
    node = np.array([3, 2, 4][:dim])
    phi[np.ravel_multi_index(node[::-1], g.nodes[::-1])] = bad
    st = g.from_numpy(phi, rng.normal(size=dim * g.num_nodes))
    pts = np.stack(inputs.node_grid(ncell, g.lo, g.hi), 1)
    val, nrm, cur = (v.cpu().numpy() for v in g.eval_points(st, pts))
    torch.cuda.synchronize()
    # a node's point lies in the cell it is the first vertex of, or in the last one
    cell = np.minimum(pts, np.array(ncell) - 1)
    touched = ((node >= cell) & (node <= cell + 1)).all(axis=1)
    assert np.array_equal(~np.isfinite(val), touched)
    assert (nrm[:, touched] == 0.0).all() and (cur[touched] == 0.0).all()
    assert np.isfinite(nrm).all() and np.isfinite(cur).all()
