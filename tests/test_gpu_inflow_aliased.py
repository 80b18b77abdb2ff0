"""Dirichlet inflow data that are the advanced state itself (boundary values held
where the flow enters): a step that ends in the workspace takes the data of its
start, a step on the way back keeps what it computed. Bit for bit against steps
whose data lie in buffers of their own."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

AFF2 = inputs.affine_params([0.3, -0.2], [0.4, 0.5], [[0.1, -1.5], [1.2, -0.1]])
AFF3 = inputs.affine_params([0.3, -0.2, 0.1], [0.4, 0.5, 0.5],
                            [[0.1, -1.5, 0.2], [1.2, -0.1, 0.0], [0.3, 0.2, 0.0]])
STREAM = np.array([0.05, 1, 3, -0.03, 4, 2])


def _grids(kind, params, ncell, dtype, n):
    lo, hi = (-0.1, 0.05, 0.0)[: len(ncell)], (1.05, 0.95, 0.9)[: len(ncell)]
    out = []
    for bc in (pkg.BC_INFLOW, pkg.BC_INFLOW, pkg.BC_NEUMANN)[:n]:
        g = pkg.Grid(ncell, lo, hi, dtype=dtype, bc=bc)
        g.set_velocity(kind, params, 1.7)
        out.append(g)
    return out


@pytest.mark.parametrize("kind,params,ncell", [
    (pkg.VORTEX, (), (40, 33)), (pkg.PSEUDO1D, (), (67, 20)), (pkg.AFFINE, AFF2, (40, 33)),
    (pkg.STREAM_SIN, STREAM, (33, 40)), (pkg.AFFINE, AFF3, (11, 9, 12)),
    (pkg.LEVEQUE3D, (), (9, 12, 10))])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("save", [False, True])
def test_data_in_the_state(kind, params, ncell, dtype, save):
    import torch
    print(f"case kind={kind} {ncell} {dtype} save={save}", flush=True)
    own, apart, plain = _grids(kind, params, ncell, dtype, 3)
    rng = np.random.default_rng(4)
    n = own.num_nodes
    st = own.from_numpy(rng.normal(size=n), rng.normal(size=len(ncell) * n))
    phit = own.plane_from_numpy(rng.normal(size=n))
    dt = 0.01
    for steps in (1, 2, 3):
        a = st.clone()
        own.set_inflow_data(a, phit)
        ck = None
        if save:
            ck = own.advance_save(a, 0.1, dt, steps, 2)
        else:
            own.advance(a, 0.1, dt, steps)
        b, states = st.clone(), []
        for k in range(steps):
            states.append(b.clone())
            t = 0.1 + k * dt
            data = b.clone()
            if k % 2:  # back from the workspace: the step's own values are the data
                plain.advance(data, t, dt, 1)
            apart.set_inflow_data(data, phit)
            apart.advance(b, t, dt, 1)
        torch.cuda.synchronize()
        va, vb = (torch.stack([own._grid_view(s[q]) for q in range(1 + own.dim)]) for s in (a, b))
        assert torch.equal(va, vb), steps
        assert not torch.equal(va, torch.stack([own._grid_view(st[q]) for q in range(1 + own.dim)]))
        if save:
            sb = own.checkpoint_bytes(1, 1)
            for k, s in enumerate(states[::2]):
                c = ck[k * sb: (k + 1) * sb].view(own.torch_dtype)[: (1 + own.dim) * own.plane]
                c = c.view(1 + own.dim, own.plane)
                for q in range(1 + own.dim):
                    assert torch.equal(own._grid_view(c[q]), own._grid_view(s[q])), (steps, k)
