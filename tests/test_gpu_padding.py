"""What the library touches of a state's planes: it copies the nodes of every row and
nothing else (the padding of the caller's planes is marked, and so is the copy's,
whose mark has to stay), and needs nothing past a plane's last node."""
import numpy as np
import pytest

import oracle
import paper_0905_3409_amd as pkg
from gpu_util import TOL64, U32, fp32_tolerances, rel, rel_psi

pytestmark = pytest.mark.gpu

STREAM = np.array([0.05, 1, 3, -0.03, 4, 2, 0.02, 2, 2])


@pytest.mark.parametrize("ncell", [(2, 5), (3, 4), (4, 3), (61, 4), (62, 3), (63, 5), (64, 2),
                                   (130, 33), (2, 4, 3), (5, 2, 6), (66, 3, 2)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("shift", [0, 1])  # elements past a 256-byte boundary
@pytest.mark.parametrize("save", [False, True])
def test_copy_of_the_state_leaves_padding_alone(ncell, dtype, shift, save):
    import torch
    print(f"case {ncell} {dtype} shift {shift} save {save}", flush=True)
    dim = len(ncell)
    g = pkg.Grid(ncell, dtype=dtype)
    if dim == 2:
        g.set_velocity(pkg.STREAM_SIN, STREAM, 2.0)
    else:
        g.set_velocity(pkg.LEVEQUE3D, (), 2.0)
    rng = np.random.default_rng(dim)
    init = g.from_numpy(rng.normal(size=g.num_nodes), rng.normal(size=dim * g.num_nodes))
    flat = torch.full((init.numel() + 8,), float("nan"), dtype=init.dtype, device=init.device)
    st = flat[shift: shift + init.numel()].view_as(init)
    for a in range(1 + dim):
        g._grid_view(st[a]).copy_(g._grid_view(init[a]))
    mark = 7.25
    if save:
        buf = torch.full((g.checkpoint_bytes(1, 1) // init.element_size(),), mark,
                         dtype=init.dtype, device=init.device)
        ck = g.advance_save(st, 0.1, 1e-3, 1, 1, ckpt=buf.view(torch.uint8))
        assert ck.data_ptr() == buf.data_ptr()
    else:
        buf = g.workspace()[: g.workspace_bytes].view(init.dtype)
        buf.fill_(mark)
        g.advance(st, 0.1, 1e-3, 1)
    torch.cuda.synchronize()
    shape = tuple(reversed(g.nodes[1:])) + (g.pitch,)
    for a in range(1 + dim):
        copy = buf[a * g.plane: (a + 1) * g.plane].view(shape)
        assert torch.equal(copy[..., : g.nodes[0]], g._grid_view(init[a]))
        assert (copy[..., g.nodes[0]:] == mark).all()
        assert torch.isfinite(g._grid_view(st[a])).all()
        assert torch.isnan(st[a].view(shape)[..., g.nodes[0]:]).all()


@pytest.mark.parametrize("ncell", [(4, 3), (5, 4), (6, 3), (61, 4), (62, 5), (63, 4), (64, 3),
                                   (2, 3, 2), (4, 5, 3), (5, 3, 4), (6, 4, 3), (63, 3, 3)])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_planes_that_end_at_their_last_node(ncell, dtype):
    """phi and each gradient plane are followed by other data right after their
    last node: wide loads at the grid's last cells hang over it."""
    import torch
    dim = len(ncell)
    print(f"case {ncell} {dtype}", flush=True)
    rng = np.random.default_rng(dim)
    n = int(np.prod([c + 1 for c in ncell]))
    phi0, psi0 = rng.normal(size=n), rng.normal(size=dim * n)
    lo, hi = (0.0,) * dim, (1.0,) * dim
    kind, params = (pkg.VORTEX, np.zeros(0)) if dim == 2 else (pkg.LEVEQUE3D, np.zeros(0))
    dt = 0.4 / max(ncell)
    g = pkg.Grid(ncell, dtype=dtype)
    g.set_velocity(kind, params, 1.7)
    full = g.from_numpy(phi0, psi0)
    span = g.plane - g.pitch + g.nodes[0]
    flat = torch.full((4 * g.plane + 64 * dim,), float("nan"), dtype=full.dtype, device=full.device)
    st = flat[: (1 + dim) * g.plane].view(1 + dim, g.plane)
    st[0, :span] = full[0, :span]
    for a in range(dim):
        st[1 + a, :span] = full[1 + a, :span]
    pts = np.clip(rng.uniform(0.6, 1.05, size=(400, dim)), 0.0, 1.0)
    val, nrm, cur = g.eval_points(st, pts)
    for k in range(2):
        g.advance(st, 0.1 + k * dt, dt, 1)
    torch.cuda.synchronize()
    for a in range(1 + dim):
        assert torch.isnan(st[a, span:]).all()
    po, so = oracle.advance(dim, ncell, lo, hi, kind, params, 1.7, phi0, psi0, 0.1, dt, 1)
    po, so = oracle.advance(dim, ncell, lo, hi, kind, params, 1.7, po, so, 0.1 + dt, dt, 1)
    p, s = g.to_numpy(st)
    ov = oracle.eval_points(dim, ncell, lo, hi, phi0, psi0, pts)["val"]
    hmin = 1.0 / max(ncell)
    val = val.double().cpu().numpy()
    if dtype == "float64":
        assert rel(p, po) <= TOL64
        assert rel_psi(s, so, po, hmin) <= TOL64
        assert rel(val, ov) <= TOL64
    else:
        tp, ts = fp32_tolerances(po, so, hmin, 2)
        assert rel(p, po) <= tp
        assert rel(s, so) <= ts
        assert rel(val, ov) <= 64 * U32
