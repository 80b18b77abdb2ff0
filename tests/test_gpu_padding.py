"""What the library copies of a state: the nodes of every row and nothing else. The
padding of the caller's planes is marked, and so is the copy's: the mark of the
copy has to stay."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from paper_0905_3409_amd import inputs

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
