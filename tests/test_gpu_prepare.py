"""The launch before an advance (the field's tables and, for an odd number of
launches, the state's copy): odd and even step counts against each other on
planes that are 16-byte aligned and planes that are not, and the padding of the
caller's planes left alone."""
import ctypes

import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

CASES = {
    "stream": ((301, 255), inputs.STREAM_SIN, np.array([0.05, 1, 3, -0.03, 4, 2, 0.02, 2, 2])),
    "affine": ((403, 401), inputs.AFFINE, inputs.rotation_params()),
    "pseudo1d": ((63, 5), inputs.PSEUDO1D, np.zeros(0)),
    "vecpot": ((20, 9, 13), inputs.VECPOT_SIN, np.array([0.05, -0.01, 0.02, 1, 3, 2])),
    "leveque": ((140, 129, 119), inputs.LEVEQUE3D, np.zeros(0)),
}


@pytest.mark.parametrize("shift", [0, 1, 3])  # elements past a 256-byte boundary
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_odd_and_even_steps(name, dtype, shift):
    import torch
    ncell, kind, params = CASES[name]
    dim = len(ncell)
    print(f"case {name} {dtype} shift {shift}", flush=True)
    g = pkg.Grid(ncell, dtype=dtype)
    g.set_velocity(kind, params, 2.0)
    rng = np.random.default_rng(dim)
    init = g.from_numpy(rng.normal(size=g.num_nodes), rng.normal(size=dim * g.num_nodes))
    shape = tuple(reversed(g.nodes[1:])) + (g.pitch,)
    pad = torch.full_like(init, float("nan"))
    for a in range(1 + dim):
        pad[a].view(shape)[..., : g.nodes[0]] = init[a].view(shape)[..., : g.nodes[0]]
    dt = 0.002

    def state():
        flat = torch.empty(pad.numel() + 8, dtype=pad.dtype, device=pad.device)
        s = flat[shift: shift + pad.numel()].view_as(pad)
        s.copy_(pad)
        return s

    def advance(s, n0, n):
        ws = g.workspace()
        pkg.check(pkg.lib().gals_advance(
            g._ctx, ctypes.c_void_p(s[0].data_ptr()), ctypes.c_void_p(s[1].data_ptr()), n0 * dt, dt,
            n, ctypes.c_void_p(ws.data_ptr()), ws.numel(),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))

    a, b, c = state(), state(), state()
    advance(a, 0, 4)
    advance(b, 0, 1)
    advance(b, 1, 3)
    for n in range(4):
        advance(c, n, 1)
    torch.cuda.synchronize()
    bits = torch.int64 if dtype == "float64" else torch.int32
    assert torch.isfinite(g._grid_view(a[0])).all()
    assert torch.equal(a.contiguous().view(bits), b.contiguous().view(bits))
    assert torch.equal(a.contiguous().view(bits), c.contiguous().view(bits))
    if g.pitch > g.nodes[0]:
        assert torch.isnan(a[0].view(shape)[..., g.nodes[0]:]).all()
