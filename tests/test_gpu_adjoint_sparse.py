"""Adjoint steps with lambda zero on most of the grid, whose waves and blocks
without a nonzero entry are skipped: linearity against dense lambda, the
multi-step sweep, and data that are not finite where lambda is zero."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu


def _setup(dtype, ncell, seed):
    rng = np.random.default_rng(seed)
    g = pkg.Grid(ncell, dtype=dtype)
    g.set_velocity(pkg.STREAM_SIN, inputs.stream_modes(rng, 8, ncell, 1.5), 1.3)
    n = g.num_nodes
    return rng, g, g.from_numpy(rng.normal(size=n), rng.normal(size=2 * n))


def _lam(g, rng, nodes):
    """lambda with random values at `nodes` (all three fields), +0 elsewhere."""
    import torch
    lam = g.empty_adjoint().zero_()
    for j, i in nodes:
        for a in range(3):
            g._grid_view(lam[a])[j, i] = float(rng.normal())
    return lam


# Two adjoints of sums and the sum of two adjoints differ by the order of FP64
# additions; FP32 rounds the seeds of a node's parameter derivative to FP32
# (relative u), which is not linear.
TOL = {"float64": (1e-13, 1e-12), "float32": (1e-13, 8 * 2.0 ** -24)}


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("ncell,dt", [((200, 90), 0.004), ((600, 260), 0.002), ((63, 3), 0.01),
                                      ((150, 140), 0.08)])
def test_sparse_lambda_adds_up(dtype, ncell, dt):
    import torch
    rng, g, st = _setup(dtype, ncell, 5)
    nx, ny = ncell
    nodes = [(0, 0), (ny, nx), (ny // 2, nx // 3), (0, nx), (ny, min(64, nx)), (ny // 3, 63)]
    sparse = _lam(g, rng, nodes)
    dense = g.empty_adjoint().zero_()
    for a in range(3):
        v = g._grid_view(dense[a])
        v.copy_(torch.from_numpy(rng.normal(size=tuple(v.shape))))
    print(f"case {dtype} {ncell}", flush=True)
    ls, ds = g.adjoint_step(st, 0.2, dt, sparse)
    ld, dd = g.adjoint_step(st, 0.2, dt, dense)
    lb, db = g.adjoint_step(st, 0.2, dt, dense + sparse)
    torch.cuda.synchronize()
    tl, td = TOL[dtype]
    for a in range(3):
        x, y = g._grid_view(ls[a]) + g._grid_view(ld[a]), g._grid_view(lb[a])
        assert float((x - y).abs().max()) <= tl * float(g._grid_view(ld[a]).abs().max() + 1.0)
    # the scale of the sums: |dS| of single nodes adds up without cancelling
    scale = float(dd.abs().max()) + float(ds.abs().max()) + np.sqrt(g.num_nodes) * dt
    assert float((ds + dd - db).abs().max()) <= td * scale
    assert float(ds.abs().max()) > 0.0
    zero, dz = g.adjoint_step(st, 0.2, dt, g.empty_adjoint().zero_())
    torch.cuda.synchronize()
    assert not zero.any() and not dz.any()


@pytest.mark.parametrize("every", [1, 3, 10])
def test_sweep_of_a_sparse_lambda(every):
    """The sweep clears lambda as it goes: it equals single steps in a row."""
    import torch
    rng, g, st = _setup("float64", (300, 170), 6)
    lam = _lam(g, rng, [(80, 100), (170, 300), (20, 250)])
    states, s = [], st.clone()
    for n in range(10):
        states.append(s.clone())
        g.advance(s, n * 0.004, 0.004, 1)
    ref, dref = lam.clone(), 0.0
    for n in reversed(range(10)):
        ref, d = g.adjoint_step(states[n], n * 0.004, 0.004, ref)
        dref = dref + d
    ck = g.advance_save(st.clone(), 0.0, 0.004, 10, every)
    out = lam.clone()
    dS = g.adjoint(ck, 0.0, 0.004, 10, every, out)
    torch.cuda.synchronize()
    for a in range(3):
        x, y = g._grid_view(out[a]), g._grid_view(ref[a])
        assert float((x - y).abs().max()) <= 1e-11 * float(y.abs().max())
    assert float((dS - dref).abs().max()) <= 1e-11 * float(dref.abs().max())


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("plane", [0, 2])
def test_data_that_are_not_finite_reach_the_derivative(bad, dtype, plane):
    import torch
    rng, g, st = _setup(dtype, (300, 170), 7)
    g._grid_view(st[plane])[120, 200] = float(bad)
    lam = _lam(g, rng, [(20, 30)])
    prev, dS = g.adjoint_step(st, 0.2, 0.002, lam)
    torch.cuda.synchronize()
    assert bool(torch.isnan(dS).all())
    assert bool(torch.isfinite(prev).all())
