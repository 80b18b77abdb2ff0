"""Launches of several steps that take fewer than planned (test_multi_regions shows
that these do): the result against calls of one step, bit for bit, for odd and even
counts, and every checkpoint on the way."""
import numpy as np
import pytest

import paper_0905_3409_amd as pkg
from test_multi_regions import SHORT

pytestmark = pytest.mark.gpu


def _grid(dtype):
    g = pkg.Grid(SHORT["ncell"], dtype=dtype)
    g.set_velocity(pkg.AFFINE, SHORT["par"], 1.0)
    rng = np.random.default_rng(3)
    n = g.num_nodes
    return g, g.from_numpy(rng.normal(size=n), rng.normal(size=2 * n))


def _views(g, s):
    import torch
    return torch.stack([g._grid_view(s[q]) for q in range(3)])


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("t0", [0.15, 0.55, 0.75])
def test_against_single_steps(dtype, t0):
    import torch
    g, st = _grid(dtype)
    dt, b = SHORT["dt"], st.clone()
    for steps in range(1, 13):
        g.advance(b, t0 + (steps - 1) * dt, dt, 1)
        a = st.clone()
        g.advance(a, t0, dt, steps)
        torch.cuda.synchronize()
        print(f"case {dtype} t0 {t0} steps {steps}", flush=True)
        assert torch.equal(_views(g, a), _views(g, b))


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("steps,every", [(8, 3), (9, 4), (11, 5), (7, 7), (12, 6)])
def test_checkpoints(dtype, steps, every):
    import torch
    g, st = _grid(dtype)
    dt, t0 = SHORT["dt"], 0.55
    print(f"case {dtype} steps {steps} every {every}", flush=True)
    a = st.clone()
    ck = g.advance_save(a, t0, dt, steps, every)
    sb = g.checkpoint_bytes(1, 1)
    b = st.clone()
    for n in range(steps):
        if n % every == 0:
            k = n // every
            c = ck[k * sb: (k + 1) * sb].view(g.torch_dtype)[: 3 * g.plane].view(3, g.plane)
            assert torch.equal(_views(g, c), _views(g, b)), n
        g.advance(b, t0 + n * dt, dt, 1)
    torch.cuda.synchronize()
    assert torch.equal(_views(g, a), _views(g, b))
