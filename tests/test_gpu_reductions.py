"""The reductions at the edges of their tiles and passes: the largest speed of a
sine stream function (tiles of 256 columns and 32 rows) and the norms (two nodes
a pass of 262144) against plain float64 sums, and results of calls from several
threads at once."""
import threading

import numpy as np
import pytest
import torch  # before the library: both load the HIP runtime

import oracle
import paper_0905_3409_amd as pkg
from gpu_util import U32
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

PARAMS = np.array([0.05, 1, 3, -0.03, 4, 2, 0.02, 2, 2, 0.01, 3, 4])


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("ncell", [(2, 2), (254, 30), (255, 31), (256, 32), (700, 3), (3, 1100)])
def test_max_speed_of_a_stream_function(ncell, dtype):
    g = pkg.Grid(ncell, (-0.1, 0.05), (1.1, 0.95), dtype=dtype)
    g.set_velocity(inputs.STREAM_SIN, PARAMS, 2.0)
    print(f"case {ncell} {dtype}", flush=True)
    o = oracle.max_speed(2, ncell, (-0.1, 0.05), (1.1, 0.95), inputs.STREAM_SIN, PARAMS, 2.0, 0.3)
    # FP32: the angles are FP32 (relative u of up to 4.4 pi) and a sum of four
    # modes rounds a few times
    tol = 1e-13 if dtype == "float64" else 64 * U32
    assert abs(g.max_speed(0.3) - o) <= tol * o


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("ncell", [(2, 2), (511, 511), (512, 510), (1023, 511), (70, 61, 59),
                                   (90, 83, 71)])
def test_norms_over_whole_and_part_passes(ncell, dtype):
    dim = len(ncell)
    g = pkg.Grid(ncell, dtype=dtype)
    rng = np.random.default_rng(sum(ncell))
    n = g.num_nodes
    a = g.from_numpy(rng.normal(size=n), rng.normal(size=dim * n))
    b = g.from_numpy(rng.normal(size=n), rng.normal(size=dim * n))
    (pa, ga), (pb, gb) = g.to_numpy(a), g.to_numpy(b)
    eps, band = 0.4, 0.2
    print(f"case {ncell} {dtype}", flush=True)
    r = g.norms(a, b, eps, band)

    def H(s):
        z = np.clip(s / eps, -1.0, 1.0)
        return 0.5 * (1.0 + z + np.sin(np.pi * z) / np.pi)
    vol = float(np.prod([1.0 / c for c in ncell]))
    e = np.abs(pa - pb)
    want = [e.max(), np.abs(ga - gb).max(), vol * np.abs(H(pa) - H(pb)).sum(),
            e[np.abs(pb) <= band].max(initial=0.0), vol * H(-pa).sum(), vol * H(-pb).sum(), 0.0,
            np.abs(pb).max()]
    # maxima of the same float64 differences are exact; sums of n <= 5e5 terms
    for k in (0, 1, 3, 6, 7):
        assert r[k] == want[k]
    for k in (2, 4, 5):
        assert abs(r[k] - want[k]) <= 1e-12 * max(want[k], 1e-3)


def test_results_of_concurrent_calls():
    fields = [PARAMS * s for s in np.linspace(0.5, 2.0, 8)]
    grids, want = [], []
    for q, p in enumerate(fields):
        p = p.copy()
        p[1::3], p[2::3] = PARAMS[1::3], PARAMS[2::3]
        g = pkg.Grid((100 + q, 90), dtype="float64")
        g.set_velocity(inputs.STREAM_SIN, p, 0.0)
        g.workspace()
        grids.append(g)
        want.append(g.max_speed(0.0))
    torch.cuda.synchronize()
    bad = []

    def work(q):
        s = torch.cuda.Stream()
        for _ in range(30):
            if grids[q].max_speed(0.0, stream=s) != want[q]:
                bad.append(q)
    ts = [threading.Thread(target=work, args=(q,)) for q in range(len(grids))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
