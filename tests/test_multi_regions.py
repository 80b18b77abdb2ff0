"""Regions of the several-steps kernel, on the CPU: its plan and the device functions
of its nodes' feet are compiled for the host, and the stencil of every foot has to
lie in the region that its block stages, whatever the field, the grid and the
numbers (overflow and not-a-number included)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_0905_3409_amd as pkg

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_0905_3409_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("probe") / "region_probe.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-x", "hip", "-O2",
                    "-march=x86-64-v3", "-std=c++17", "-ffp-contract=on", "-fPIC", "-shared",
                    "-I" + CSRC, "-o", so, os.path.join(HERE, "host", "region_probe.hip")],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.probe.restype = ctypes.c_long
    D = ctypes.c_double

    def call(f32, affine, ncell, par, dt, period=0.0, t0=0.0, bc=pkg.BC_NEUMANN, lo=(0.0, 0.0),
             hi=(1.0, 1.0)):
        par = np.ascontiguousarray(par, dtype=np.float64).ravel()
        k = ctypes.c_int()
        bad = lib.probe(int(f32), int(affine), bc, (ctypes.c_long * 2)(*ncell), (D * 2)(*lo),
                        (D * 2)(*hi), par.ctypes.data_as(ctypes.c_void_p), D(period), D(t0), D(dt),
                        ctypes.byref(k))
        return bad, k.value
    return call


AFF = [0.2, -0.1, 0.45, 0.55]


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("bc", [pkg.BC_NEUMANN, pkg.BC_EXTRAPOLATE])
def test_ordinary_fields(probe, f32, bc):
    rng = np.random.default_rng(1)
    several = 0
    for _ in range(150):
        ncell = [int(v) for v in np.exp(rng.uniform(np.log(2), np.log(200), 2))]
        dt = float(np.exp(rng.uniform(np.log(1e-3), np.log(3.0)))) / max(ncell)
        period, t0 = float(rng.choice([0.0, 0.7])), float(rng.uniform(0, 2))
        lo = rng.uniform(-1, 0, 2)
        hi = lo + rng.uniform(0.3, 3, 2)
        for affine, par in ((1, AFF + list(rng.normal(size=4) * 3)), (0, rng.normal(size=16) * 0.1)):
            bad, k = probe(f32, affine, ncell, par, dt, period, t0, bc, lo, hi)
            assert bad == 0, (affine, ncell, par, dt, period, t0, lo, hi)
            several += k > 1
    assert several > 100


@pytest.mark.parametrize("f32", [False, True])
def test_feet_across_long_thin_grids(probe, f32):
    """A displacement of n cells rounds by up to n 2^-24 cells in FP32."""
    rng = np.random.default_rng(2)
    for nx in (100, 5000, 8192, 8193, 20000, 26000, 40000):
        for _ in range(6):
            shift = rng.uniform(0.2, 0.9) + rng.uniform(-1, 1) * 1e-5  # of the domain, a step
            bad, k = probe(f32, 1, (nx, 2), [shift, 0.0, 0, 0, 0, 0, 0, 0], 1.0)
            assert bad == 0, (nx, shift, k)
            # feet at whole cells, up to the rounding
            cells = round(shift * nx)
            for eps in (-1.9e-3, -1e-3, -1e-9, 0.0, 1e-9, 1e-3, 1.9e-3):
                bad, k = probe(f32, 1, (nx, 2), [(cells + eps) / nx, 0, 0, 0, 0, 0, 0, 0], 1.0)
                assert bad == 0, (nx, cells, eps, k)


@pytest.mark.parametrize("f32", [False, True])
def test_numbers_out_of_range(probe, f32):
    for big in (1e30, 1e38, 1e39, 1e200, 1.7e308):
        for ncell in ((40, 30), (200, 2)):
            for dt in (1.0, 1e-3, 1.0 / big, 1e-300, 1e300):
                for par in ([big, 0, 0, 0, 0, 0, 0, 0], [big, big, 0, 0, 0, 1, -1, 0],
                            [0, 0, 0, 0, big, 0, 0, -big], [0, 0, big, -big, 0, 1, -1, 0],
                            [-big, big, big, big, big, -big, big, big]):
                    bad, k = probe(f32, 1, ncell, par, dt)
                    assert bad == 0, (ncell, dt, par, k)
                S = np.zeros(16)
                for s in (big, -big, 1.0 / big):
                    S[5], S[2] = s, s
                    bad, k = probe(f32, 0, ncell, S, dt)
                    assert bad == 0, (ncell, dt, s, k)


SHORT = dict(ncell=(200, 200), par=[0, 0, 0.5, 0.5, 7, 0, 0, 7], dt=0.1)


@pytest.mark.parametrize("f32", [False, True])
def test_a_launch_takes_fewer_steps_than_planned(probe, f32):
    """The case of test_gpu_multi_short: a contracting field that expands when its
    time factor changes sign."""
    assert probe(f32, 1, SHORT["ncell"], SHORT["par"], SHORT["dt"])[1] == 4
    taken = {probe(f32, 1, SHORT["ncell"], SHORT["par"], SHORT["dt"], 1.0, 0.55 + 0.1 * n)[1]
             for n in range(8)}
    print("steps taken", taken)
    assert min(taken) < 4
