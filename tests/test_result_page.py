"""Host side of the reductions that synchronise, on the CPU against a HIP runtime
that runs nothing (host/fake_hip.c): where their results go and what is allocated
when. Each test is a process of its own, as the page belongs to the process."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.path.insert(0, %r)
fake = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_0905_3409_amd as pkg
L = pkg.lib()
knob = lambda name, t=ctypes.c_int: t.in_dll(fake, "fake_" + name)
ctx = ctypes.c_void_p()
nc = (ctypes.c_int64 * 2)(8, 8)
pkg.check(L.gals_create(ctypes.byref(ctx), 2, nc, (ctypes.c_double * 2)(0, 0),
                        (ctypes.c_double * 2)(1, 1), pkg.F64, 0, 0, 0))
n = ctypes.c_size_t()
pkg.check(L.gals_workspace_bytes(ctx, ctypes.byref(n)))
raw = np.zeros(n.value + 256, dtype=np.uint8)
ws = raw.ctypes.data + (-raw.ctypes.data) %% 256
pkg.check(L.gals_set_velocity(ctx, pkg.VORTEX, None, 0, 0.0))

def speed(value):
    knob("value", ctypes.c_double).value = value
    out = ctypes.c_double(-1.0)
    rc = L.gals_max_speed(ctx, 0.0, ctypes.byref(out), ws, n.value, None)
    return rc, out.value, ctypes.c_void_p.in_dll(fake, "fake_out").value

in_ws = lambda p: ws <= p < ws + n.value
mallocs, copies = knob("mallocs", ctypes.c_long), knob("copies", ctypes.c_long)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "host", "fake_hip.c")], check=True)
    return so


def _run(fake, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE % (ROOT, fake) + body], capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_creating_a_context_touches_no_device(fake):
    _run(fake, """
assert mallocs.value == 0 and knob("set_device", ctypes.c_long).value == 0
""")


def test_results_come_through_one_page(fake):
    _run(fake, """
for k in range(100):
    rc, v, where = speed(3.5 + k)
    assert (rc, v) == (pkg.OK, 3.5 + k) and not in_ws(where)
assert mallocs.value == 1 and copies.value == 0
""")


def test_without_a_page_the_workspace_serves_and_the_page_is_asked_for_again(fake):
    _run(fake, """
knob("malloc_fails").value = 1
for k in range(3):
    rc, v, where = speed(3.5 + k)
    assert (rc, v) == (pkg.OK, 3.5 + k) and in_ws(where)
assert copies.value == 3
knob("malloc_fails").value = 0
rc, v, where = speed(9.0)
assert (rc, v) == (pkg.OK, 9.0) and not in_ws(where) and copies.value == 3
""")


def test_a_slot_whose_wait_failed_is_not_used_again(fake):
    _run(fake, """
knob("sync_fails").value = 1
lost = set()
for k in range(70):
    rc, v, where = speed(3.5)
    assert rc == pkg.EHIP and where not in lost
    if in_ws(where):
        break
    assert v == -1.0
    lost.add(where)
assert len(lost) == 64  # then every slot is lost, and the workspace serves
knob("sync_fails").value = 0
for p in lost:  # the kernels of the failed calls write at last
    ctypes.memmove(p, np.full(8, -7.0).ctypes.data, 64)
for k in range(3):
    rc, v, where = speed(4.0 + k)
    assert (rc, v) == (pkg.OK, 4.0 + k) and in_ws(where)
""")
