"""The adjoint's workspace holds what the sweep uses: the advance's workspace, the
states of a segment after its checkpoint, one adjoint state and the partial sums."""
import ctypes

import pytest

import paper_0905_3409_amd as pkg


@pytest.mark.parametrize("prec,es", [(pkg.F32, 4), (pkg.F64, 8)])
@pytest.mark.parametrize("ncell", [(2, 2), (63, 64), (300, 171)])
def test_bytes(prec, es, ncell):
    L = pkg.lib()
    ctx = ctypes.c_void_p()
    d = ctypes.c_double * 2
    pkg.check(L.gals_create(ctypes.byref(ctx), 2, (ctypes.c_int64 * 2)(*ncell), d(0, 0), d(1, 1),
                            prec, 0, 0, -1))
    plane, ws = ctypes.c_int64(), ctypes.c_size_t()
    pkg.check(L.gals_layout(ctx, None, None, ctypes.byref(plane)))
    pkg.check(L.gals_workspace_bytes(ctx, ctypes.byref(ws)))
    up = lambda b: (b + 255) // 256 * 256
    tiles = (ncell[0] // 64 + 1) * (ncell[1] // 4 + 1)
    rest = up(ws.value) + up(3 * plane.value * 8) + up(16 * 8 * ((tiles + 7) // 8 * 8))
    for every in (1, 2, 7):
        b = ctypes.c_size_t()
        pkg.check(L.gals_adjoint_workspace_bytes(ctx, every, ctypes.byref(b)))
        assert b.value == rest + (every - 1) * up(3 * plane.value * es)
    L.gals_destroy(ctx)
