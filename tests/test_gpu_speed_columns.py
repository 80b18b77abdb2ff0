"""The largest speed of a sine stream function on grids of a few columns: node by
node below twelve of them, in tiles from there on, both against the oracle."""
import numpy as np
import pytest

import oracle
import paper_0905_3409_amd as pkg
from gpu_util import U32
from paper_0905_3409_amd import inputs

pytestmark = pytest.mark.gpu

PARAMS = np.array([0.05, 1, 3, -0.03, 4, 2, 0.02, 2, 2, 0.01, 3, 4])


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("ncell", [(2, 3000), (10, 70), (11, 70), (12, 63)])
def test_few_columns(ncell, dtype):
    g = pkg.Grid(ncell, (-0.1, 0.05), (1.1, 0.95), dtype=dtype)
    g.set_velocity(inputs.STREAM_SIN, PARAMS, 2.0)
    print(f"case {ncell} {dtype}", flush=True)
    o = oracle.max_speed(2, ncell, (-0.1, 0.05), (1.1, 0.95), inputs.STREAM_SIN, PARAMS, 2.0, 0.3)
    # FP32: FP32 angles (up to 4.4 pi) and sums of four modes
    assert abs(g.max_speed(0.3) - o) <= (1e-13 if dtype == "float64" else 64 * U32) * o
