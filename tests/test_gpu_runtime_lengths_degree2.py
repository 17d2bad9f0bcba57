"""The second-degree exponential (variant 2) in the kernels with a run-time row length, against the
oracle: every kernel family at the edges of its lane layouts, 32-bit and packed arithmetic, rows
near INT32_MIN, masked scores, an additive table, and calls of few rows."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import gpu_softmax

pytestmark = pytest.mark.gpu
I32_MIN = -(2 ** 31)


@pytest.mark.parametrize("cols", [1, 3, 29, 30, 50, 61, 64, 125, 196, 250, 401, 635, 640, 1024, 4095, 4097, 13307, 26619])
@pytest.mark.parametrize("s_delta", [2.0 ** -4, 2.0 ** -8.3, 2.0 ** -14])
def test_degree2_matches_the_oracle(cols, s_delta):
    rng = np.random.default_rng(cols)
    rows = 4001 if cols <= 64 else (3100 if cols <= 256 else max(3, 40000 // cols))   # few and many rows
    p = prepare.softmax_prepare(s_delta, cols, 2, int(cols % 2))
    x = np.rint(rng.standard_normal((rows, cols)) * 3.0 * p.i0).astype(np.int64)
    x[rng.random(x.shape) < 0.03] = I32_MIN
    x[0] = I32_MIN                                          # fully masked
    if rows > 2:
        x[1] = I32_MIN + rng.integers(0, 2 * p.i0, size=cols)   # the clamp cannot separate masked scores here
    x = x.astype(np.int32)
    for period in (0, 64):
        bias = None if period == 0 else np.rint(rng.standard_normal((period, cols)) * p.i0).astype(np.int32)
        want = ref.softmax_i32(x, p, bias, period)
        for algo in (0, 2, 3, 4):
            assert np.array_equal(gpu_softmax(x, p, bias, period, algo=algo), want), (period, algo)
