"""An additive table beside rows of 7 to 16 passes of a wavefront and of 7 to 13 of a workgroup of 8, at the
first and the last row length of each number of passes (a different number of table loads in flight
each), against the oracle: saturating sums, masked entries, a table shorter and longer than the call."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_softmax

pytestmark = pytest.mark.gpu
I32_MIN = -(2 ** 31)
LENGTHS = [n for p in range(7, 17) for n in (256 * (p - 1) + 1, 256 * p)] + [13317] + [n for p in range(7, 14) for n in (2048 * (p - 1) + 1, 2048 * p)][1:]


@pytest.mark.parametrize("cols", LENGTHS)
def test_table_beside_long_rows(cols):
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng(cols)
    for variant, rows, period, pre in ((1, 9, 4, False), (0, 5, 8, True), (2, 9, 4, False)):
        p = prepare.softmax_prepare(float(2.0 ** rng.uniform(-9, -5)), cols, variant)
        if pre:
            p.pre_m, p.pre_s = 20000, 21
        unit = p.i0 * (100 if pre else 1)
        x = np.rint(rng.standard_normal((rows, cols)) * 2 * unit).astype(np.int32)
        bias = np.rint(rng.standard_normal((period, cols)) * unit).astype(np.int32)
        for a in (x, bias):
            a[rng.random(a.shape) < 0.02] = I32_MIN
        x[1, ::3], bias[1, ::3] = 2 ** 31 - 5, 2 ** 31 - 3 * unit           # sums beyond the largest integer
        x[3, : cols // 2] = I32_MIN + 7                                     # and below the smallest
        for algo in (ip.ALGO_AUTO, ip.ALGO_WIDE):
            d_y = torch.full((rows, cols), 0x5A, dtype=torch.uint8, device="cuda")
            ip.softmax_i32(torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda(), period, d_y, rows, cols, lib_softmax(p, algo))
            assert np.array_equal(d_y.cpu().numpy(), ref.softmax_i32(x, p, bias, period)), (variant, algo)
