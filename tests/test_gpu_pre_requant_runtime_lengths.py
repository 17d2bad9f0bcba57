"""The requantization in front, folded into Eq. 6 in the kernels with a run-time row length, against the
oracle: rows near INT32_MIN (where the clamp of the raw differences cannot separate masked scores
from live ones) beside ordinary ones, masked scores, fully masked rows, tables, post steps."""
import numpy as np
import pytest

import paper_2511_15369_amd as ip
from oracle import prepare, ref
from tests.helpers import gpu_softmax

pytestmark = pytest.mark.gpu
I32_MIN = -(2 ** 31)


@pytest.mark.parametrize("cols", [1, 3, 25, 30, 50, 64, 100, 145, 250, 401, 500, 635, 700, 1025, 2040, 2049, 3000])
@pytest.mark.parametrize("pre", [(20000, 21), (32767, 16), (1, 16), (255, 24), (20000, 24), (300, 31)])
def test_folded_requantization_matches_the_oracle(cols, pre):
    rng = np.random.default_rng(cols * 100 + pre[1])
    rows = max(5, min(3600, 60000 // cols))                  # slab and one-wavefront-per-row routes
    for variant, s_delta, post in ((1, 2.0 ** -4, None), (0, 2.0 ** -7.5, (1, 0, -128)), (1, 2.0 ** -9, (3, 2, 5))):
        signed = 1 if post == (1, 0, -128) else 0
        p = prepare.softmax_prepare(s_delta, cols, variant, signed)
        p.pre_m, p.pre_s = pre
        if post is not None:
            p.post = ref.Dyadic(post[0], post[1], post[2], -128 if signed else 0, 127 if signed else 255)
        scale = min(2.0 * p.i0 * 2.0 ** pre[1] / pre[0], 2.0 ** 30)
        x = np.rint(rng.standard_normal((rows, cols)) * scale)
        near = I32_MIN + np.rint(np.abs(rng.standard_normal((rows, cols))) * min(scale, 2.0 ** 28)) + 1
        low = rng.random(rows) < 0.3
        x = np.where(low[:, None], near, x)
        x = np.clip(x, I32_MIN, 2 ** 31 - 1).astype(np.int32)
        x[rng.random(x.shape) < 0.1] = I32_MIN
        x[0] = I32_MIN
        x[1] = 2 ** 31 - 1
        for period in (0, 64):
            bias = None if period == 0 else np.rint(rng.standard_normal((period, cols)) * scale / 4).astype(np.int32)
            want = ref.softmax_i32(x, p, bias, period)
            for algo in (0, 2, 3):
                assert np.array_equal(gpu_softmax(x, p, bias, period, algo=algo), want), (variant, period, algo)
