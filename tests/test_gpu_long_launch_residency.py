"""Launches of more than 50 (75, 90, 110, 120, 150) million scores, where the kernels ask for LDS to bound the
workgroups that share a compute unit: the same bytes as the rows give in short launches (unbounded),
and the oracle's on the first and the last row.  (tests/test_dispatch.py: that these launches are bounded.)"""
import numpy as np
import pytest

import paper_2511_15369_amd as ip
from oracle import ref
from tests.helpers import lib_softmax

pytestmark = pytest.mark.gpu


# one row length for each bound: slabs of 4 and 16 lanes per row; 4, 6, 10, 14, 15 and 16 passes of a
# wavefront; 6, 8, 9 and 10 of four, 8 of eight
LONGEST = {197: 120, 198: 90, 401: 110, 600: 110, 8192: 75, 9300: 110, 16000: 150}


@pytest.mark.parametrize("cols", [197, 198, 401, 600, 900, 1000, 1500, 2500, 3400, 3600, 4093, 6001, 8150, 8192, 9000, 9300, 16000])
def test_long_launch_equals_short_ones(cols):
    import torch
    rows = LONGEST.get(cols, 60) * 1_000_000 // cols + 3
    gen = torch.Generator(device="cuda").manual_seed(cols)
    x = torch.randint(-9000, 9000, (rows, cols), generator=gen, device="cuda", dtype=torch.int32)
    p = ref.SoftmaxParams(variant=1, i0=117, n_shift=8, m_bits=31)
    lp = lib_softmax(p)
    whole = torch.empty((rows, cols), dtype=torch.uint8, device="cuda")
    parts = torch.empty_like(whole)
    ip.softmax_i32(x, None, 0, whole, rows, cols, lp)
    step = rows // 8 // 4 * 4                      # parts start on the 16-byte grid, as the whole does
    for r in range(0, rows, step):
        n = min(step, rows - r)
        ip.softmax_i32(x[r:r + n], None, 0, parts[r:r + n], n, cols, lp)
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)
    for r in (0, rows - 1):
        want = ref.softmax_i32(x[r:r + 1].cpu().numpy(), p)
        assert np.array_equal(whole[r:r + 1].cpu().numpy(), want.reshape(1, cols))
