"""Row counts that are no multiple of a slab's rows: the last slab starts earlier and makes some rows a
second time, from any row of its tables and masks.  Every remainder of the widest slab, and calls with fewer
rows than a slab, in the compiled and the run-time row lengths; tables that end inside a chunk of four
scores; guard bytes around every output."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_softmax

pytestmark = pytest.mark.gpu
INT32_MIN = -(2 ** 31)


def _run(x, p, bias, period, off, call=None):
    import torch
    import paper_2511_15369_amd as ip
    rows, cols = x.shape
    larger = torch.zeros(x.size + 8, dtype=torch.int32, device="cuda")
    larger[off:off + x.size] = torch.from_numpy(x.reshape(-1)).cuda()
    guarded = torch.full((x.size + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    d_y = guarded[32 + off:32 + off + x.size]
    d_b = None if bias is None else torch.from_numpy(bias).cuda()
    d_x, q = larger[off:off + x.size], lib_softmax(p, ip.ALGO_SLAB)
    if call is None:
        ip.softmax_i32(d_x, d_b, period, d_y, rows, cols, q)
    else:
        call(ip, d_x, d_b, d_y, q)
    g = guarded.cpu().numpy()
    assert (g[:32 + off] == 0x5A).all() and (g[32 + off + x.size:] == 0x5A).all()
    return g[32 + off:32 + off + x.size].reshape(rows, cols)


# lanes per row 2, 4, 4, 8, 8, 16 (compiled), then 1, 1, 2, 4, 8, 16
@pytest.mark.parametrize("cols", [49, 144, 197, 198, 257, 577, 7, 29, 36, 81, 145, 401])
def test_every_remainder(cols):
    rng = np.random.default_rng([41, cols])
    p = prepare.softmax_prepare(0.011, cols, cols % 2, 0)
    for r, rows in enumerate([1, 3, 5, 63] + list(range(64, 64 + (64 if cols < 100 else 17)))):
        x = np.rint(rng.standard_normal((rows, cols)) * 700).astype(np.int32)
        period = (0, 64, 65, 71, 130)[r % 5]          # with none; cols * period a multiple of four or not
        bias = np.rint(rng.standard_normal((period, cols)) * 90).astype(np.int32) if period else None
        if r % 7 == 3:
            x[-1, :] = INT32_MIN
            if period:
                bias[:, 1] = INT32_MIN
        assert np.array_equal(_run(x, p, bias, period, r % 4), ref.softmax_i32(x, p, bias, period)), (rows, period)


@pytest.mark.parametrize("cols", [49, 144, 36, 64, 81, 169])
@pytest.mark.parametrize("packed", [False, True])
def test_masks_beside_a_moved_slab(cols, packed):
    import torch
    rng = np.random.default_rng([43, cols, packed])
    windows, heads = 3, 2
    mask = np.where(rng.random((windows, cols, cols)) < 0.3, INT32_MIN, 0).astype(np.int32)
    mask[1] = 0
    bias = np.rint(rng.standard_normal((heads * cols, cols)) * 90).astype(np.int32)
    p = prepare.softmax_prepare(0.011, cols, 1, 0)
    d_m = torch.from_numpy(mask).cuda()
    for rows in (windows * heads * cols - 1, windows * heads * cols + 2, 5 * cols + 3, 65, 5):
        x = np.rint(rng.standard_normal((rows, cols)) * 700).astype(np.int32)

        def call(ip, d_x, d_b, d_y, q):
            if packed:
                bits = torch.empty((windows, cols, (cols + 63) // 64), dtype=torch.int64, device="cuda")
                ip.pack_window_mask(d_m, windows, cols, bits)
                ip.softmax_i32_windowed_bits(d_x, d_b, heads * cols, bits, windows, heads, d_y, rows, cols, q)
            else:
                ip.softmax_i32_windowed(d_x, d_b, heads * cols, d_m, windows, heads, d_y, rows, cols, q)

        got = _run(x, p, bias, heads * cols, rows % 4, call)
        assert np.array_equal(got, ref.softmax_i32_windowed(x, p, bias, heads * cols, mask, heads)), rows
