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


# lanes per row 2, 4, 8, 8, 8, 16 (compiled; 197 and 198 have four in the longest launches, below), then 1, 1, 2, 4,
# 8, 16
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


@pytest.mark.parametrize("cols", [7, 29])
def test_table_that_wraps_twice(cols):
    """One lane per row: 64 rows per slab, tables of 32 rows and more."""
    rng = np.random.default_rng([47, cols])
    p = prepare.softmax_prepare(0.011, cols, 1, 0)
    for period in (32, 33, 50, 63):
        bias = np.rint(rng.standard_normal((period, cols)) * 90).astype(np.int32)
        for rows in list(range(64, 129, 3)) + [1000, 1001, 1002, 1003]:
            x = np.rint(rng.standard_normal((rows, cols)) * 700).astype(np.int32)
            assert np.array_equal(_run(x, p, bias, period, rows % 4), ref.softmax_i32(x, p, bias, period)), (rows, period)


@pytest.mark.parametrize("cols", [197, 198])
def test_four_lanes_per_row_beside_a_table(cols):
    """Launches of more than 90 million scores: 16 rows per slab, a ragged row count, and a table that ends inside a
    chunk of four; the same bytes as short launches give, and the oracle's on the rows that are made twice."""
    import torch
    import paper_2511_15369_amd as ip
    period = 67
    rows = 90_000_000 // cols // (16 * period) * 16 * period + 16 * period + 5
    assert rows * cols > 90_000_000 and (period * cols) % 4 != 0
    gen = torch.Generator(device="cuda").manual_seed(cols)
    x = torch.randint(-2000, 2000, (rows, cols), generator=gen, device="cuda", dtype=torch.int32)
    bias = torch.randint(-300, 300, (period, cols), generator=gen, device="cuda", dtype=torch.int32)
    p = prepare.softmax_prepare(0.011, cols, 1, 0)
    q = lib_softmax(p)
    guarded = torch.full((rows * cols + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    whole, parts = guarded[32:32 + rows * cols].view(rows, cols), torch.empty((rows, cols), dtype=torch.uint8, device="cuda")
    ip.softmax_i32(x, bias, period, whole, rows, cols, q)
    step = period * 512
    for r in range(0, rows, step):
        n = min(step, rows - r)
        ip.softmax_i32(x[r:r + n], bias, period, parts[r:r + n], n, cols, q)
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)
    assert bool((guarded[:32] == 0x5A).all()) and bool((guarded[-32:] == 0x5A).all())
    last, h_bias = rows - rows % period - period, bias.cpu().numpy()      # a multiple of the period
    assert last <= rows - 32
    assert np.array_equal(whole[last:].cpu().numpy(), ref.softmax_i32(x[last:].cpu().numpy(), p, h_bias, period))
