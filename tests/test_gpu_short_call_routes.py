"""Short calls of run-time row lengths near the rows at which the choice between the slab kernel, one wavefront
per row and the three-pass kernel changes: whole and ragged row counts, views off the 16-byte grid, tables that
one wavefront per row does not take; single calls and pairs.  (tests/test_dispatch.py: which kernel each takes.)"""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_softmax

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols,variant,period", [(9, 2, 0), (25, 1, 40), (25, 1, 41), (29, 2, 40), (64, 2, 0), (81, 2, 100), (128, 2, 0),
                                                 (196, 2, 77), (225, 2, 0), (256, 2, 0)])
def test_unmasked(cols, variant, period):
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng([59, cols, period])
    p = prepare.softmax_prepare(0.011, cols, variant, 0)
    q = lib_softmax(p)
    bias = np.rint(rng.standard_normal((period, cols)) * 90).astype(np.int32) if period else None
    d_b = None if bias is None else torch.from_numpy(bias).cuda()
    for rows in (600, 3073, 3586, 4611, 6147, 7168, 8192, 8195):
        n = rows * cols
        x = np.rint(rng.standard_normal((rows, cols)) * 700).astype(np.int32)
        want = ref.softmax_i32(x, p, bias, period)
        for off in (0, 1 + rows % 3):
            larger = torch.zeros(n + 4, dtype=torch.int32, device="cuda")
            larger[off:off + n] = torch.from_numpy(x.reshape(-1)).cuda()
            d_x, d_y = larger[off:off + n], torch.full((2, n), 0x5A, dtype=torch.uint8, device="cuda")
            ip.softmax_i32(d_x, d_b, period, d_y[0], rows, cols, q)
            assert np.array_equal(d_y[0].cpu().numpy().reshape(rows, cols), want), (rows, off)
            ip.softmax_i32_batch([ip.softmax_problem(d_x, d_b, period, d_y[i], rows, cols, q) for i in range(2)], 2, cols)
            assert all(np.array_equal(y.reshape(rows, cols), want) for y in d_y.cpu().numpy()), (rows, off)


@pytest.mark.parametrize("cols", [9, 29, 64, 81, 121, 196, 256])
@pytest.mark.parametrize("packed,table", [(False, True), (False, False), (True, True), (True, False)])
def test_masked(cols, packed, table):
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng([61, cols, packed, table])
    windows, heads = 3, 2
    mask = np.where(rng.random((windows, cols, cols)) < 0.3, -2 ** 31, 0).astype(np.int32)
    mask[1] = 0
    period = heads * cols if table else 0
    bias = np.rint(rng.standard_normal((period, cols)) * 90).astype(np.int32) if table else None
    d_b, d_m = None if bias is None else torch.from_numpy(bias).cuda(), torch.from_numpy(mask).cuda()
    bits = torch.empty((windows, cols, (cols + 63) // 64), dtype=torch.int64, device="cuda")
    ip.pack_window_mask(d_m, windows, cols, bits)
    p = prepare.softmax_prepare(0.011, cols, 1 + cols % 2, 0)
    q = lib_softmax(p)
    for rows in (258, 259, 704, 3075, 4611, 7169, 8192, 8193):
        x = np.rint(rng.standard_normal((rows, cols)) * 700).astype(np.int32)
        d_x, d_y = torch.from_numpy(x).cuda(), torch.full(x.shape, 0x5A, dtype=torch.uint8, device="cuda")
        if packed:
            ip.softmax_i32_windowed_bits(d_x, d_b, period, bits, windows, heads, d_y, rows, cols, q)
        else:
            ip.softmax_i32_windowed(d_x, d_b, period, d_m, windows, heads, d_y, rows, cols, q)
        assert np.array_equal(d_y.cpu().numpy(), ref.softmax_i32_windowed(x, p, bias, period, mask, heads)), rows
