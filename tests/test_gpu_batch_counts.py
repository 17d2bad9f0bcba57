"""Batches of every number of problems at which the search for a workgroup's own problem changes (one
line of first workgroups, looked at in two parts) or a batch is cut into two launches; each problem has
parameters of its own and spans several workgroups, so that a wrong choice shows."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_gelu, lib_softmax

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers", [1, 2, 4, 5, 13, 14, 15, 16, 17])
def test_layers_take_their_own_parameters(layers):
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng([37, layers])
    n = 9 * 4096 + 5                                  # nine workgroups, the first of them with the last bytes too
    x = rng.integers(-128, 128, size=(layers, n), dtype=np.int8)
    gp = [prepare.gelu_prepare(2.0 ** -(4 + l % 5), 2.0 ** -(5 + l % 3), 0, l, l % 2) for l in range(layers)]
    d_x, d_y = torch.from_numpy(x).cuda(), torch.full(x.shape, 0x5A, dtype=torch.int8, device="cuda")
    ip.gelu_i8_layers(d_x, n, d_y, n, n, layers, [lib_gelu(q) for q in gp])
    y = d_y.cpu().numpy()
    for l in range(layers):
        assert np.array_equal(y[l], ref.gelu_i8(x[l], gp[l])), l
    for rows, cols in ((291, 49), (1165, 23), (291, 50)):    # a compiled row length; one and two lanes per row
        s = np.rint(rng.standard_normal((layers, rows, cols)) * 900).astype(np.int32)
        sp = [prepare.softmax_prepare(2.0 ** (-5 - 0.25 * l), cols, l % 2) for l in range(layers)]
        want = [ref.softmax_i32(s[l], sp[l]) for l in range(layers)]
        d_s = torch.from_numpy(s).cuda()
        # (a single call of so few rows, and the one that seventeen leave, goes to one wavefront per row by
        # itself: the slab kernel of one problem only where it is asked for)
        for algo in (ip.ALGO_AUTO, ip.ALGO_SLAB):
            d_p = torch.full(s.shape, 0x5A, dtype=torch.uint8, device="cuda")
            ip.softmax_i32_layers(d_s, rows * cols, d_p, rows * cols, rows, cols, layers, [lib_softmax(q, algo) for q in sp])
            got = d_p.cpu().numpy()
            for l in range(layers):
                assert np.array_equal(got[l], want[l]), (cols, l, algo)


@pytest.mark.parametrize("problems", [1, 4, 5, 14, 15, 16])
@pytest.mark.parametrize("cols", [49, 144, 36])          # two compiled window sizes and a run-time one
@pytest.mark.parametrize("form", ["table", "int32 mask", "packed mask"])
def test_problems_take_their_own_tables(problems, cols, form):
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng([53, problems, cols, len(form)])
    windows, heads = 2, 3
    kept, batch, want = [], [], []
    for i in range(problems):
        rows = windows * heads * cols + 3 * i            # each ends at another place of its tables
        x = np.rint(rng.standard_normal((rows, cols)) * 900).astype(np.int32)
        bias = np.rint(rng.standard_normal((heads * cols, cols)) * 90).astype(np.int32)
        p = prepare.softmax_prepare(2.0 ** (-5 - 0.25 * (i % 8)), cols, i % 2)
        mask = None
        d_x, d_b, d_y = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda(), torch.full(x.shape, 0x5A, dtype=torch.uint8, device="cuda")
        d_m = d_bits = None
        if form != "table":
            mask = np.where(rng.random((windows, cols, cols)) < 0.3, -2 ** 31, 0).astype(np.int32)
            d_m = torch.from_numpy(mask).cuda()
            if form == "packed mask":
                d_bits = torch.empty((windows, cols, (cols + 63) // 64), dtype=torch.int64, device="cuda")
                ip.pack_window_mask(d_m, windows, cols, d_bits)
                d_m = None
        batch.append(ip.softmax_problem(d_x, d_b, heads * cols, d_y, rows, cols, lib_softmax(p, ip.ALGO_SLAB), d_m,
                                        windows if mask is not None else 0, heads if mask is not None else 0, d_bits))
        kept.append((d_x, d_b, d_y, d_m, d_bits))
        want.append(ref.softmax_i32(x, p, bias, heads * cols) if mask is None
                    else ref.softmax_i32_windowed(x, p, bias, heads * cols, mask, heads))
    ip.softmax_i32_batch(batch, problems, cols)
    for i in range(problems):
        assert np.array_equal(kept[i][2].cpu().numpy(), want[i]), i
