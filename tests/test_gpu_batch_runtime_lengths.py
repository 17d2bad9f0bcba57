"""Several problems of one run-time row length in one launch: each must equal the oracle, with guard
bytes around every output, whatever else is in the batch.  Row lengths are the edges of the lane
layouts (1 to 16 lanes per row, the fewest and the most blocks); 16 problems are more than one launch
of that kernel holds."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_softmax

pytestmark = pytest.mark.gpu
INT32_MIN = -(2 ** 31)


@pytest.mark.parametrize("cols", [1, 4, 29, 30, 61, 62, 145, 196, 253, 254, 401, 512, 635])
@pytest.mark.parametrize("n_problems", [2, 16])
def test_batch_of_run_time_row_lengths(cols, n_problems):
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng([31, cols, n_problems])
    specs = []
    for i in range(n_problems):
        rows = int(rng.integers(1, 300))
        x = np.rint(rng.standard_normal((rows, cols)) * float(rng.choice([200, 3000]))).astype(np.int32)
        if i % 4 == 1:
            x[0, :] = INT32_MIN                                   # a fully masked row
            x[-1, -1] = INT32_MIN + 1                             # and a row close to INT32_MIN
        p = prepare.softmax_prepare(float(2.0 ** rng.uniform(-10, -4)), cols, i % 3, int(i % 5 == 0))
        if i == 3:
            p.post = ref.Dyadic(3, 1, 7, 0, 255) if not p.out_is_signed else ref.Dyadic(3, 1, 7, -128, 127)
        if i == 4:
            p.pre_m, p.pre_s = 20000, 21                          # a launch of its own
        if i == 6:
            p = ref.SoftmaxParams(variant=1, i0=2 ** 14, n_shift=0, out_is_signed=0)   # 32-bit arithmetic
        bias, period = None, 0
        if i % 3 == 2:
            period = 96 + i
            bias = np.rint(rng.standard_normal((period, cols)) * 50).astype(np.int32)
        specs.append((x, p, bias, period, i % 4))
    probs, keep = [], []
    for x, p, bias, period, off in specs:
        larger = torch.zeros(x.size + 8, dtype=torch.int32, device="cuda")
        larger[off:off + x.size] = torch.from_numpy(x.reshape(-1)).cuda()
        guarded = torch.full((x.size + 64,), 0x5A, dtype=torch.int8 if p.out_is_signed else torch.uint8, device="cuda")
        d_x, d_y = larger[off:off + x.size], guarded[32 + off:32 + off + x.size]
        d_b = None if bias is None else torch.from_numpy(bias).cuda()
        keep.append((larger, guarded, d_x, d_y, d_b))
        probs.append(ip.softmax_problem(d_x, d_b, period, d_y, x.shape[0], cols, lib_softmax(p)))
    ip.softmax_i32_batch(probs, n_problems, cols)
    torch.cuda.synchronize()
    for (x, p, bias, period, off), (_, guarded, _, d_y, _) in zip(specs, keep):
        assert np.array_equal(d_y.cpu().numpy().reshape(x.shape), ref.softmax_i32(x, p, bias, period))
        g = guarded.cpu().numpy()
        assert (g[:32 + off] == 0x5A).all() and (g[32 + off + x.size:] == 0x5A).all()


def test_problems_that_share_memory_keep_their_order():
    """Two problems into one output: the bytes are those of the second, as one call after the other
    leaves them."""
    import torch
    import paper_2511_15369_amd as ip
    rng = np.random.default_rng(7)
    x = np.rint(rng.standard_normal((9000, 145)) * 900).astype(np.int32)
    p0, p1 = prepare.softmax_prepare(2.0 ** -9, 145, 1, 0), prepare.softmax_prepare(2.0 ** -5, 145, 0, 0)
    d_x, d_y = torch.from_numpy(x).cuda(), torch.full(x.shape, 0x5A, dtype=torch.uint8, device="cuda")
    probs = [ip.softmax_problem(d_x, None, 0, d_y, len(x), 145, lib_softmax(p)) for p in (p0, p1)]
    ip.softmax_i32_batch(probs, 2, 145)
    assert np.array_equal(d_y.cpu().numpy(), ref.softmax_i32(x, p1))
