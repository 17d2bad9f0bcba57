"""Rows of up to 65536 scores (one walking workgroup per row, the next row fetched while this one is
computed) against the oracle: every pass count at its edges, one and several rows per workgroup,
partly filled last passes, tensors off the 16-byte grid, rows near INT32_MIN in between ordinary
ones, tables and the requantization in front, 32-bit and packed arithmetic, guard bytes."""
import numpy as np
import pytest

import paper_2511_15369_amd as ip
from oracle import prepare, ref
from tests.helpers import lib_softmax

pytestmark = pytest.mark.gpu
I32_MIN = -(2 ** 31)
PASS = 4096                                                 # scores per pass of the workgroup


def _check(x, p, bias, period, off, ooff):
    import torch
    rows, cols = x.shape
    want = ref.softmax_i32(x, p, bias, period).view(np.uint8).reshape(-1)
    n = rows * cols
    d_in = torch.zeros(n + 8, dtype=torch.int32, device="cuda")
    d_in[off:off + n] = torch.from_numpy(x.reshape(-1)).cuda()
    d_bias = None if bias is None else torch.from_numpy(bias).cuda()
    for algo in (0, 3):
        d_out = torch.full((n + 32,), 0x5A, dtype=torch.uint8, device="cuda")
        view = d_out.view(torch.int8) if p.out_is_signed else d_out
        ip.softmax_i32(d_in[off:off + n], d_bias, period, view[ooff:ooff + n], rows, cols, lib_softmax(p, algo))
        torch.cuda.synchronize()
        got = d_out.cpu().numpy()
        assert np.array_equal(got[ooff:ooff + n], want), algo
        assert (got[:ooff] == 0x5A).all() and (got[ooff + n:] == 0x5A).all()


def _scores(rng, rows, cols, i0):
    x = np.rint(rng.standard_normal((rows, cols)) * 2.0 * i0).astype(np.int64)
    x[rng.random(x.shape) < 0.01] = I32_MIN
    x[min(1, rows - 1), : cols // 2] = I32_MIN
    if rows > 2:
        x[2] = I32_MIN                                      # fully masked
        x[rows - 1] = I32_MIN + rng.integers(0, 2 * i0, size=cols)     # the clamp cannot separate masked scores here
    return x.astype(np.int32)


@pytest.mark.parametrize("slots", range(7, 17))
@pytest.mark.parametrize("edge", [-3, 0, 1, 6])
def test_pass_counts(slots, edge):
    cols = min(slots * PASS + edge, 65536)
    rng = np.random.default_rng(slots * 10 + edge)
    for variant, s_delta, signed, off in ((1, 2.0 ** -8.5, 0, 0), (0, 2.0 ** -5, 1, 3), (2, 2.0 ** -13, 0, 1)):
        p = prepare.softmax_prepare(s_delta, cols, variant, signed)
        rows = int(rng.integers(1, 6))
        _check(_scores(rng, rows, cols, p.i0), p, None, 0, off, int(rng.integers(0, 17)))


@pytest.mark.parametrize("cols", [26620, 32768, 40001, 53249, 65536])
def test_several_rows_per_workgroup(cols):
    """More rows than workgroups: the prefetch of the next row, the last row ending off the grid."""
    import torch
    rng = np.random.default_rng(cols)
    p = prepare.softmax_prepare(2.0 ** -7.5, cols, 1)
    few = _scores(rng, 7, cols, p.i0)
    want_few = torch.from_numpy(ref.softmax_i32(few, p)).cuda()
    rows = 599                                              # not a multiple of the grid or of 7
    which = torch.arange(rows, device="cuda") % 7
    x = torch.from_numpy(few).cuda()[which].contiguous()
    out = torch.full((rows, cols), 0x5A, dtype=torch.uint8, device="cuda")
    ip.softmax_i32(x, None, 0, out, rows, cols, lib_softmax(p))
    torch.cuda.synchronize()
    assert torch.equal(out, want_few[which])


@pytest.mark.parametrize("cols", [26624, 45056, 65536])
def test_tables_requantization_and_post_steps(cols):
    rng = np.random.default_rng(cols + 1)
    for variant, s_delta, pre, post in ((1, 2.0 ** -6, (20000, 20), None), (0, 2.0 ** -9, (1, 0), (3, 2, 5)), (2, 2.0 ** -12, (300, 9), (1, 0, -128))):
        signed = 1 if post == (1, 0, -128) else 0
        p = prepare.softmax_prepare(s_delta, cols, variant, signed)
        p.pre_m, p.pre_s = pre
        if post is not None:
            p.post = ref.Dyadic(post[0], post[1], post[2], -128 if signed else 0, 127 if signed else 255)
        x = _scores(rng, 5, cols, p.i0 * (1 << pre[1]) // pre[0])
        bias = np.rint(rng.standard_normal((2, cols)) * 3 * p.i0).astype(np.int32)
        bias[rng.random(bias.shape) < 0.01] = I32_MIN
        _check(x, p, None, 0, 2, 1)
        _check(x, p, bias, 2, 0, 5)
