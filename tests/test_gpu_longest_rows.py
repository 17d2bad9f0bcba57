"""Rows of up to 65536 scores (a workgroup of 16 wavefronts per row, up to 40957 scores for some calls,
else workgroups that walk over rows and fetch the next one while one is computed) against the oracle:
every pass count at its edges, one and several rows per workgroup, partly filled last passes, tensors
off the 16-byte grid, rows near INT32_MIN in between ordinary ones, tables and the requantization in
front, 32-bit and packed arithmetic, guard bytes, more than 2^31 scores."""
import ctypes

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


@pytest.mark.parametrize("cols", [26620, 26625, 32768, 40001, 53249, 65536])
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


def _packed(p):
    fn = ip.load().iptq_debug_softmax_packed
    fn.argtypes = [ctypes.POINTER(ip.SoftmaxParams), ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]
    packed, div8 = ctypes.c_int32(-1), ctypes.c_int32()
    lp = lib_softmax(p)
    assert fn(ctypes.byref(lp), ctypes.byref(packed), ctypes.byref(div8)) == 0
    return packed.value


# five rows for most workgroups, and more than a requantization in front leaves to a workgroup per row
WALKED_ROWS = 1200
WALKS = [
    # variant, scale, packed arithmetic (0 none, 1 multiply-high divider, 2 byte divider), requantization in
    # front, post step, table: each arithmetic with and without either of the last two, in every variant
    (0, 2.0 ** -7, 2, (1, 0), None, False),
    (1, 2.0 ** -13, 0, (1, 0), None, False),
    (1, 2.0 ** -6, 2, (1, 0), (3, 2, 5), False),
    (2, 2.0 ** -6, 2, (1, 0), (1, 0, -128), False),
    (1, 2.0 ** -6, 2, (20000, 20), None, False),
    (0, 2.0 ** -13, 0, (300, 9), (3, 2, 5), False),
    (2, 2.0 ** -6, 2, (1, 0), None, True),
    (1, 2.0 ** -6, 2, (1, 0), (3, 2, 5), True),
    (0, 2.0 ** -13, 0, (20000, 20), None, True),
    (2, 2.0 ** -12, 0, (300, 9), (1, 0, -128), True),
    (0, 2.0 ** -13, 0, (1, 0), None, False),
    (2, 2.0 ** -13, 0, (1, 0), None, False),
    (1, 2.0 ** -13, 0, (300, 9), None, True),
    (0, 2.0 ** -6, 2, (1, 0), (3, 2, 5), True),
    (0, 1 / 2000.5, 1, (1, 0), None, False),
    (1, 1 / 2896.5, 1, (1, 0), (3, 2, 5), False),
    (2, 1 / 3139.5, 1, (1, 0), (1, 0, -128), False),
    (0, 1 / 2896.5, 1, (20000, 16), None, False),
    (1, 1 / 2000.5, 1, (1, 0), None, True),
    (2, 1 / 2000.5, 1, (20000, 16), (3, 2, 5), True),
]


@pytest.mark.parametrize("cols", [26625, 28672, 33001, 36864, 36866, 40957, 41000, 53251, 65533])
@pytest.mark.parametrize("walk", range(len(WALKS)))
def test_every_kernel_walks(cols, walk):
    """Several rows per workgroup in every instantiation (three arithmetics, three variants, with and without
    a table or a requantization): the prefetch of the next row beside them, every post step, 7 passes to 16,
    either side of the 9 passes that LDS holds and 10 of the workgroup per row, tensors that start and end
    off the grid."""
    import torch
    variant, s_delta, packed, pre, post, table = WALKS[walk]
    signed = 1 if post == (1, 0, -128) else 0
    rng = np.random.default_rng(cols * 10 + walk)
    p = prepare.softmax_prepare(s_delta, cols, variant, signed)
    p.pre_m, p.pre_s = pre
    if post is not None:
        p.post = ref.Dyadic(post[0], post[1], post[2], -128 if signed else 0, 127 if signed else 255)
    assert _packed(p) == packed
    unit = p.i0 * (1 << pre[1]) // pre[0]
    few = _scores(rng, 28, cols, unit)                                # a multiple of four: the table's size too
    few[4:26:2] = _scores(rng, 15, cols, 4 * unit)[3:14]              # rows with large probabilities
    bias, period, off = None, 0, (cols + walk) % 4
    if table:                                                         # needs both tensors on the grid
        period, off = 28, 0
        bias = np.rint(rng.standard_normal((period, cols)) * 3 * p.i0).astype(np.int32)
        bias[rng.random(bias.shape) < 0.01] = I32_MIN
    want_few = torch.from_numpy(ref.softmax_i32(few, p, bias, period).view(np.uint8)).cuda()
    rows, n = WALKED_ROWS, WALKED_ROWS * cols
    which = torch.arange(rows, device="cuda") % 28
    d_in = torch.zeros(n + 4, dtype=torch.int32, device="cuda")
    d_in[off:off + n].view(rows, cols)[:] = torch.from_numpy(few).cuda()[which]
    d_bias = None if bias is None else torch.from_numpy(bias).cuda()
    d_out = torch.full((n + 16,), 0x5A, dtype=torch.uint8, device="cuda")
    ooff = walk % 3
    view = d_out.view(torch.int8) if signed else d_out
    print("walk", walk, "of", rows, "x", cols, "at", off, flush=True)
    ip.softmax_i32(d_in[off:off + n], d_bias, period, view[ooff:ooff + n], rows, cols, lib_softmax(p))
    torch.cuda.synchronize()
    assert torch.equal(d_out[ooff:ooff + n].view(rows, cols), want_few[which])
    assert bool((d_out[:ooff] == 0x5A).all()) and bool((d_out[ooff + n:] == 0x5A).all())


@pytest.mark.parametrize("cols", [20001, 50177])
def test_more_than_2_31_scores(cols):
    """64-bit element offsets in the workgroup-per-row kernels, row by row and walking."""
    import torch
    rng = np.random.default_rng(cols)
    p = prepare.softmax_prepare(2.0 ** -7.4, cols, 1)
    few = _scores(rng, 7, cols, p.i0)
    want_few = torch.from_numpy(ref.softmax_i32(few, p)).cuda()
    rows = 2 ** 31 // cols + 300
    which = torch.arange(rows, device="cuda") % 7
    print("softmax of", rows, "x", cols, flush=True)
    x = torch.from_numpy(few).cuda()[which]
    out = torch.full((rows, cols), 0x5A, dtype=torch.uint8, device="cuda")
    ip.softmax_i32(x, None, 0, out, rows, cols, lib_softmax(p))
    torch.cuda.synchronize()
    del x
    for lo in range(0, rows, 8192):
        assert torch.equal(out[lo:lo + 8192], want_few[which[lo:lo + 8192]]), lo
