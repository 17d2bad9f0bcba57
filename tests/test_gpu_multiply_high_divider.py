"""The packed arithmetic's multiply-high divider (i0 of about 1070 to 3270, scales below 2^-10, which the
other tests' scales do not reach) in every family of kernels: each against the oracle, and, on the recording
runtime, that the calls do reach those instantiations."""
import numpy as np
import pytest

import paper_2511_15369_amd as ip
from oracle import ref
from tests import host_library
from tests.helpers import lib_softmax

I32_MIN = -(2 ** 31)
I0 = (1100, 2000, 2896, 3139)
# rows, row length, kernel, table beside the scores, algorithm
CASES = [
    (331, 49, "softmax_rows_kernel", "", ip.ALGO_SLAB), (331, 197, "softmax_rows_kernel", "", ip.ALGO_SLAB),
    (331, 198, "softmax_rows_kernel", "bias", ip.ALGO_SLAB), (331, 257, "softmax_rows_kernel", "bias", ip.ALGO_SLAB),
    (331, 577, "softmax_rows_kernel", "", ip.ALGO_SLAB), (331, 144, "softmax_rows_kernel", "bias", ip.ALGO_SLAB),
    (457_000, 197, "softmax_rows_kernel", "", ip.ALGO_AUTO), (455_003, 198, "softmax_rows_kernel", "", ip.ALGO_AUTO),
    (588, 49, "softmax_rows_masked_kernel", "int32", ip.ALGO_SLAB), (864, 144, "softmax_rows_masked_kernel", "int32", ip.ALGO_SLAB),
    (588, 49, "softmax_rows_maskbits_kernel", "bits", ip.ALGO_SLAB), (864, 144, "softmax_rows_maskbits_kernel", "bits", ip.ALGO_SLAB),
    (331, 5, "softmax_rowsdyn_kernel", "", ip.ALGO_SLAB), (331, 29, "softmax_rowsdyn_kernel", "bias", ip.ALGO_SLAB),
    (331, 61, "softmax_rowsdyn_kernel", "", ip.ALGO_SLAB), (331, 100, "softmax_rowsdyn_kernel", "", ip.ALGO_SLAB),
    (331, 196, "softmax_rowsdyn_kernel", "bias", ip.ALGO_SLAB), (331, 401, "softmax_rowsdyn_kernel", "", ip.ALGO_SLAB),
    (331, 635, "softmax_rowsdyn_kernel", "", ip.ALGO_SLAB), (768, 64, "softmax_rowsdyn_kernel", "int32", ip.ALGO_SLAB),
    (486, 81, "softmax_rowsdyn_kernel", "bits", ip.ALGO_SLAB),
    (61, 197, "softmax_wide_kernel", "", ip.ALGO_WIDE), (61, 700, "softmax_wide_kernel", "", ip.ALGO_WIDE),
    (61, 1025, "softmax_wide_kernel", "", ip.ALGO_WIDE), (60, 2048, "softmax_wide_kernel", "bias", ip.ALGO_WIDE),
    (61, 2049, "softmax_wide_kernel", "", ip.ALGO_WIDE), (61, 3073, "softmax_wide_kernel", "", ip.ALGO_WIDE),
    (61, 4093, "softmax_wide_kernel", "", ip.ALGO_WIDE),
    (21, 4097, "softmax_wgrow_kernel", "", ip.ALGO_AUTO), (21, 8192, "softmax_wgrow_kernel", "", ip.ALGO_AUTO),
    (20, 12288, "softmax_wgrow_kernel", "bias", ip.ALGO_AUTO), (21, 13313, "softmax_wgrow_kernel", "", ip.ALGO_AUTO),
    (21, 20481, "softmax_wgrow_kernel", "", ip.ALGO_AUTO), (21, 26621, "softmax_wgrow_kernel", "", ip.ALGO_AUTO),
    (21, 30001, "softmax_wgrow_kernel", "", ip.ALGO_AUTO), (20, 40960, "softmax_wgrow_kernel", "bias", ip.ALGO_AUTO),
    (21, 41001, "softmax_long_kernel", "", ip.ALGO_AUTO), (20, 65536, "softmax_long_kernel", "bias", ip.ALGO_AUTO),
]
MODE_AT = dict(softmax_rows_kernel=2, softmax_rows_masked_kernel=2, softmax_rows_maskbits_kernel=2, softmax_rows_requant_kernel=2,
               softmax_rowsdyn_kernel=2, softmax_wide_kernel=1, softmax_wgrow_kernel=2, softmax_long_kernel=1)
WINDOWS, HEADS = 3, 2


def _params(case, variant, pre):
    """i0 by turns; scores in front of the requantization are 3.3 times as large."""
    rows, cols = case[:2]
    i0 = I0[(rows + cols + variant) % len(I0)] if cols < 40000 else 2000
    n = 15 - i0.bit_length()
    while cols * (i0 << n) > 1 << 30:
        n -= 1
    post = (ref.Dyadic(1, 0, 0, 0, 255), ref.Dyadic(1, 0, 0, 0, 127), ref.Dyadic(3, 1, 5, 0, 255))[(rows + variant + pre) % 3]
    return ref.SoftmaxParams(variant=variant, i0=i0, n_shift=n, pre_m=20000 if pre else 1, pre_s=16 if pre else 0, post=post)


def _combinations():
    for case in CASES:
        for variant in (0, 1, 2):
            if not (case[2] == "softmax_wgrow_kernel" and case[1] > 26624 and variant == 2):   # (first degree only)
                yield case, variant, False
        yield case, 1, True


def test_the_calls_reach_those_kernels(recording_library):
    so = recording_library
    seen, folded = set(), set()
    for case, variant, pre in _combinations():
        rows, cols, kernel, table, algo = case
        q = ip.SoftmaxProblem(d_scores=1 << 40, d_out=1 << 44, rows=rows, params=lib_softmax(_params(case, variant, pre), algo))
        if table:
            q.d_bias, q.bias_period_rows = 1 << 36, HEADS * cols if table in ("int32", "bits") else 64
        if table == "int32":
            q.d_mask, q.n_windows, q.heads = 1 << 38, WINDOWS, HEADS
        if table == "bits":
            q.d_mask_bits, q.n_windows, q.heads = 1 << 38, WINDOWS, HEADS
        got = host_library.launches(so, lambda: so.iptq_softmax_i32_batch((ip.SoftmaxProblem * 1)(q), 1, cols, None))
        assert len(got) == 1, (case, got)
        name = got[0].kernel
        assert name in (kernel, "softmax_rows_requant_kernel") and got[0].arguments[MODE_AT[name]] == 1, (case, variant, pre, got)
        seen.add((name, got[0].arguments))
        if pre and (name == "softmax_rows_requant_kernel" or got[0].arguments[-1] == "true"):
            folded.add(name)
    # the requantization folded into the exponential too, and more and fewer lanes per row at 197 and 198
    assert folded >= {"softmax_rows_requant_kernel", "softmax_rowsdyn_kernel", "softmax_wide_kernel"}
    lanes = {a[:2] for n, a in seen if n == "softmax_rows_kernel"}
    assert lanes >= {(197, 4), (197, 8), (198, 4), (198, 8), (49, 2), (144, 4), (257, 8), (577, 16)}
    assert {a[0] for n, a in seen if n == "softmax_wgrow_kernel"} == {4, 8, 16}


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d-%s" % (c[0], c[1], c[3]))
def test_multiply_high_divider(case):
    import torch
    rows, cols, _, table, algo = case
    rng = np.random.default_rng([rows, cols])
    few = rows if rows < 1000 else 331                      # the rest are copies of these
    for c, variant, pre in _combinations():
        if c is not case:
            continue
        p = _params(case, variant, pre)
        unit = p.i0 * (3.3 if pre else 1)
        x = np.rint(rng.standard_normal((few, cols)) * rng.choice([0.5, 2.0, 6.0], (few, 1)) * unit).astype(np.int32)
        x[rng.random(x.shape) < 0.01] = I32_MIN
        x[1] = I32_MIN
        x[2] = I32_MIN + rng.integers(0, int(2 * unit), cols)
        bias, period, mask = None, 0, None
        if table:
            period = HEADS * cols if table in ("int32", "bits") else 64
            bias = np.rint(rng.standard_normal((period, cols)) * unit / 4).astype(np.int32)
        if table in ("int32", "bits"):
            mask = np.where(rng.random((WINDOWS, cols, cols)) < 0.3, I32_MIN, 0).astype(np.int32)
            mask[1] = 0
            want = ref.softmax_i32_windowed(x, p, bias, period, mask, HEADS)
        else:
            want = ref.softmax_i32(x, p, bias, period)
        which = torch.arange(rows, device="cuda") % few
        d_x = torch.from_numpy(x).cuda()[which]
        d_y = torch.full((rows, cols), 0x5A, dtype=torch.uint8, device="cuda")
        d_b = None if bias is None else torch.from_numpy(bias).cuda()
        lp = lib_softmax(p, algo)
        if mask is None:
            ip.softmax_i32(d_x, d_b, period, d_y, rows, cols, lp)
        else:
            d_m = torch.from_numpy(mask).cuda()
            if table == "int32":
                ip.softmax_i32_windowed(d_x, d_b, period, d_m, WINDOWS, HEADS, d_y, rows, cols, lp)
            else:
                bits = torch.empty((WINDOWS, cols, (cols + 63) // 64), dtype=torch.int64, device="cuda")
                ip.pack_window_mask(d_m, WINDOWS, cols, bits)
                ip.softmax_i32_windowed_bits(d_x, d_b, period, bits, WINDOWS, HEADS, d_y, rows, cols, lp)
        torch.cuda.synchronize()
        assert torch.equal(d_y, torch.from_numpy(np.ascontiguousarray(want)).cuda().view(torch.uint8).reshape(few, cols)[which]), (variant, pre)


@pytest.mark.gpu
@pytest.mark.parametrize("cols", [49, 197])
def test_batch_with_both_dividers(cols):
    """Problems of either divider in turn, one of them in 32-bit arithmetic: every one its own bytes."""
    import torch
    rng = np.random.default_rng(cols)
    probs, keep = [], []
    for i in range(16):
        i0 = (100, 1100, 2000)[i % 3] if i != 7 else 2 ** 14
        p = ref.SoftmaxParams(variant=i % 3, i0=i0, n_shift=max(0, 15 - i0.bit_length()))
        x = np.rint(rng.standard_normal((60 + i, cols)) * 2 * i0).astype(np.int32)
        d_x, d_y = torch.from_numpy(x).cuda(), torch.full(x.shape, 0x5A, dtype=torch.uint8, device="cuda")
        keep.append((x, p, d_x, d_y))
        probs.append(ip.softmax_problem(d_x, None, 0, d_y, len(x), cols, lib_softmax(p)))
    ip.softmax_i32_batch(probs, 16, cols)
    for x, p, _, d_y in keep:
        assert np.array_equal(d_y.cpu().numpy(), ref.softmax_i32(x, p))
