"""The dispatch of calls and batches to kernels, on the recording runtime (no GPU)."""
import ctypes
import os
import shutil
import subprocess
import sys

import pytest

import paper_2511_15369_amd as ip
from tests import host_library

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")
SCORES, OUT = 1 << 40, 1 << 44                            # addresses that nothing follows


@pytest.fixture
def lib(recording_library):
    return recording_library


def problems(specs, cols):
    """specs: [(rows, params, optional dict of fields)] -> array of problems, each with memory of its own."""
    arr = (ip.SoftmaxProblem * len(specs))()
    for i, (rows, params, *fields) in enumerate(specs):
        q = arr[i]
        q.d_scores, q.d_out, q.rows, q.params = SCORES + (i << 34), OUT + (i << 32), rows, params
        for k, v in (fields[0] if fields else {}).items():
            setattr(q, k, v)
    return arr


def batch(so, specs, cols):
    arr = problems(specs, cols)
    return host_library.launches(so, lambda: so.iptq_softmax_i32_batch(arr, len(specs), cols, None))


def test_batch_without_a_layout_goes_to_the_next_kernel(tmp_path):
    """A full batch of the run-time-row-length kernel whose launcher holds no such layout: every call is
    served by the next kernel, and nothing is written past the batch (the library traps on that)."""
    code = """
import re, sys, paper_2511_15369_amd as ip
from paper_2511_15369_amd import build
from tests import host_library, test_dispatch as t
text = open(build.CSRC + "/softmax_rowsdyn_k8.hip").read()
so = host_library.build(sys.argv[1], {"softmax_rowsdyn_k8.hip": re.sub(r"IPTQ_ROWSDYN_CASE\\(.*\\)", "", text)})
got = t.batch(so, [(4000, ip.softmax_prepare(0.01, 145, 1, 0))] * 16, 145)
assert len(got) == 16 and {l.kernel for l in got} == {"softmax_wide_kernel"}, got
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    subprocess.run([sys.executable, "-c", code, str(tmp_path)], cwd=root, check=True)


def test_batch_of_dependent_problems_keeps_its_order(lib):
    """Problems that write what another one reads or writes: one launch each, in their order.  Problems
    that only read the same memory share a launch."""
    p = ip.softmax_prepare(0.01, 145, 1, 0)
    n = 4000 * 145

    def starts(*fields, cols=145):
        got = batch(lib, [(4000, p, f) for f in fields], cols)
        return [l.kernel for l in got], [l.first_word for l in got]

    one_launch = (["softmax_rowsdyn_batch_kernel"], [2])
    apart = ["softmax_rowsdyn_kernel"] * 2
    shared = SCORES + (1 << 30)
    assert starts({}, {}) == one_launch
    assert starts(dict(d_scores=SCORES), dict(d_scores=SCORES)) == one_launch
    assert starts(dict(d_bias=shared, bias_period_rows=64), dict(d_bias=shared, bias_period_rows=64)) == one_launch
    assert starts(dict(d_out=OUT), dict(d_out=OUT + n)) == one_launch                  # side by side
    for fields in ((dict(d_out=OUT), dict(d_out=OUT)),                                 # the last one wins
                   (dict(d_out=OUT), dict(d_out=OUT + n - 1)),
                   (dict(d_scores=SCORES, d_out=OUT), dict(d_scores=SCORES + (1 << 35), d_out=SCORES + 4 * n - 1)),
                   (dict(d_out=SCORES + (1 << 35) + 4 * n - 1), dict(d_scores=SCORES + (1 << 35))),
                   (dict(d_out=shared), dict(d_bias=shared, bias_period_rows=64)),
                   (dict(d_bias=shared, bias_period_rows=64), dict(d_out=shared + 4 * 64 * 145 - 1))):
        kernels, words = starts(*fields)
        assert kernels == apart, fields
        first = [f.get("d_scores", SCORES + (i << 34)) & 0xffffffff for i, f in enumerate(fields)]
        assert words == first                                                          # the first argument: d_scores
    # beside a call that the batch kernel does not take (a window mask), and one of its own output
    assert starts({}, dict(d_mask=shared, n_windows=2, heads=1), dict(d_out=OUT))[0] == ["softmax_rowsdyn_kernel"] * 3
    assert starts({}, dict(d_mask=shared, n_windows=2, heads=1), dict(d_out=shared))[0] == ["softmax_rowsdyn_kernel"] * 3
    assert starts({}, dict(d_mask=shared, n_windows=2, heads=1), {})[0] == ["softmax_rowsdyn_batch_kernel", "softmax_rowsdyn_kernel"]


def packed_softmax(i0, cols, variant=1):
    """Parameters with that i0: packed arithmetic with the byte divider (i0 up to about 1050), with the
    multiply-high divider (to about 3270), or none."""
    p = ip.softmax_prepare(0.01, cols, variant, 0)
    p.i0, p.n_shift = i0, max(0, 15 - i0.bit_length())
    return p


@pytest.mark.parametrize("order", [(100, 1100), (1100, 100), (1100, 1100, 100, 100, 2000)])
def test_batch_with_both_dividers(lib, order):
    """Layers of a compiled row length whose scales lie on both sides of the byte divider's range: one
    launch for each divider, in whatever order they come."""
    specs = [(4000, packed_softmax(order[i % len(order)], 197)) for i in range(16)]
    got = batch(lib, specs, 197)
    high = sum(q.i0 > 1050 for _, q in specs)
    assert sorted((l.kernel, l.arguments[2], l.problems) for l in got) == [
        ("softmax_rows_kernel", 1, high), ("softmax_rows_kernel", 2, 16 - high)]
    # one launch where each can have the multiply-high divider
    wide = [(4000, packed_softmax(max(q.i0, 257 + i), 197)) for i, (_, q) in enumerate(specs)]
    assert [l.arguments[2] for l in batch(lib, wide, 197)] == [1]
    assert [l.arguments[2] for l in batch(lib, [w for w in wide if w[1].i0 < 1000], 197)] == [2]
    # a layer in 32-bit arithmetic ends the launches in front of it, as it always did
    specs[8] = (4000, packed_softmax(2 ** 14, 197))
    got = batch(lib, specs, 197)
    assert [l.arguments[2] for l in got] == [2, 1, 0, 2, 1] and sum(l.problems for l in got) == 16


def test_two_short_calls_share_a_launch(lib):
    """Two short calls of the second degree or with a short table, which one by one go to one wavefront per
    row: a second launch costs more than that chain is shorter."""
    table = dict(d_bias=SCORES + (1 << 30), bias_period_rows=40)

    def kernels(n, rows, cols, variant, fields, algo=0):
        p = ip.softmax_prepare(0.0085, cols, variant, 0)
        p.algo = algo
        return [l.kernel for l in batch(lib, [(rows, p, fields)] * n, cols)]

    together = ["softmax_rowsdyn_batch_kernel"]
    for args in ((600, 25, 1, table), (1000, 29, 2, table), (600, 64, 2, {}),
                 (64, 25, 1, table), (4000, 25, 1, table), (600, 16, 1, table), (600, 25, 1, {}), (600, 64, 1, {}), (600, 145, 2, {}),
                 (600, 25, 1, dict(table, bias_period_rows=64))):
        assert args[0] > 3072 or kernels(1, *args) == ["softmax_wide_kernel"], args
        assert kernels(2, *args) == kernels(3, *args) == kernels(2, *args, algo=ip.ALGO_DYNAMIC) == together, args


@pytest.mark.parametrize("cols,variant,fields,other", [
    (100, 1, dict(d_bias=SCORES + (1 << 30), bias_period_rows=200, d_mask=SCORES + (1 << 31), n_windows=4, heads=2), "softmax_generic_kernel"),
    (81, 1, dict(d_mask=SCORES + (1 << 31), n_windows=4, heads=2), "softmax_generic_kernel"),
    (121, 1, dict(d_bias=SCORES + (1 << 30), bias_period_rows=242, d_mask_bits=SCORES + (1 << 31), n_windows=4, heads=2), "softmax_generic_kernel"),
    (29, 2, dict(d_mask_bits=SCORES + (1 << 31), n_windows=4, heads=2), "softmax_generic_kernel"),
    (64, 2, {}, "softmax_wide_kernel"), (225, 2, {}, "softmax_wide_kernel"), (9, 2, {}, "softmax_wide_kernel"),
    (81, 2, dict(d_bias=SCORES + (1 << 30), bias_period_rows=100), "softmax_wide_kernel"),
    (25, 1, dict(d_bias=SCORES + (1 << 30), bias_period_rows=40), "softmax_wide_kernel"),
    (25, 1, dict(d_bias=SCORES + (1 << 30), bias_period_rows=41), "softmax_generic_kernel"),      # not a multiple of four scores
    (25, 2, dict(d_bias=SCORES + (1 << 30) + 4, bias_period_rows=40), "softmax_generic_kernel")])  # off the 16-byte grid
def test_ragged_short_calls_are_chosen_like_whole_ones(lib, cols, variant, fields, other):
    """A short call leaves the run-time-row-length slab kernel up to some number of rows and stays from there
    on, whatever the row count is a multiple of."""
    p = ip.softmax_prepare(0.0085, cols, variant, 0)
    seen = []
    for rows in range(600, 9300, 61):
        got = [l.kernel for l in batch(lib, [(rows, p, fields)], cols)]
        assert got in ([other], ["softmax_rowsdyn_kernel"]), (rows, got)
        seen.append(got[0] == other)
    assert seen == sorted(seen, reverse=True) and seen[0] and not seen[-1]


@pytest.mark.parametrize("rows,cols,most", [
    # one wavefront per row: the fewest and the most passes with each bound, and the lines between
    (50_000_000 // 816 + 1, 816, 0), (50_000_000 // 820 + 1, 820, 6), (50_000_000 // 948 + 1, 948, 6), (50_000_000 // 952 + 1, 952, 5),
    (50_000_000 // 949 + 1, 949, 0), (50_000_000 // 950 + 1, 950, 6), (50_000_000 // 952, 952, 0),
    (50_000_000 // 1500 + 1, 1500, 4), (28_000_000 // 1500 + 1, 1500, 5), (28_000_000 // 1500, 1500, 0), (50_000_000 // 2500 + 1, 2500, 4),
    (50_000_000 // 3330 + 1, 3330, 3), (50_000_000 // 3756 + 1, 3756, 3), (50_000_000 // 3760 + 1, 3760, 2), (50_000_000 // 4093 + 1, 4093, 2),
    # one workgroup per row
    (50_000_000 // 6001 + 1, 6001, 5),
    (50_000_000 // 8000 + 1, 8000, 4), (50_000_000 // 8150 + 1, 8150, 4), (75_000_000 // 8192 + 1, 8192, 3), (75_000_000 // 8192, 8192, 4), (50_000_000 // 8192, 8192, 0),
    (50_000_000 // 9000 + 1, 9000, 4), (110_000_000 // 9300, 9300, 0), (110_000_000 // 9300 + 1, 9300, 3), (110_000_000 // 10240 + 1, 10240, 3),
    (150_000_000 // 16000 + 1, 16000, 2), (150_000_000 // 16000, 16000, 0)])
def test_workgroups_per_compute_unit(lib, rows, cols, most):
    """The LDS that long launches ask for: that many workgroups fit the 160 KB of a compute unit beside their
    own (less than 1 KB), handed out in units of 1280 bytes, and one more does not."""
    got = batch(lib, [(rows, ip.softmax_prepare(0.0085, cols, 1, 0))], cols)
    assert len(got) == 1 and got[0].kernel in ("softmax_wide_kernel", "softmax_wgrow_kernel")
    if most == 0:
        assert got[0].lds == 0
    else:
        for own in (1, 1024):
            assert 128 // -(-(got[0].lds + own) // 1280) == most


@pytest.mark.parametrize("problems,rows,cols,bounded", [
    (1, 115_000_000 // 197, 197, False), (1, 121_000_000 // 197, 197, True), (3, 302_592, 197, True), (4, 245_000, 197, False),
    (4, 260_000, 197, True), (16, 63_000, 197, False), (16, 64_000, 197, True), (1, 95_000_000 // 198, 198, True), (3, 302_592, 198, True),
    (4, 125_000, 198, False), (8, 64_000, 198, True), (12, 302_592, 198, True), (12, 37_000, 198, False)])
def test_slab_kernels_bound_their_long_launches(lib, problems, rows, cols, bounded):
    """Rows of 197 and 198 scores, four lanes per row: two workgroups on a compute unit instead of three, single
    calls and batches; not beside the second degree."""
    got = batch(lib, [(rows, packed_softmax(100, cols))] * problems, cols)
    assert [(l.kernel, l.problems, l.lds > 0) for l in got] == [("softmax_rows_kernel", problems, bounded)]
    own = 4 * 16 * cols * 4
    assert not bounded or (128 // -(-(got[0].lds + own) // 1280), 128 // -(-own // 1280)) == (2, 3)
    assert batch(lib, [(rows, ip.softmax_prepare(0.0085, cols, 2, 0))] * problems, cols)[0].lds == 0


@pytest.mark.parametrize("rows,cols,plain,others", [
    # (with a table, with a requantization in front, of the second degree)
    (70_000, 900, 6, (0, 0, 0)), (70_000, 1000, 5, (5, 0, 5)), (20_000, 3400, 3, (2, 3, 3)), (20_000, 3600, 3, (2, 3, 3)),
    (14_000, 3800, 2, (2, 2, 2)), (14_000, 4096, 2, (2, 2, 2)), (9_200, 8192, 3, (4, 4, 4)), (12_000, 9300, 3, (0, 0, 0)),
    (12_000, 6400, 5, (5, 5, 5)), (45_000, 1500, 4, (4, 4, 4))])
def test_workgroups_beside_more_arithmetic(lib, rows, cols, plain, others):
    """Where a table, a requantization or the second degree fills the time, fewer bounds apply."""
    def fits(variant, fields, pre):
        p = ip.softmax_prepare(0.0085, cols, variant, 0)
        if pre:
            p.pre_m, p.pre_s = 300, 9
        lds = batch(lib, [(rows, p, fields)], cols)[0].lds
        return 0 if lds == 0 else 128 // -(-(lds + 1024) // 1280)

    table = dict(d_bias=SCORES + (1 << 38), bias_period_rows=64)
    if 50 < rows * cols / 1e6 < 60:
        assert fits(1, table, False) == fits(1, {}, True) == 0
        rows = 60_000_000 // cols + 1
    assert (fits(1, {}, False), (fits(1, table, False), fits(1, {}, True), fits(2, {}, False))) == (plain, others)


@pytest.mark.parametrize("rows,cols,own,fit", [
    (612_000, 197, 4 * 16 * 197 * 4, 2), (455_000, 198, 4 * 16 * 198 * 4, 2), (600_000, 197, None, None), (454_000, 198, None, None),
    (340_000, 577, None, None), (275_000, 401, 0, 5), (274_000, 401, None, None), (185_000, 600, 0, 3), (183_000, 600, None, None),
    (196_000, 566, None, None), (196_000, 568, None, None), (175_000, 632, None, None)])
def test_slabs_per_compute_unit(lib, rows, cols, own, fit):
    """The same for the slab kernels, whose workgroups keep their rows in LDS."""
    def lds(n, variant=1, pre=False, **fields):
        p = ip.softmax_prepare(0.0085, cols, variant, 0)
        if pre:
            p.pre_m, p.pre_s = 300, 9
        got = batch(lib, [(n, p, fields)], cols)
        assert len(got) == 1
        return got[0].lds

    short = lds(6400)
    if fit is None:
        assert lds(rows) == short
    else:
        for lut in (16, 1024 if own else 0):
            assert 128 // -(-(lds(rows) + own + lut * bool(own)) // 1280) == fit
    if cols == 198:                                   # one problem or three, not four
        p = ip.softmax_prepare(0.0085, cols, 1, 0)
        of_batch = [batch(lib, [(rows // n + 1, p)] * n, cols)[0].lds for n in (1, 3, 4)]
        assert of_batch == [lds(rows)] * 2 + [short]
    assert lds(rows, variant=2) == lds(rows, pre=True) == lds(rows, d_bias=SCORES + (1 << 38), bias_period_rows=64) == short
