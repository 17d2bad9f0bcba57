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
    assert sorted((l.kernel, l.arguments[2], l.first_word) for l in got) == [
        ("softmax_rows_kernel", 1, high), ("softmax_rows_kernel", 2, 16 - high)]
    # one launch where each can have the multiply-high divider
    wide = [(4000, packed_softmax(max(q.i0, 257 + i), 197)) for i, (_, q) in enumerate(specs)]
    assert [l.arguments[2] for l in batch(lib, wide, 197)] == [1]
    assert [l.arguments[2] for l in batch(lib, [w for w in wide if w[1].i0 < 1000], 197)] == [2]
    # a layer in 32-bit arithmetic ends the launches in front of it, as it always did
    specs[8] = (4000, packed_softmax(2 ** 14, 197))
    got = batch(lib, specs, 197)
    assert [l.arguments[2] for l in got] == [2, 1, 0, 2, 1] and sum(l.first_word for l in got) == 16


def test_two_short_calls_that_are_sooner_done_apart(lib):
    """Two short calls of the second degree or with a short table, where two launches of a shorter chain
    end sooner; three of them, other calls and longer ones share a launch."""
    table = dict(d_bias=SCORES + (1 << 30), bias_period_rows=40)

    def kernels(n, rows, cols, variant, fields, algo=0):
        p = ip.softmax_prepare(0.0085, cols, variant, 0)
        p.algo = algo
        return [l.kernel for l in batch(lib, [(rows, p, fields)] * n, cols)]

    together = ["softmax_rowsdyn_batch_kernel"]
    for args in ((600, 25, 1, table), (1000, 29, 2, table), (600, 64, 2, {})):
        assert kernels(2, *args) == ["softmax_wide_kernel"] * 2
        assert kernels(2, *args, algo=ip.ALGO_DYNAMIC) == together
        assert kernels(3, *args) == together
    for args in ((64, 25, 1, table), (4000, 25, 1, table), (600, 16, 1, table), (600, 25, 1, {}), (600, 64, 1, {}), (600, 145, 2, {}),
                 (600, 25, 1, dict(table, bias_period_rows=64))):
        assert kernels(2, *args) == together, args
