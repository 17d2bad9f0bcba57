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


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_library.build(str(tmp_path_factory.mktemp("recording")))


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
