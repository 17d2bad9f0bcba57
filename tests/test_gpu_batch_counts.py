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
    n = 9 * 4096 + 5                                  # ten workgroups, the last with a few bytes
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
        d_s, d_p = torch.from_numpy(s).cuda(), torch.full(s.shape, 0x5A, dtype=torch.uint8, device="cuda")
        ip.softmax_i32_layers(d_s, rows * cols, d_p, rows * cols, rows, cols, layers, [lib_softmax(q) for q in sp])
        got = d_p.cpu().numpy()
        for l in range(layers):
            assert np.array_equal(got[l], ref.softmax_i32(s[l], sp[l])), (cols, l)
