"""int32 GELU and requantization at the sizes where a thread's number of chunks or the form of its loop
changes (one chunk; the resident grid and one more; the grid rules' lines; more than four trips of the
long grid), at odd offsets, against the formula in 64 bits and the oracle's value of every code."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_gelu

pytestmark = pytest.mark.gpu
ONE = 4 * 256 * 2048                                     # values that give every resident thread one chunk
LONG = 4 * 256 * 16384 * 4                               # and four chunks to every thread of the long grid


@pytest.mark.parametrize("n", [63, 64, 67, 1025, ONE - 4, ONE, ONE + 1, ONE + 1027, 2 * ONE + 5, 2_800_001, 4_200_003,
                               24_000_002, 25_000_000, 25_000_003, 29_000_000, 29_000_003, 30_000_000, 30_000_001, 40_000_003, LONG, LONG + 9])
@pytest.mark.parametrize("offset", [0, 3])
def test_gelu_i32_and_requant_over_the_grids(n, offset):
    import torch
    import paper_2511_15369_amd as ip
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    whole = torch.randint(-2 ** 22, 2 ** 22, (n + 16,), device="cuda", generator=g, dtype=torch.int32)
    x = whole[offset:offset + n]
    p = prepare.gelu_prepare(2.0 ** -5, 2.0 ** -6, 0, -7, 1, 127)
    codes = np.arange(-127, 128, dtype=np.int32)
    table = torch.from_numpy(ref.gelu_i32(codes, p)).cuda()
    p.pre_m, p.pre_s = 20000, 24
    step = 1 << 24
    for what in ("gelu", "requant"):
        out = torch.full((n + 64,), 0x5A, dtype=torch.int8, device="cuda")
        y = out[16 + offset:16 + offset + n]
        if what == "gelu":
            ip.gelu_i32(x, y, n, lib_gelu(p))
        else:
            ip.requant(x, y, n, 1, ip.Dyadic(20480, 25, 3, -128, 127))
        torch.cuda.synchronize()
        for a in range(0, n, step):
            w = x[a:a + step].long()
            if what == "gelu":
                want = table[((w * 20000 + (1 << 23)) >> 24).clamp(-127, 127) + 127]
            else:
                want = (((w * 20480 + (1 << 24)) >> 25) + 3).clamp(-128, 127).to(torch.int8)
            assert torch.equal(y[a:a + step], want), (what, a)
        assert bool((out[:16 + offset] == 0x5A).all()) and bool((out[16 + offset + n:] == 0x5A).all())
