"""int8 GELU on both sides of every line of the rule that picks its store policy, at odd sizes and
offsets and in place: the oracle's value of each of the 256 codes, gathered."""
import numpy as np
import pytest

from oracle import prepare, ref
from tests.helpers import lib_gelu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 4097, 2_000_000, 2_000_013, 17_999_999, 18_000_000, 18_000_016, 92_000_000, 92_000_031])
@pytest.mark.parametrize("offset,in_place", [(0, False), (5, False), (3, True)])
def test_gelu_i8_store_policies(n, offset, in_place):
    import torch
    import paper_2511_15369_amd as ip
    p = prepare.gelu_prepare(2.0 ** -5, 2.0 ** -6, 3, -7, 1)
    codes = np.arange(-128, 128, dtype=np.int8)
    table = torch.from_numpy(ref.gelu_i8(codes, p)).cuda()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    whole = torch.randint(-128, 128, (n + 64,), device="cuda", generator=g, dtype=torch.int8)
    before = whole.clone()
    x = whole[16 + offset:16 + offset + n]
    out = whole if in_place else torch.full_like(whole, 0x5A)
    y = out[16 + offset:16 + offset + n]
    want = table[x.long() + 128]
    ip.gelu_i8(x, y, n, lib_gelu(p))
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    guard = before if in_place else torch.full_like(whole, 0x5A)
    assert torch.equal(out[:16 + offset], guard[:16 + offset]) and torch.equal(out[16 + offset + n:], guard[16 + offset + n:])
