"""Per-window masks, both forms, for windows of any size in the run-time-row-length slab kernel,
against the oracle: every lane layout's edges, first and last mask rows (blocks that reach past either
end of the table), ragged row counts, with and without a bias, views off the 16-byte grid."""
import numpy as np
import pytest

import paper_2511_15369_amd as ip
from oracle import prepare, ref
from tests.helpers import gpu_softmax_windowed, gpu_softmax_windowed_bits, lib_softmax

pytestmark = pytest.mark.gpu
I32_MIN = -(2 ** 31)


def _problem(t, heads, n_w, images, drop, seed):
    rng = np.random.default_rng(seed)
    rows = images * n_w * heads * t - drop
    scores = np.rint(rng.standard_normal((rows, t)) * 400).astype(np.int32)
    scores[rng.random(scores.shape) < 0.01] = I32_MIN
    bias = np.rint(rng.standard_normal((heads * t, t)) * 8).astype(np.int32)
    bias[rng.random(bias.shape) < 0.01] = I32_MIN
    bias[0, 0] = I32_MIN + 5                                 # saturates low: minus infinity from there on
    mask = np.where(rng.random((n_w, t, t)) < 0.4, I32_MIN, 0).astype(np.int32)
    mask[n_w - 1, t - 1, :] = I32_MIN                        # the table's last row masked in full
    return rng, scores, bias, mask


@pytest.mark.parametrize("t,heads,n_w", [
    (1, 3, 5), (2, 40, 3), (3, 12, 2), (4, 8, 3), (9, 4, 3), (16, 2, 3), (25, 2, 4), (25, 1, 4), (25, 3, 4), (29, 2, 3),
    (30, 1, 3), (36, 3, 4), (49, 2, 4), (58, 2, 3), (61, 2, 3), (62, 2, 3), (64, 3, 4), (65, 1, 3), (100, 3, 3), (125, 1, 3),
    (126, 2, 2), (128, 1, 3), (129, 1, 3), (144, 2, 3), (196, 2, 3), (225, 1, 3), (253, 1, 2), (256, 1, 2), (257, 1, 2),
    (400, 1, 2), (511, 1, 1), (577, 1, 2), (576, 1, 2), (635, 1, 1)])
def test_masks_match_the_oracle(t, heads, n_w):
    images = 4 if t < 100 else 2
    rng, scores, bias, mask = _problem(t, heads, n_w, images, int(np.random.default_rng(t).integers(0, min(t, 30))), t * 100 + heads)
    finite = mask.copy()
    finite[0] = np.rint(rng.standard_normal((t, t)) * 150).astype(np.int32)      # ordinary addends
    if n_w > 1:
        finite[1, 0, :] = 2 ** 31 - 1                        # saturates high
    bits = ref.pack_window_mask(mask)
    if t % 64:
        bits[:, :, -1] |= np.uint64(((1 << 64) - 1) ^ ((1 << (t % 64)) - 1))     # no such keys
    for variant, signed, s_delta in ((1, 0, 2.0 ** -6.5), (0, 1, 2.0 ** -14), (2, 0, 2.0 ** -5)):
        p = prepare.softmax_prepare(s_delta, t, variant, signed)
        for b, period in ((bias, heads * t), (None, 0)):
            want = ref.softmax_i32_windowed(scores, p, b, period, mask, heads)
            for algo in (0, 4):                              # 0 leaves some short calls to the three-pass kernel
                assert np.array_equal(gpu_softmax_windowed_bits(scores, p, b, period, bits, heads, algo=algo), want)
            want = ref.softmax_i32_windowed(scores, p, b, period, finite, heads)
            for algo in (0, 4):
                assert np.array_equal(gpu_softmax_windowed(scores, p, b, period, finite, heads, algo=algo), want)


@pytest.mark.parametrize("t", [25, 64, 100, 196])
def test_views_off_the_grid_and_requantization(t):
    import torch
    heads, n_w, images = 3, 3, 2
    rng, scores, bias, mask = _problem(t, heads, n_w, images, 1, t)
    scores = np.where(scores == I32_MIN, I32_MIN, scores * 40).astype(np.int32)
    p = prepare.softmax_prepare(2.0 ** -5, t, 1)
    p.pre_m, p.pre_s = 20000, 20
    want = ref.softmax_i32_windowed(scores, p, bias, heads * t, mask, heads).reshape(-1)
    n = scores.size
    d_bits = torch.from_numpy(ref.pack_window_mask(mask).view(np.int64)).cuda()
    d_mask = torch.zeros(mask.size + 8, dtype=torch.int32, device="cuda")
    for off in (0, 1, 2, 3):
        d_in = torch.zeros(n + 8, dtype=torch.int32, device="cuda")
        d_in[off:off + n] = torch.from_numpy(scores.reshape(-1)).cuda()
        d_bias = torch.zeros(bias.size + 8, dtype=torch.int32, device="cuda")
        d_bias[off:off + bias.size] = torch.from_numpy(bias.reshape(-1)).cuda()
        d_mask[off:off + mask.size] = torch.from_numpy(mask.reshape(-1)).cuda()
        for kind, algo in (("int32", 0), ("bits", 0), ("int32", 4), ("bits", 4)):
            d_out = torch.full((n + 16,), 0x5A, dtype=torch.uint8, device="cuda")
            b = d_bias[off:off + bias.size]
            if kind == "int32":
                ip.softmax_i32_windowed(d_in[off:off + n], b, heads * t, d_mask[off:off + mask.size], n_w, heads,
                                        d_out[off:off + n], scores.shape[0], t, lib_softmax(p, algo))
            else:
                ip.softmax_i32_windowed_bits(d_in[off:off + n], b, heads * t, d_bits, n_w, heads,
                                             d_out[off:off + n], scores.shape[0], t, lib_softmax(p, algo))
            torch.cuda.synchronize()
            got = d_out.cpu().numpy()
            assert np.array_equal(got[off:off + n], want), (kind, algo, off)
            assert (got[:off] == 0x5A).all() and (got[off + n:] == 0x5A).all(), (kind, algo, off)


@pytest.mark.parametrize("t", [49, 64, 144])
def test_minus_infinity_at_every_stage(t):
    """A score, a bias entry, their (saturated) sum or a mask entry that is INT32_MIN masks the key,
    whatever is added to it afterwards; one above INT32_MIN does not."""
    heads, n_w, images = 2, 3, 3
    rng = np.random.default_rng(t)
    rows = images * n_w * heads * t - 3
    scores = rng.choice(np.array([I32_MIN, I32_MIN + 1, I32_MIN + 10, I32_MIN + 100], np.int32), size=(rows, t))
    scores[::3] = rng.choice(np.array([I32_MIN, I32_MIN + 1, -50, 0, 50], np.int32), size=scores[::3].shape)
    bias = rng.choice(np.array([I32_MIN, -100, -10, -1, 0, 1, 100], np.int32), size=(heads * t, t))
    # windows 0 and 1: what a masked key would be lifted to lies as high as the live keys of its row
    mask = rng.choice(np.array([I32_MIN, 0, 1, 99], np.int32), size=(n_w, t, t))
    mask[1] = rng.choice(np.array([I32_MIN, 2 ** 31 - 1], np.int32), size=(t, t))
    first = scores[:heads * t].astype(np.int64) + bias
    lifted = (first <= I32_MIN) & (scores[:heads * t] != I32_MIN) & (bias != I32_MIN) & (np.tile(mask[0], (heads, 1)) > 0)
    assert lifted.sum() > t                                  # the sum alone masks it, the mask entry is positive
    for variant, signed, s_delta in ((1, 0, 2.0 ** -6.5), (0, 1, 2.0 ** -14), (2, 0, 2.0 ** -5)):
        p = prepare.softmax_prepare(s_delta, t, variant, signed)
        want = ref.softmax_i32_windowed(scores, p, bias, heads * t, mask, heads)
        for algo in (0, 1, 4):
            got = gpu_softmax_windowed(scores, p, bias, heads * t, mask, heads, algo=algo)
            assert np.array_equal(got, want), (variant, signed, algo)
