"""The packed arithmetic's byte divider: wherever the plan enables it, the top byte of the 24-bit
product must be n div i0 for every reachable n, and every scale from 2^-10 to 2^-4 must have it."""
import ctypes

import numpy as np

import paper_2511_15369_amd as ip
from oracle import ref
from tests.helpers import lib_softmax


def _packed(p):
    fn = ip.load().iptq_debug_softmax_packed
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.POINTER(ip.SoftmaxParams), ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32)]
    packed, div8 = ctypes.c_int32(-1), ctypes.c_int32(-1)
    assert fn(ctypes.byref(p), ctypes.byref(packed), ctypes.byref(div8)) == 0
    return packed.value, div8.value


def _plan(p):
    fn = ip.load().iptq_debug_softmax_plan
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.POINTER(ip.SoftmaxParams), ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int64,
                   ctypes.POINTER(ctypes.c_int64)]
    out = (ctypes.c_int64 * 12)()
    assert fn(ctypes.byref(p), 1, 1, 0, 0, out) == 0
    return list(out)


def test_byte_divider_is_exact_wherever_it_is_enabled():
    kinds = {0: 0, 1: 0, 2: 0}
    for i0 in list(range(16, 3400)) + [4000, 5000, 2 ** 14, 2 ** 15 - 1, 2 ** 16, 2 ** 20]:
        for n_shift in {max(0, 15 - i0.bit_length()), 0}:
            p = lib_softmax(ref.SoftmaxParams(variant=1, i0=i0, n_shift=n_shift))
            packed, div8 = _packed(p)
            o = _plan(p)
            D, i0n, p_shift, n_max, mg24 = o[2], o[3], o[4], o[7], o[9]
            kinds[packed] += 1
            # everything that fits 16 bits has one of the dividers (a shifted multiply-high one, exact for
            # every such n, shows what fits)
            fits = D <= 32767 and i0n < 2 ** 15 and p_shift <= 24 and i0n >= 2 ** p.out_bits
            t = max(0, (2 ** 32 // i0 + 1).bit_length() - 24)
            fits = fits and (n_max << t) <= 65535
            assert (packed != 0) == fits, i0
            assert packed != 1 or mg24 != 0
            assert (packed == 2) == (div8 != 0)
            if packed != 2:
                continue
            assert n_max <= 32768 and 0 < -div8 < 2 ** 23         # both factors fit a signed 24-bit multiply
            n = np.arange(0, n_max + 1, dtype=np.int64)
            product = n * -div8
            assert int(product[-1]) < 2 ** 31
            assert np.array_equal(product >> 24, n // i0), i0
    assert kinds[2] > 2000 and kinds[1] > 1000 and kinds[0] > 0
    for log2s in np.linspace(-10, -4, 200):
        assert _packed(ip.softmax_prepare(float(2.0 ** log2s), 197, 1, 0))[0] == 2
