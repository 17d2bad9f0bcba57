"""The short form of the arguments of the one-wavefront-per-row kernels: every field that a kernel reads
comes back as plan_softmax made it, for random and extreme parameters of the whole domain, and the
largest value of every packed field is among them."""
import os
import shutil
import subprocess

import pytest

from paper_2511_15369_amd import build as lib_build

DRIVER = r"""
#include <hip/hip_runtime.h>
#include <stdio.h>
#include "softmax_wide.h"
using namespace iptq;
static uint64_t s = 0x9E3779B97F4A7C15ull;
static uint64_t rnd() { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return s; }
static int32_t pick(int32_t lo, int32_t hi)       // the ends as often as everything between
{
    const uint64_t r = rnd() % 4;
    return r == 0 ? lo : r == 1 ? hi : lo + (int32_t)(rnd() % (uint64_t)((int64_t)hi - lo + 1));
}
#define SAME(F) if (A.F != U.F) { printf("%s: %lld became %lld\n", #F, (long long)A.F, (long long)U.F); return 1; }
#define LARGEST(F) static long long max_##F; if ((long long)A.P.F > max_##F) max_##F = (long long)A.P.F;
#define PRINT(F) printf(#F " %lld\n", max_##F);
int main()
{
    long n = 0, packed[3] = {0, 0, 0}, folded = 0;
    for (long t = 0; t < 3000000; ++t) {
        iptq_softmax_params_t p;
        p.variant = pick(0, 2);
        p.i0 = pick(16, pick(0, 1) ? 3300 : (1 << 24) - 1);
        p.n_shift = pick(0, 20);
        p.m_bits = pick(1, 31);
        p.out_bits = pick(2, 8);
        p.pre_m = pick(1, 32767);
        const int32_t shifts[] = {0, 15, 16, 31, 32, 33, 62};
        p.pre_s = pick(0, 1) ? shifts[rnd() % 7] : pick(0, 62);
        if (rnd() % 8 == 0) { p.pre_m = 1; p.pre_s = 0; }
        p.out_is_signed = pick(0, 1);
        p.post.m = pick(-32767, 32767);
        p.post.s = pick(0, 62);
        p.post.zp = pick(-(1 << 24), 1 << 24);
        p.post.qmin = p.out_is_signed ? pick(-128, 127) : pick(0, 255);
        p.post.qmax = pick(p.post.qmin, p.out_is_signed ? 127 : 255);
        if (rnd() % 8 == 0) { p.out_is_signed = 1; p.post = {1, 0, -128, -128, pick(0, 127)}; }
        p.algo = 0;
        WideArgs A;
        const int64_t rows = pick(0, INT32_MAX);
        const int32_t cols = pick(1, 4096);
        if (plan_softmax(&p, rows, cols, pick(0, 1), pick(1, INT32_MAX), &A.P) != IPTQ_OK) continue;
        ++n;
        ++packed[A.P.packed];
        folded += A.P.pre_rowconst;
        A.scores = (const int32_t *)rnd(); A.bias = (const int32_t *)rnd(); A.out = (uint8_t *)rnd();
        A.rows = rows; A.cols = cols; A.base_off = pick(0, 3); A.cut_el = pick(0, 3); A.post_mode = pick(0, 2);
        const WideArgs U = wide_unpack(wide_pack(A));
        SAME(scores) SAME(bias) SAME(out) SAME(rows) SAME(cols) SAME(base_off) SAME(cut_el) SAME(post_mode)
        SAME(P.i0) SAME(P.i0n) SAME(P.n_shift) SAME(P.magic) SAME(P.magic_sh) SAME(P.d_clamp) SAME(P.m_bits) SAME(P.p_shift)
        SAME(P.pre_m) SAME(P.pre_s) SAME(P.pre_mode) SAME(P.pre_sh2) SAME(P.pre_rowconst) SAME(P.pre_dmax)
        if (A.P.pre_mode == 1) { SAME(P.pre_mul) SAME(P.pre_rnd) }
        SAME(P.post_m) SAME(P.post_s) SAME(P.post_zp) SAME(P.qmin) SAME(P.qmax) SAME(P.post_xor) SAME(P.variant)
        SAME(P.d2_magic) SAME(P.d2_sh) SAME(P.bias_period_rows) SAME(P.period_magic) SAME(P.period_sh)
        if (A.P.packed == 1) SAME(P.mg24)
        if (A.P.packed == 2) SAME(P.div8)
        LARGEST(n_shift) LARGEST(m_bits) LARGEST(p_shift) LARGEST(pre_s) LARGEST(pre_sh2) LARGEST(post_s) LARGEST(pre_m)
        LARGEST(post_m) LARGEST(qmax) LARGEST(pre_mode) LARGEST(variant) LARGEST(magic_sh) LARGEST(d2_sh) LARGEST(period_sh)
        if (t + 1 < 3000000 && n < 400000) continue;
        PRINT(n_shift) PRINT(m_bits) PRINT(p_shift) PRINT(pre_s) PRINT(pre_sh2) PRINT(post_s) PRINT(pre_m)
        PRINT(post_m) PRINT(qmax) PRINT(pre_mode) PRINT(variant) PRINT(magic_sh) PRINT(d2_sh) PRINT(period_sh)
        printf("packed %ld %ld %ld folded %ld\n", packed[0], packed[1], packed[2], folded);
        return 0;
    }
    printf("too few of the parameters are in the domain\n");
    return 1;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not installed")
def test_every_field_comes_back(tmp_path):
    src = tmp_path / "driver.hip"
    src.write_text(DRIVER)
    objs = []
    for path in (str(src), os.path.join(lib_build.CSRC, "plan.cpp")):
        objs.append(str(tmp_path / os.path.basename(path)) + ".o")
        subprocess.check_call(["hipcc", "-x", "hip", "-c", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                               "-I" + lib_build.CSRC, path, "-o", objs[-1]], stderr=subprocess.DEVNULL)
    exe = str(tmp_path / "driver")
    subprocess.check_call(["hipcc"] + objs + ["-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    largest = dict(line.split() for line in out.stdout.splitlines()[:-1])
    assert {k: int(v) for k, v in largest.items()} == dict(
        n_shift=19, m_bits=31, p_shift=30, pre_s=62, pre_sh2=30, post_s=62, pre_m=32767, post_m=32767, qmax=255, pre_mode=2,
        variant=2, magic_sh=21, d2_sh=16, period_sh=30), out.stdout
    counts = [int(v) for v in out.stdout.splitlines()[-1].split() if v.isdigit()]      # no packed arithmetic, either divider, folded
    assert len(counts) == 4 and min(counts) > 1000, out.stdout
