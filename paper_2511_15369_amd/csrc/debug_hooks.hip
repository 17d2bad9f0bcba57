// Test hooks of the library (include/iptq_debug.h): internals exposed so that the tests can
// check them one by one - the integer helpers compiled for the host, the host-side plans and
// layouts, and the two exponential code paths on their own.  Not part of the product API.
#include <hip/hip_runtime.h>

#include "../../include/iptq.h"
#include "../../include/iptq_debug.h"
#include "device_common.h"
#include "kernels.h"
#include "plan.h"
#include "softmax_rows.h"

using namespace iptq;

extern "C" uint32_t iptq_debug_floor_pow2_div(int32_t m_bits, uint32_t sigma)
{
    return floor_pow2_div(m_bits, sigma);
}

extern "C" int iptq_debug_softmax_plan(const iptq_softmax_params_t *p, int64_t rows, int32_t cols,
                                       int32_t has_bias, int64_t bias_period_rows, int64_t *out12)
{
    SoftmaxDev dev;
    int rc = plan_softmax(p, rows, cols, has_bias, bias_period_rows, &dev);
    if (rc != IPTQ_OK || !out12) return rc;
    out12[0] = dev.magic; out12[1] = dev.magic_sh; out12[2] = dev.d_clamp; out12[3] = dev.i0n;
    out12[4] = dev.p_shift; out12[5] = dev.period_magic; out12[6] = dev.period_sh;
    out12[7] = neg_qp_of(dev.d_clamp);
    out12[8] = dev.packed; out12[9] = dev.mg24; out12[10] = -(int64_t)dev.div8;
    out12[11] = dev.pre_rowconst ? (int64_t)dev.pre_dmax : 0;
    return rc;
}

extern "C" int iptq_debug_softmax_packed(const iptq_softmax_params_t *p, int32_t *packed, int32_t *div8)
{
    SoftmaxDev dev;
    const int rc = plan_softmax(p, 1, 1, 0, 0, &dev);
    if (rc != IPTQ_OK || !packed || !div8) return rc;
    *packed = dev.packed;
    *div8 = dev.div8;
    return rc;
}

// Layout the run-time-row-length kernels would use for a row length:
// out12 = {slab ok, its lanes per row, its blocks per lane, the same again, wide ok, wide passes, wide slots,
//          1 if the row length has a compiled kernel, passes of the walking workgroup (0: none),
//          workgroup-per-row ok, its wavefronts, its slots}.
extern "C" int iptq_debug_softmax_layout(int32_t cols, int32_t *out12)
{
    if (!out12) return IPTQ_ERR_NULL;
    if (cols < 1 || cols > IPTQ_COLS_MAX) return IPTQ_ERR_SHAPE;
    int a = 0, b = 0;
    out12[0] = rowsdyn_geometry(cols, &a, &b) ? 1 : 0;
    out12[1] = a; out12[2] = b; out12[3] = b;
    a = b = 0;
    out12[4] = wide_geometry(cols, &a, &b) ? 1 : 0;
    out12[5] = a; out12[6] = b;
    a = b = 0;
    out12[7] = softmax_rows_compiled(cols) ? 1 : 0;
    a = b = 0;
    out12[8] = long_geometry(cols, &a) ? a : 0;
    a = b = 0;
    out12[9] = wgrow_geometry(cols, &a, &b) ? 1 : 0;
    out12[10] = a; out12[11] = b;
    return IPTQ_OK;
}

extern "C" int iptq_debug_rowsdyn_loses_short_call(int64_t rows, int32_t cols, int32_t has_bias, int32_t mask_kind)
{
    return rowsdyn_loses_short_call(rows, cols, has_bias != 0, mask_kind == 1, mask_kind == 2) ? 1 : 0;
}

extern "C" int iptq_debug_wgrow16_is_faster(int64_t rows, int32_t has_bias, int32_t has_pre, int32_t variant)
{
    return wgrow16_is_faster(rows, has_bias != 0, has_pre != 0, variant) ? 1 : 0;
}

extern "C" int iptq_debug_gelu32_looping_grid(int64_t n, int32_t out_on_line)
{
    return gelu32_looping_grid(n, out_on_line != 0) ? 1 : 0;
}

// Exponentials of an array of stabilised scores (row maximum 0) through both arithmetic
// paths of the softmax kernels: out32 from the 32-bit lanes, out16 from the packed 16-bit
// lanes (pairs (2i, 2i+1); 0xFFFFFFFF where the plan does not enable that path).  n even.
__global__ void __launch_bounds__(256)
debug_bit_exp_kernel(const int32_t *delta, uint32_t *out32, uint32_t *out16, int64_t n, SoftmaxDev P)
{
    const int64_t i = 2 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    if (i + 1 >= n + 1 || i >= n) return;
    const int32_t xa = delta[i], xb = delta[i + 1];
    const int32_t lower = -P.d_clamp;
    if (P.variant == 0) {
        out32[i] = bit_exp_dev<0, true>(xa, lower, 0, P);
        out32[i + 1] = bit_exp_dev<0, true>(xb, lower, 0, P);
    } else if (P.variant == 1) {
        out32[i] = bit_exp_dev<1, true>(xa, lower, 0, P);
        out32[i + 1] = bit_exp_dev<1, true>(xb, lower, 0, P);
    } else {
        out32[i] = bit_exp_dev<2, true>(xa, lower, 0, P);
        out32[i + 1] = bit_exp_dev<2, true>(xb, lower, 0, P);
    }
    if (P.packed == 0) {
        out16[i] = out16[i + 1] = 0xFFFFFFFFu;
    } else {
        const int32_t x[4] = {xa, xb, xb, xa};
        uint32_t e[2];
        if (P.packed == 1) {
            if (P.variant == 0) bit_exp_block<0, false>(x, 0, lower, P, e);
            else if (P.variant == 1) bit_exp_block<1, false>(x, 0, lower, P, e);
            else bit_exp_block<2, false>(x, 0, lower, P, e);
        } else {
            if (P.variant == 0) bit_exp_block<0, true>(x, 0, lower, P, e);
            else if (P.variant == 1) bit_exp_block<1, true>(x, 0, lower, P, e);
            else bit_exp_block<2, true>(x, 0, lower, P, e);
        }
        out16[i] = e[0] & 0xffffu;
        out16[i + 1] = e[0] >> 16;
        if ((e[1] >> 16 | e[1] << 16) != e[0]) out16[i] = 0xFFFFFFFEu;      // the halves of a block disagree
    }
}

extern "C" int iptq_debug_bit_exp(const int32_t *d_delta, uint32_t *d_out32, uint32_t *d_out16,
                                  int64_t n, const iptq_softmax_params_t *p, void *stream)
{
    if (!p || !d_delta || !d_out32 || !d_out16) return IPTQ_ERR_NULL;
    if (n < 0 || (n & 1)) return IPTQ_ERR_SHAPE;
    SoftmaxDev dev;
    int rc = plan_softmax(p, 1, 1, 0, 0, &dev);
    if (rc != IPTQ_OK || n == 0) return rc;
    hipLaunchKernelGGL(debug_bit_exp_kernel, dim3((unsigned)((n / 2 + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), d_delta, d_out32, d_out16, n, dev);
    return hipGetLastError() == hipSuccess ? IPTQ_OK : IPTQ_ERR_HIP;
}
