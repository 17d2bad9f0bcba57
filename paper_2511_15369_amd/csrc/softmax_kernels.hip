// Integer softmax for gfx950 (Section 4.4, Eq. 6-15): the any-row-length kernel and the
// dispatch between it and the others.
//   softmax_generic_kernel - run-time row length, one wavefront per row, three passes.
//                          Serves what no other kernel takes (tables and masks beside long rows
//                          that do not qualify) and short calls whose kernel would start later.
#include <hip/hip_runtime.h>

#include "../../include/iptq.h"
#include "device_common.h"
#include "kernels.h"
#include "plan.h"
#include "softmax_rows.h"

namespace iptq {

// ---------------------------------------------------------------------------------------
// Any row length: one wavefront per row, three passes over the row (maximum, sum of
// exponentials, normalise).  The row is re-read from global memory in each pass; a row of
// a few hundred scores stays in the L1/L2 cache between passes.
template <int VARIANT>
__global__ void __launch_bounds__(256)
softmax_generic_kernel(const int32_t *__restrict__ scores, const int32_t *__restrict__ bias,
                       const int32_t *__restrict__ mask, const uint64_t *__restrict__ mask_bits,
                       uint8_t *__restrict__ out, int64_t row_begin, int64_t row_end, int32_t cols,
                       int32_t has_bias, int32_t has_pre, SoftmaxDev P)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = row_begin + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= row_end) return;
    const int32_t *srow = scores + row * cols;
    const int32_t *brow = nullptr;
    if (has_bias) brow = bias + (int64_t)row_mod_period((uint32_t)row, P) * cols;
    const int32_t *mrow = nullptr;
    const uint64_t *mbits = nullptr;                  // the row's mask one bit per key
    if (mask || mask_bits) {
        // rows are ordered [image, window, head, query]: window (r mod period) div (heads * cols),
        // query (r mod (heads * cols)) mod cols; cols is a run-time value here, so the last one is
        // a subtraction loop over the heads in front (once per row)
        const uint32_t r = (uint32_t)row;
        uint32_t rm = 0;
        if (P.mask_period_rows >= 2)
            rm = r - (mulhi_u32(r, P.mperiod_magic) >> P.mperiod_sh) * (uint32_t)P.mask_period_rows;
        const uint32_t w = P.group_rows >= 2 ? mulhi_u32(rm, P.group_magic) >> P.group_sh : rm;
        uint32_t q = rm - w * (uint32_t)P.group_rows;
        while (q >= (uint32_t)cols) q -= (uint32_t)cols;
        if (mask) mrow = mask + ((int64_t)w * cols + q) * cols;
        else mbits = mask_bits + ((int64_t)w * cols + q) * ((cols + 63) >> 6);
    }

    auto fetch = [&](int c) -> int32_t {
        int32_t v = srow[c];
        if (has_bias) v = add_table_entry(v, brow[c]);
        if (mrow) v = add_table_entry(v, mrow[c]);
        if (mbits && ((mbits[c >> 6] >> (c & 63)) & 1)) v = kI32Min;
        if (has_pre && v != kI32Min) v = pre_requant_dev(v, P.pre_m, P.pre_s);
        return v;
    };

    int32_t mx = kI32Min;
    for (int c = lane; c < cols; c += 64) mx = max(mx, fetch(c));
    mx = wave_max_i32(mx);

    const int32_t D = P.d_clamp;
    const int32_t lower = (mx < kI32Min + D) ? kI32Min : mx - D;
    uint32_t sum = 0;
    for (int c = lane; c < cols; c += 64) sum += bit_exp_dev<VARIANT, true>(fetch(c), lower, mx, P);
    sum = wave_sum_u32(sum);

    const uint32_t f = floor_pow2_div(P.m_bits, sum);
    uint8_t *orow = out + row * cols;
    for (int c = lane; c < cols; c += 64) {
        const uint32_t q = bit_exp_dev<VARIANT, true>(fetch(c), lower, mx, P);
        const uint32_t p = (q * f) >> P.p_shift;
        orow[c] = (uint8_t)post_dev<PM_GENERAL>(p, P);
    }
}

// ---------------------------------------------------------------------------------------
// A 0 / INT32_MIN window mask as one bit per key: thread x = query row, block y = word of that
// row; each thread reads up to 64 entries of its mask row.  Run once per model (a few hundred
// kilobytes), not on the inference path.
__global__ void __launch_bounds__(256)
pack_window_mask_kernel(const int32_t *__restrict__ mask, int64_t n_queries, int32_t cols,
                        int32_t words, uint64_t *__restrict__ bits)
{
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= n_queries) return;
    const int32_t wd = (int32_t)blockIdx.y;
    const int32_t *m = mask + row * cols;
    const int32_t k0 = wd * 64;
    const int32_t k1 = min(cols, k0 + 64);
    uint64_t w = 0;
    for (int32_t k = k0; k < k1; ++k)
        if (m[k] == kI32Min) w |= (uint64_t)1 << (k - k0);
    bits[row * words + wd] = w;
}

hipError_t pack_window_mask_dispatch(const int32_t *mask, int64_t n_queries, int32_t cols, uint64_t *bits,
                                     hipStream_t stream)
{
    const int32_t words = (cols + 63) / 64;           // at most 1024
    if (n_queries <= 0) return hipSuccess;
    launch_kernel(pack_window_mask_kernel, dim3((unsigned)((n_queries + 255) / 256), (unsigned)words),
                       dim3(256), 0, stream, mask, n_queries, cols, words, bits);
    return take_launch_status();
}

// ---------------------------------------------------------------------------------------
// Host-side dispatch.

static int post_mode_of(const SoftmaxDev &P, int out_bits)
{
    if (P.post_xor != 0) return PM_NONE;              // p - 128: one exclusive-or on the packed bytes
    const bool identity = P.post_m == 1 && P.post_s == 0 && P.post_zp == 0 && P.qmin <= 0;
    if (!identity) return PM_GENERAL;
    if (P.qmax >= (1 << (out_bits - 1))) return PM_NONE;
    return (P.qmax == 127 && out_bits == 8) ? PM_CLAMP127 : PM_GENERAL;
}

static hipError_t launch_generic(const int32_t *scores, const int32_t *bias, const int32_t *mask,
                                 const uint64_t *mask_bits, uint8_t *out, int64_t row_begin, int64_t row_end, int32_t cols,
                                 bool has_bias, bool has_pre, const SoftmaxDev &P, hipStream_t stream)
{
    const int64_t n = row_end - row_begin;
    if (n <= 0) return hipSuccess;
    const dim3 grid((unsigned)((n + 3) / 4)), block(256);
    if (P.variant == 0)
        launch_kernel(softmax_generic_kernel<0>, grid, block, 0, stream, scores, bias, mask, mask_bits, out,
                           row_begin, row_end, cols, (int32_t)has_bias, (int32_t)has_pre, P);
    else if (P.variant == 1)
        launch_kernel(softmax_generic_kernel<1>, grid, block, 0, stream, scores, bias, mask, mask_bits, out,
                           row_begin, row_end, cols, (int32_t)has_bias, (int32_t)has_pre, P);
    else
        launch_kernel(softmax_generic_kernel<2>, grid, block, 0, stream, scores, bias, mask, mask_bits, out,
                           row_begin, row_end, cols, (int32_t)has_bias, (int32_t)has_pre, P);
    return take_launch_status();
}

// Whether no call writes what another one reads or writes.  First the layers of one tensor, whose outputs
// follow each other away from everything that is read: one pass (16 layers 0.2 us); else pair by pair (1.6 us).
struct Range { uintptr_t from, to; };
static bool meet(Range a, Range b) { return a.from < b.to && b.from < a.to; }
static Range range_of(const void *p, int64_t bytes)
{
    const uintptr_t from = reinterpret_cast<uintptr_t>(p);
    return {from, p == nullptr ? from : from + (uintptr_t)bytes};     // (a null one is empty and meets nothing)
}
static bool independent(const SoftmaxCall *calls, int n_calls, int32_t cols)
{
    struct { Range out, in[4]; } r[kBatchMax];
    Range outs = {UINTPTR_MAX, 0}, ins = {UINTPTR_MAX, 0};
    bool in_sequence = true;
    for (int i = 0; i < n_calls; ++i) {
        const SoftmaxCall &c = calls[i];
        const int64_t n = c.rows * cols, queries = (int64_t)c.P.n_windows * cols;
        r[i].out = range_of(c.out, n);
        r[i].in[0] = range_of(c.scores, 4 * n);
        r[i].in[1] = range_of(c.bias, 4 * (int64_t)c.P.bias_period_rows * cols);
        r[i].in[2] = range_of(c.mask, 4 * queries * cols);
        r[i].in[3] = range_of(c.mask_bits, 8 * queries * ((cols + 63) / 64));
        in_sequence = in_sequence && r[i].out.from >= outs.to;
        if (i == 0) outs.from = r[i].out.from;
        outs.to = r[i].out.to;
        for (const Range &in : r[i].in) {
            if (in.from == in.to) continue;
            if (in.from < ins.from) ins.from = in.from;
            if (in.to > ins.to) ins.to = in.to;
        }
    }
    if (in_sequence && !meet(outs, ins)) return true;
    for (int i = 0; i < n_calls; ++i)
        for (int j = 0; j < n_calls; ++j) {
            if (i == j) continue;
            if (meet(r[i].out, r[j].out)) return false;
            for (const Range &in : r[j].in)
                if (meet(r[i].out, in)) return false;
        }
    return true;
}

// Enqueue the softmax of every call (all with the same row length).  Calls that can use a
// fixed-row-length kernel are grouped, up to kBatchMax per launch, while they agree on what
// the kernel instantiation fixes (bias or not, post step, arithmetic); the
// rows a slab decomposition leaves over, and calls it cannot serve, go to the generic kernel.
bool softmax_rows_compiled(int32_t cols)
{
#define IPTQ_IS_ROWS_SHAPE(COLS, K) if (cols == COLS) return true;
    IPTQ_ROWS_SHAPES(IPTQ_IS_ROWS_SHAPE)
#undef IPTQ_IS_ROWS_SHAPE
    return false;
}

hipError_t softmax_dispatch(const SoftmaxCall *calls, int n_calls, int32_t cols, hipStream_t stream)
{
    // A single call of a few thousand rows is one generation of wavefronts whatever the kernel:
    // its duration is one wavefront's chain of load, arithmetic and store, and one wavefront per
    // row has the shortest.  Graph times, one wavefront per row and the slab kernel: 512 / 2560 / 3072 / 4608 rows of
    // 197 scores 2.8 / 3.57 / 3.65 / 4.05 us and 3.35 / 3.84 / 3.91 / 4.01, of 49 with a table 3.06 / 3.61 / 3.62 / 4.08
    // and 3.85 / 4.01 / 4.03 / 3.97, of 577 3.31 / 4.67 / 4.77 / 5.63 and 3.99 / 4.85 / 4.96 / 6.36; ragged row counts the
    // same.  They cross between 2300 rows (of 36 scores) and 7000 (of 64 and 256): of 600 calls of 256 to 3072 rows of
    // 16 to 600 scores, with and without a table, this line loses in 7, at most 7 % (the slab kernel always: 20 % on
    // average); from there to 8192 rows the slab kernel is 4.8 % slower on average, most in rows of 64 and 256.
    constexpr int64_t kTinyRows = 3072;
    // (a per-window mask exists in the slab kernels, compiled and run-time row length, and in the
    // three-pass kernel)
    auto slab_only = [](const SoftmaxCall &c) { return c.mask != nullptr || c.mask_bits != nullptr; };
    if (n_calls == 1 && calls[0].algo == IPTQ_ALGO_AUTO && calls[0].rows <= kTinyRows && !slab_only(calls[0])) {
        int64_t served = 0;
        const hipError_t e = softmax_wide_launch(calls[0], cols, post_mode_of(calls[0].P, calls[0].out_bits),
                                                 &served, stream);
        if (e != hipSuccess) return e;
        if (served == calls[0].rows) return hipSuccess;      // every row or none
    }
    int rpw = 0;                                      // rows per wavefront of the compiled row length
    hipError_t (*launch)(const SoftmaxBatch &, unsigned, bool, int, bool, int, int, hipStream_t) = nullptr;
#define IPTQ_PICK_ROWS_SHAPE(COLS, K)                                                             \
    if (cols == COLS) { rpw = 64 / K; launch = launch_softmax_rows<COLS, K>; }
    IPTQ_ROWS_SHAPES(IPTQ_PICK_ROWS_SHAPE)
    int64_t total_rows = 0;
    for (int i = 0; i < n_calls; ++i) total_rows += calls[i].rows;
    if (total_rows * cols <= kRowsAltMaxElements) {   // a short launch: more lanes per row
        IPTQ_ROWS_SHAPES_ALT(IPTQ_PICK_ROWS_SHAPE)
    }
#undef IPTQ_PICK_ROWS_SHAPE
    // Calls of either packed arithmetic are collected side by side (a kernel has one of the dividers), so
    // that layers whose scales lie on both sides of the byte divider's range take two launches, in
    // whatever order they come: [1] multiply-high divider, [0] the rest.  One launch where every call can
    // have the multiply-high divider (i0 > 256): a launch costs 3 us, its six more instructions per four
    // scores less than that.
    struct Group {
        SoftmaxBatch B;
        unsigned total_wgs;
        bool fold;
    } group[2];
    for (Group &g : group) { g.B.head.clear(); g.total_wgs = 0; g.fold = false; }
    bool g_bias = false;
    int g_mask = 0, g_pm = 0, g_mode = 0;             // g_mask: 0 none, 1 int32 table, 2 one bit per key; g_mode: group[0]'s
    hipError_t err = hipSuccess;
    auto flush = [&]() {
        for (int i = 0; i < 2; ++i) {
            Group &g = group[i];
            if (g.B.head.n_items == 0 || err != hipSuccess) continue;
            err = launch(g.B, g.total_wgs, g_bias, g_mask, g.fold, i == 1 ? 1 : g_mode, g_pm, stream);
            g.fold = false;
            g.B.head.clear();
            g.total_wgs = 0;
        }
    };
    int64_t done[kBatchMax];
    for (int base = 0; base < n_calls; base += kBatchMax) {
        const int cnt = n_calls - base < kBatchMax ? n_calls - base : kBatchMax;
        bool any_high = false, all_high = true;
        for (int i = 0; i < cnt; ++i) {
            const SoftmaxDev &P = calls[base + i].P;
            any_high = any_high || P.packed == 1;
            all_high = all_high && (P.packed != 2 || P.mg24 != 0);
        }
        for (int i = 0; i < cnt; ++i) {
            const SoftmaxCall &c = calls[base + i];
            done[i] = 0;
            const bool has_bias = c.bias != nullptr;
            // the slab kernels load and store 16 bytes at any element address: views that start
            // off the 16-byte grid need nothing but their natural alignment
            const bool aligned =
                ((reinterpret_cast<uintptr_t>(c.scores) | reinterpret_cast<uintptr_t>(c.bias)) & 3) == 0;
            // the fused bias wraps at most once per slab, and its byte offsets are 32-bit
            const bool bias_ok = !has_bias || ((int64_t)c.P.bias_period_rows * cols >= 4 &&
                                       (int64_t)c.P.bias_period_rows * cols < ((int64_t)1 << 30) &&
                                               c.P.bias_period_rows >= rpw);
            const bool slab_algo = c.algo == IPTQ_ALGO_AUTO || c.algo == IPTQ_ALGO_SLAB;
            const int has_mask = c.mask != nullptr ? 1 : (c.mask_bits != nullptr ? 2 : 0);
            // the mask is compiled in beside a bias, for window sizes whose slab has no more rows
            // than a window has queries (49 and 144 tokens, in either form of the mask)
            bool mask_ok = true;
            if (has_mask == 1)
                mask_ok = has_bias && rows_mask_compiled(cols) && rpw <= cols &&
                          (reinterpret_cast<uintptr_t>(c.mask) & 3) == 0;
            else if (has_mask == 2)
                mask_ok = has_bias && rows_maskbits_compiled(cols) &&
                          (reinterpret_cast<uintptr_t>(c.mask_bits) & 7) == 0;
            if (rpw == 0 || !slab_algo || !aligned || !bias_ok || !mask_ok) continue;
            if (c.rows == 0) continue;
            const int pm = post_mode_of(c.P, c.out_bits);
            const int mode = c.P.packed == 2 && any_high && all_high ? 1 : c.P.packed;
            const bool first = group[0].B.head.n_items == 0 && group[1].B.head.n_items == 0;
            // (32-bit arithmetic is a launch of its own, and ends the ones in front of it)
            const bool compatible = first || (has_bias == g_bias && has_mask == g_mask && pm == g_pm && (mode == 0) == (g_mode == 0));
            if (!compatible) flush();
            if (first || !compatible) { g_bias = has_bias; g_mask = has_mask; g_pm = pm; g_mode = mode == 0 ? 0 : 2; }
            Group &g = group[mode == 1 ? 1 : 0];      // (at most kBatchMax calls before the flush below)
            if (c.P.pre_rowconst != 0) g.fold = true;
            SoftmaxItem &it = g.B.item[g.B.head.add(g.total_wgs)];
            it.scores = c.scores; it.bias = c.bias; it.mask = c.mask; it.mask_bits = c.mask_bits; it.out = c.out;
            it.P = c.P;
            it.set_rows(c.rows, rpw);
            const int64_t n_slabs = it.n_slabs;
            it.share_q = 0; it.share_magic = 0; it.share_sh = 0;
            int64_t n_wgs = (n_slabs + kRowsWpb - 1) / kRowsWpb;
            if (has_bias) {
                // rows after which the tables repeat: the bias period, or with an int32 mask the least
                // common multiple of both periods.  (A packed mask is too small to be worth sharing:
                // with it in the period 589,824 rows of 12 x 12-token windows take 69.2 us against
                // 66.8 us, 7 x 7 tokens the same.)
                int64_t period = c.P.bias_period_rows;
                if (has_mask == 1) {
                    int64_t a = period, b = c.P.mask_period_rows;
                    while (b != 0) { const int64_t t = a % b; a = b; b = t; }
                    period = period / a * c.P.mask_period_rows;
                }
                int64_t a = period, b = rpw;
                while (b != 0) { const int64_t t = a % b; a = b; b = t; }      // a = gcd
                const int64_t q = period / a;
                if (q >= 2 && q < 65536 && q * kRowsWpb <= n_slabs &&
                    make_magic_u32((uint32_t)q, 31, &it.share_magic, &it.share_sh)) {
                    it.share_q = (uint32_t)q;
                    n_wgs = (n_slabs + kRowsWpb * q - 1) / (kRowsWpb * q) * q;
                }
            }
            g.total_wgs += (unsigned)n_wgs;
            done[i] = c.rows;
        }
        flush();
        // a call no compiled row length served goes to the run-time-row-length kernels; the slab kernel
        // leaves short calls with a mask, a second-degree exponential or a table of fewer rows than its
        // slab to the others where they are faster
        auto leave = [&](const SoftmaxCall &c) {
            const bool may_lose = slab_only(c) || c.P.variant == 2 || (c.bias != nullptr && c.P.bias_period_rows < 64 && cols <= 29);
            if (c.algo != IPTQ_ALGO_AUTO || !may_lose) return false;
            if (!slab_only(c) && softmax_wide_serves(c, cols)) return rowsdyn_loses_to_wavefronts(c.rows, cols);
            return rowsdyn_loses_short_call(c.rows, cols, c.bias != nullptr, c.mask != nullptr, c.mask_bits != nullptr);
        };
        // several calls of the run-time-row-length kernel in one launch, also the short ones that it would leave
        // one by one: a launch costs more than their chains differ (two calls of 64 to 4000 rows of 25 to 121
        // scores, second degree or a table, 4.8 to 5.4 us call after call, 6.3 to 7.6 as two launches of one
        // wavefront per row; 960 such pairs in a graph 2.9 to 6.9 us against 4.3 to 12, at most 8 % and on average
        // 0.1 % slower).  Where
        // one writes what another one reads or writes, they are made in their order, one launch each
        int pending = 0;
        for (int i = 0; i < cnt; ++i) pending += done[i] == 0;
        if (pending > 1 && err == hipSuccess && independent(calls + base, cnt, cols)) {
            int post_modes[kBatchMax];
            for (int i = 0; i < cnt; ++i) post_modes[i] = post_mode_of(calls[base + i].P, calls[base + i].out_bits);
            err = softmax_rowsdyn_launch_batch(calls + base, post_modes, cnt, cols, done, stream);
        }
        for (int i = 0; i < cnt && err == hipSuccess; ++i) {
            const SoftmaxCall &c = calls[base + i];
            const bool has_pre = !(c.P.pre_m == 1 && c.P.pre_s == 0);
            if (done[i] == 0 && !leave(c) && (c.algo == IPTQ_ALGO_AUTO || c.algo == IPTQ_ALGO_DYNAMIC || c.algo == IPTQ_ALGO_SLAB)) {
                err = softmax_rowsdyn_launch(c, cols, post_mode_of(c.P, c.out_bits), &done[i], stream);
                if (err != hipSuccess) break;
            }
            if (done[i] == 0 && !slab_only(c) && (c.algo == IPTQ_ALGO_AUTO || c.algo == IPTQ_ALGO_WIDE)) {
                err = softmax_wide_launch(c, cols, post_mode_of(c.P, c.out_bits), &done[i], stream);
                if (err != hipSuccess) break;
            }
            if (done[i] == 0 && !slab_only(c) && (c.algo == IPTQ_ALGO_AUTO || c.algo == IPTQ_ALGO_WIDE)) {
                err = softmax_wgrow_launch(c, cols, post_mode_of(c.P, c.out_bits), &done[i], stream);
                if (err != hipSuccess) break;
            }
            if (done[i] == 0 && !slab_only(c) && (c.algo == IPTQ_ALGO_AUTO || c.algo == IPTQ_ALGO_WIDE)) {
                err = softmax_long_launch(c, cols, post_mode_of(c.P, c.out_bits), &done[i], stream);
                if (err != hipSuccess) break;
            }
            err = launch_generic(c.scores, c.bias, c.mask, c.mask_bits, c.out, done[i], c.rows, cols, c.bias != nullptr,
                                 has_pre, c.P, stream);
        }
        if (err != hipSuccess) return err;
    }
    return err;
}

}  // namespace iptq
