// Integer softmax (Section 4.4, Eq. 6-15) for long rows: one wavefront per row, the row
// held in registers, no LDS staging.  All 64 lanes share the row: lane l of pass s owns the
// 16-byte block s * 64 + l of the aligned block range that covers the row, so a pass is one
// fully coalesced 1 KiB load.  A row that does not start on a 16-byte boundary shares its first
// and last block with its neighbours: their elements are masked on the way in and those
// blocks are written back with byte stores, every other block with one dword store at whatever
// byte address it has (so the tensor may start anywhere on the 4-byte grid and the output
// anywhere at all).  The
// arithmetic is the slab kernels' (softmax_slab_math with 64 lanes per row).
// SLOTS is exactly the number of passes a row of this length needs at its worst alignment,
// ceil(B / 64) with B the most blocks it can touch: a row touches B or B - 1 blocks, so the
// blocks of passes 0 .. SLOTS-2 exist in every row, only the last pass clamps its block
// index (the last two do: one instruction), and only passes 0, SLOTS-2 and SLOTS-1 can hold a
// row's first or last block (element masks, byte stores).  No branch depends on the row
// length.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"
#include "plan.h"
#include "softmax_rows.h"

namespace iptq {

struct WideArgs {
    const int32_t *scores;   // the tensor's address rounded down to 16 bytes
    const int32_t *bias;     // NULL or 16-byte aligned, period * cols a multiple of 4 (base_off == 0 then)
    uint8_t *out;            // the output's address minus base_off (any byte address)
    int64_t rows;
    int32_t base_off;        // scores between the rounded-down address and the tensor: 0..3
    int32_t cols;            // >= 8 when cut_el != 0 (host)
    int32_t cut_el;          // scores in the tensor's final 16-byte block if the tensor ends off the
                             // 16-byte grid (the last row must not load that block whole), else 0
    int32_t post_mode;       // PM_NONE / PM_CLAMP127 / PM_GENERAL, applied to the packed bytes
    SoftmaxDev P;
};

// The same in 88 bytes instead of 208: a launch's arguments are written into device memory by the host,
// about 0.3 us for the difference, and a call of one image lasts 3 us.  What fits a few bits shares a
// word, and what follows from other fields is derived again.  (The fields have no room to spare and are not
// masked: tests/test_wide_arguments.py holds them against plan_softmax over its whole domain.)
struct WidePacked {
    const int32_t *scores, *bias;
    uint8_t *out;
    int32_t rows, cols;                               // rows < 2^31 (plan_softmax)
    int32_t i0;
    uint32_t magic;
    int32_t d_clamp;
    uint32_t divider;     // div8 or mg24, whichever the kernel takes
    uint32_t w0;          // n_shift 5, magic_sh 5, free 4, m_bits 5, p_shift 5, free 2, pre_mode 2, variant 2
    uint32_t w1;          // pre_s 6, pre_sh2 5, pre_rowconst 1, post_s 6, d2_sh 5, period_sh 5, base_off 2, cut_el 2
    uint32_t w2;          // pre_m 16, post_m 16 (signed)
    uint32_t w3;          // qmin 10 (signed), qmax 10 (signed), post_mode 2, post_xor 1
    int32_t post_zp;
    uint32_t pre_dmax, d2_magic;
    int32_t bias_period_rows;
    uint32_t period_magic;
};
IPTQ_HD WidePacked wide_pack(const WideArgs &A)
{
    const SoftmaxDev &P = A.P;
    WidePacked W;
    W.scores = A.scores; W.bias = A.bias; W.out = A.out;
    W.rows = (int32_t)A.rows; W.cols = A.cols;
    W.i0 = P.i0; W.magic = P.magic; W.d_clamp = P.d_clamp; W.divider = P.packed == 2 ? (uint32_t)P.div8 : P.mg24;
    W.w0 = (uint32_t)P.n_shift | (uint32_t)P.magic_sh << 5 | (uint32_t)P.m_bits << 14 |
           (uint32_t)P.p_shift << 19 | (uint32_t)P.pre_mode << 26 | (uint32_t)P.variant << 28;
    W.w1 = (uint32_t)P.pre_s | (uint32_t)P.pre_sh2 << 6 | (uint32_t)P.pre_rowconst << 11 | (uint32_t)P.post_s << 12 |
           (uint32_t)P.d2_sh << 18 | (uint32_t)P.period_sh << 23 | (uint32_t)A.base_off << 28 | (uint32_t)A.cut_el << 30;
    W.w2 = ((uint32_t)P.pre_m & 0xffffu) | (uint32_t)P.post_m << 16;
    W.w3 = ((uint32_t)P.qmin & 0x3ffu) | ((uint32_t)P.qmax & 0x3ffu) << 10 | (uint32_t)A.post_mode << 20 |
           (P.post_xor != 0 ? 1u << 22 : 0u);
    W.post_zp = P.post_zp; W.pre_dmax = P.pre_dmax; W.d2_magic = P.d2_magic;
    W.bias_period_rows = P.bias_period_rows; W.period_magic = P.period_magic;
    return W;
}
IPTQ_HD WideArgs wide_unpack(const WidePacked &W)
{
    WideArgs A;
    SoftmaxDev &P = A.P;
    A.scores = W.scores; A.bias = W.bias; A.out = W.out;
    A.rows = W.rows; A.cols = W.cols;
    A.base_off = (int32_t)(W.w1 >> 28 & 3u); A.cut_el = (int32_t)(W.w1 >> 30);
    A.post_mode = (int32_t)(W.w3 >> 20 & 3u);
    P.i0 = W.i0; P.magic = W.magic; P.d_clamp = W.d_clamp; P.div8 = (int32_t)W.divider; P.mg24 = W.divider;
    P.n_shift = (int32_t)(W.w0 & 31u); P.magic_sh = (int32_t)(W.w0 >> 5 & 31u);
    P.m_bits = (int32_t)(W.w0 >> 14 & 31u); P.p_shift = (int32_t)(W.w0 >> 19 & 31u);
    P.pre_mode = (int32_t)(W.w0 >> 26 & 3u); P.variant = (int32_t)(W.w0 >> 28 & 3u);
    P.i0n = P.i0 << P.n_shift;
    P.pre_s = (int32_t)(W.w1 & 63u); P.pre_sh2 = (int32_t)(W.w1 >> 6 & 31u); P.pre_rowconst = (int32_t)(W.w1 >> 11 & 1u);
    P.post_s = (int32_t)(W.w1 >> 12 & 63u); P.d2_sh = (int32_t)(W.w1 >> 18 & 31u); P.period_sh = (int32_t)(W.w1 >> 23 & 31u);
    P.pre_m = (int32_t)(W.w2 & 0xffffu); P.post_m = (int32_t)W.w2 >> 16;
    P.pre_mul = pre_mul_of(P.pre_m, P.pre_s);         // (pre_mode 1 alone uses them)
    P.pre_rnd = pre_rnd_of(P.pre_s);
    P.qmin = (int32_t)(W.w3 << 22) >> 22; P.qmax = (int32_t)(W.w3 << 12) >> 22;
    P.post_zp = W.post_zp;
    P.post_xor = (W.w3 >> 22 & 1u) != 0 ? kPostXor : 0u;
    P.pre_dmax = W.pre_dmax; P.d2_magic = W.d2_magic;
    P.bias_period_rows = W.bias_period_rows; P.period_magic = W.period_magic;
    P.packed = 0;                                     // not read by these kernels
    P.n_windows = P.group_rows = P.mask_period_rows = P.mperiod_sh = P.group_sh = 0;     // no mask in these kernels
    P.mperiod_magic = P.group_magic = 0;
    return A;
}

// PRE: the requantization in front folded into Eq. 6, as in the slab kernel (60,000 rows of 1025
// scores 52.6 us against 53.9 us).  Up to eight passes: with more the folded form needs so many
// registers that it is the slower one (12,000 rows of 3000 scores 33.2 against 32.3 us).
constexpr int kWideFoldMaxSlots = 8;
// Loads of the table in flight (add_table_blocks; 0: in the compiler's order).
constexpr int wide_table_ahead(int slots) { return slots == 8 || slots == 9 ? 8 : 0; }
template <int SLOTS, int MODE, int VARIANT, bool PRE>
__global__ void __launch_bounds__(256)
softmax_wide_kernel(WidePacked W)
{
    __shared__ uint8_t lut_all[4][kPostLutBytes];
    touch_kernel_arguments<sizeof(WidePacked)>();
    const WideArgs A = wide_unpack(W);
    const SoftmaxDev &P = A.P;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // the row index as a scalar
    const int64_t row = (int64_t)blockIdx.x * 4 + wv;
    if (row >= A.rows) return;                        // no workgroup barrier below

    uint8_t *lut = lut_all[wv];
    const int post_mode = A.post_mode;
    if (post_mode == PM_GENERAL) {
        const int p_max = 1 << (P.m_bits - P.p_shift);
        for (int p = lane; p <= p_max; p += 64) lut[p] = (uint8_t)post_dev<PM_GENERAL>((uint32_t)p, P);
        wave_lds_fence();
    }

    const int cols = A.cols;
    const int64_t e0 = row * cols + A.base_off;       // the row's first element on the 16-byte grid
    const int phi = (int)(e0 & 3);                    // its offset inside its 16-byte block
    const int nb = (phi + cols + 3) >> 2;             // blocks the row touches (wavefront-uniform)
    const i32x4 *src = reinterpret_cast<const i32x4 *>(A.scores) + (e0 >> 2);
    // the last row of a tensor that ends off the 16-byte grid: its final block is loaded
    // element by element below (wavefront-uniform case)
    const bool cut = A.cut_el != 0 && row == A.rows - 1;
    const int nb_whole = cut ? nb - 1 : nb;           // blocks that can be loaded whole, >= 1
    auto block_of = [&](int s, int n) {               // lanes beyond block n - 1 load it again
        const int b = s * 64 + lane;
        return s >= SLOTS - 2 ? min(b, n - 1) : b;
    };
    auto edge_slot = [](int s) { return s == 0 || s >= SLOTS - 2; };

    // ---- the row's blocks; every load is issued before the first use and none sits behind a
    // branch
    i32x4 v[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) v[s] = stream_load(src + block_of(s, nb_whole));
    if (cut) {
        const int32_t *last = reinterpret_cast<const int32_t *>(src + (nb - 1));
#pragma unroll
        for (int s = SLOTS >= 2 ? SLOTS - 2 : 0; s < SLOTS; ++s) {
            if (s * 64 + lane == nb - 1) {            // elements beyond cut_el are masked below
                v[s].x = last[0];
                if (A.cut_el > 1) v[s].y = last[1];
                if (A.cut_el > 2) v[s].z = last[2];
            }
        }
    }
    if (A.bias != nullptr) {
        // the bias row starts at the same offset inside a block (period * cols % 4 == 0)
        const int64_t eb = (int64_t)row_mod_period((uint32_t)row, P) * cols;
        const i32x4 *bsrc = reinterpret_cast<const i32x4 *>(A.bias) + (eb >> 2);
        if constexpr (wide_table_ahead(SLOTS) != 0) {
            add_table_blocks<SLOTS, wide_table_ahead(SLOTS)>(v, [&](int s) { return bsrc[block_of(s, nb)]; });
        } else {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const i32x4 bv = bsrc[block_of(s, nb)];
                v[s] = add_table_chunk(v[s], bv);
            }
        }
    }

    // ---- elements outside the row become "minus infinity"
    int32_t x[SLOTS][4];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        x[s][0] = v[s].x; x[s][1] = v[s].y; x[s][2] = v[s].z; x[s][3] = v[s].w;
        if (edge_slot(s)) {
            const int c0 = 4 * (s * 64 + lane) - phi;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((unsigned)(c0 + e) >= (unsigned)cols) x[s][e] = kI32Min;
        }
    }

    uint32_t w[SLOTS];                                // four probabilities per block, one per byte
    if constexpr (PRE) {
        int32_t mr = kI32Min;                         // the raw row maximum (the requantization is monotone)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) mr = max(mr, x[s][e]);
        mr = group_max_i32<64>(mr);
        if (__builtin_expect(pre_fold_low_row(mr, P), 0)) {
            // The clamp of the differences cannot tell masked scores from live ones: they take the
            // (wrapping) value whose difference is the clamp, where the exponential is 0.  Nothing
            // else of the folded form depends on where the row lies.
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    x[s][e] = x[s][e] == kI32Min ? (int32_t)((uint32_t)mr - P.pre_dmax) : x[s][e];
        }
        softmax_slab_math<64, SLOTS, MODE, VARIANT, PM_NONE, LaneGroupSum<64>, true>(
            x, w, mr, 0, false, lut, P, LaneGroupSum<64>(), pre_fold_row_constant(mr, P));
    } else {
    // ---- fused requantization of the scores (after the bias, before the maximum)
    pre_requant_registers<SLOTS>(x, P);

    // ---- Eq. 6: row maximum
    int32_t mx = kI32Min;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = max(mx, x[s][e]);
    mx = group_max_i32<64>(mx);

    const int32_t D = P.d_clamp;
    const bool low_row = mx < kI32Min + D;            // wavefront-uniform here; see softmax_rows_kernel
    const int32_t lower = low_row ? kI32Min : mx - D;
    softmax_slab_math<64, SLOTS, MODE, VARIANT, PM_NONE>(x, w, mx, lower, low_row, lut, P);
    }

    // ---- post step on the packed bytes (a probability is at most 128)
    if (post_mode == PM_CLAMP127) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) w[s] = clamp127_bytes(w[s]);
    } else if (post_mode == PM_GENERAL) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) w[s] = post_lut_gather(lut, w[s]);
    } else if (P.post_xor != 0) {                     // signed output around the zero-point -128
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) w[s] ^= P.post_xor;
    }

    // ---- write back: whole blocks as dwords, the two shared edge blocks byte by byte
    uint8_t *dst8 = A.out + (e0 - phi);               // the byte of the row's first block
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int b = s * 64 + lane;
        const int c0 = 4 * b - phi;
        if (!edge_slot(s)) {                          // every lane's block lies inside the row
            stream_store_bytes4(w[s], dst8 + 4 * b);
        } else if (b < nb) {
            if (c0 >= 0 && c0 + 3 < cols) {
                stream_store_bytes4(w[s], dst8 + 4 * b);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((unsigned)(c0 + e) < (unsigned)cols) dst8[4 * b + e] = (uint8_t)(w[s] >> (8 * e));
            }
        }
    }
}

// LDS to ask for beside a kernel's own (less than 1 KB), so that no more than `most` of its workgroups
// share a compute unit; LDS is handed out in units of 1280 bytes.  0: no bound.
constexpr size_t lds_for_at_most(int most) { return most != 0 ? 160 * 1024 / most / 1280 * 1280 - 1024 : 0; }

// Most workgroups per compute unit in a long launch, where registers would allow more of them than is
// good: with that many rows in flight it takes longer.  0: no bound; the numbers of passes without one
// gain nothing by it or lose.
// More than 28 million scores: 30 to 45 million in rows of 1500 25.9 us against 26.3 without the bound,
// of 2000 26.2 against 26.7, of 2200 38.2 against 39.1, of 2950 38.8 against 39.3.  At 25 to 28 million
// both take the same time, and 15 million are faster with all that fit (rows of 2200 14.6 us against
// 15.2, of 2950 14.9 against 16.0).
// More than 50 million, with a table or a requantization in front 60 (56 million of 4096 with a table 51.9 us
// with what fits, 54.2 with two; of 1500 requantized 46.7 and 47.6 with four): 90 / 190 million in rows of 1500
// 72.7 / 150 us with four against 73.6 / 155 with five, of 2500 73.8 / 153 with four against 75.0 / 156 without a
// bound, of 3800 73.8 / 150 with two against 75.8 / 157, of 4096 72.4 / 148 against 78.1 / 162 (52 / 60 million 44.3 /
// 50.1 against 45.7 / 52.2); at 45 million none is more than 2 % faster than what fits.  Rows of 3330 79.1 / 155.0
// with three, 81.6 / 159.9 with two, 79.6 / 156.8 without; of 3600 78.0 / 151.4, 78.8 / 153.2 and 79.4 / 155.7; from
// 3760 on, and with a table (3400 105.7 us at 115 million against 108.1), two are as good or better.  Four passes,
// which shorter arithmetic had made up to 4 % slower: rows of 880 70.6 / 146.6 with six against 72.0 / 150.7
// without, of 900 72.7 / 152.4 against 73.8 / 155.2, of 960 70.8 / 146.3 with five against 72.7 / 154.5, of 1000 71.6 /
// 149.0 against 73.6 / 157.0 (with a table 80.5 / 167.5 against 81.9 / 172.6, second degree 71.7 / 148.1 against 73.1 /
// 155.6), of 1001 151.9 with six against 152.8; below 820 six are slower (800 72.9 us against 69.9), and so are
// six and five where more arithmetic fills the time (900 of the second degree 151.2 against 150.9, 1000 with a
// requantization in front 95.2 against 92.9 at 115 million).
constexpr int wide_most_workgroups(int slots, int32_t cols, bool very_long, bool bias, bool pre, bool degree2)
{
    if (very_long && slots >= 14) return slots == 16 || cols >= 3760 || bias ? 2 : 3;
    if (very_long && slots == 4 && cols >= 820 && !pre) {
        if (cols % 4 == 0 && cols >= 950) return 5;
        return !bias && !degree2 && (cols % 4 == 0 || cols >= 950) ? 6 : 0;
    }
    if (very_long && (slots == 6 || slots == 10)) return 4;
    return slots >= 5 && slots <= 7 ? 5 : (slots == 8 || slots == 9 || slots == 11 || slots == 12 ? 4 : 0);
}
inline size_t wide_extra_lds(int slots, const WideArgs &A)
{
    const int64_t scores = A.rows * A.cols;
    const bool bias = A.bias != nullptr, pre = A.P.pre_mode != 0;
    if (scores <= 28 * 1000 * 1000) return 0;
    return lds_for_at_most(wide_most_workgroups(slots, A.cols, scores > (bias || pre ? 60 : 50) * 1000 * 1000, bias, pre,
                                                A.P.variant == 2));
}

// mode: SoftmaxDev::packed
template <int SLOTS>
static void wide_launch_s(const WideArgs &A, int mode, dim3 grid, hipStream_t stream)
{
    const size_t lds = wide_extra_lds(SLOTS, A);
    const WidePacked W = wide_pack(A);
    if constexpr (SLOTS <= kWideFoldMaxSlots) {
        if (A.P.pre_rowconst != 0) {                  // packed arithmetic and a first-degree exponential
            if (mode == 2 && A.P.variant == 0) launch_kernel((softmax_wide_kernel<SLOTS, 2, 0, true>), grid, dim3(256), lds, stream, W);
            else if (mode == 2) launch_kernel((softmax_wide_kernel<SLOTS, 2, 1, true>), grid, dim3(256), lds, stream, W);
            else if (A.P.variant == 0) launch_kernel((softmax_wide_kernel<SLOTS, 1, 0, true>), grid, dim3(256), lds, stream, W);
            else launch_kernel((softmax_wide_kernel<SLOTS, 1, 1, true>), grid, dim3(256), lds, stream, W);
            return;
        }
    }
#define IPTQ_WIDE_LAUNCH(MODE)                                                                    \
    do {                                                                                          \
        if (A.P.variant == 0) launch_kernel((softmax_wide_kernel<SLOTS, MODE, 0, false>), grid, dim3(256), lds, stream, W);      \
        else if (A.P.variant == 1) launch_kernel((softmax_wide_kernel<SLOTS, MODE, 1, false>), grid, dim3(256), lds, stream, W); \
        else launch_kernel((softmax_wide_kernel<SLOTS, MODE, 2, false>), grid, dim3(256), lds, stream, W);                       \
    } while (0)
    if (mode == 0) IPTQ_WIDE_LAUNCH(0);
    else if (mode == 1) IPTQ_WIDE_LAUNCH(1);
    else IPTQ_WIDE_LAUNCH(2);
#undef IPTQ_WIDE_LAUNCH
}

// one translation unit per group of pass counts; each returns false for a count it does not hold
bool wide_launch_p1_6(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);
bool wide_launch_p7_10(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);
bool wide_launch_p11_13(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);
bool wide_launch_p14_16(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);

#define IPTQ_WIDE_CASE(S)                                                                         \
    case S: wide_launch_s<S>(A, mode, grid, stream); return true;

}  // namespace iptq
