// Integer softmax (Section 4.4, Eq. 6-15) for row lengths that have no compiled
// instantiation: the slab scheme and the register-resident arithmetic of the
// fixed-row-length kernel (softmax_rows.h) with the row length as a run-time value.  What is
// fixed at compile time is the lane layout: K lanes per row and exactly SLOTS 16-byte blocks
// per lane, SLOTS = ceil(B / K) with B the most blocks a row of that length can touch.  That
// pins down everything the code's shape depends on:
//   * a row touches B or B - 1 blocks, so the blocks of slots 0 .. SLOTS-2 exist in every
//     row and only the last slot's block index needs a clamp;
//   * a row's last (possibly cut) block lies in slot SLOTS-2 or SLOTS-1, its first in slot 0:
//     element masks and byte-wise output are confined to those three slots;
//   * the slab is SLOTS or SLOTS-1 passes of 64 chunks, of which all but the last two are
//     full: only those two clamp their chunk index.
// So the kernel has no branch that depends on the row length apart from lane predicates on
// LDS writes; the host instantiates one kernel per (K, SLOTS) and picks by row length.
#pragma once

#include <hip/hip_runtime.h>

#include <stddef.h>

#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "plan.h"
#include "softmax_rows.h"

namespace iptq {

struct DynArgs {
    const int32_t *scores;
    const int32_t *bias;
    uint8_t *out;
    uint32_t n_slabs, last_row0;      // as in SoftmaxItem, and so is few_rows
    int32_t few_rows;
    int32_t cols;
    int32_t wave_lds;     // LDS bytes per wavefront: slab (16-byte multiple) + post table
    int32_t post_mode;    // PM_NONE / PM_CLAMP127 / PM_GENERAL, applied to the packed bytes
    // with an additive table: the wavefronts of a workgroup take slabs share_q apart, which read
    // the same table rows (see SoftmaxItem); 0: consecutive slabs
    uint32_t share_q, share_magic;
    int32_t share_sh;
    uint32_t wpb;         // wavefronts per workgroup (here and not from the launch's implicit arguments,
                          // which lie behind the lines touched at entry: a cold read in front of all else)
    SoftmaxDev P;
    // (last, so that a kernel without a mask does not touch them)
    // per-window mask, at most one form: int32 entries (MASKKIND 1) or one bit per key (2)
    const int32_t *mask;
    const uint64_t *mask_bits;
    uint32_t cols_magic;  // query of a row (row mod cols) by multiply-high, cols >= 2
    int32_t cols_sh;
};

constexpr int kDynBatchMax = 14;                      // calls per launch of the batch kernel
struct DynBatch;

// Four entries of a row-major table of `total` entries from entry `idx` on, where idx may lie up
// to three entries before the table or run past its end (the first and last block of a row that
// starts off the 16-byte grid): the load is moved inside the table and the entries that exist are
// shifted back to their places (a rare case, one wavefront-uniform branch); the others are
// arbitrary.  total >= 4.
IPTQ_DEV i32x4 table_block_at(const int32_t *table, int32_t idx, int32_t total)
{
    const int32_t a = clamp_i32(idx, 0, total - 4);
    i32x4 m = load_i32x4_at(table, 4u * (uint32_t)a);
    const int32_t d = idx - a;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(d != 0) != 0, 0)) {
        const i32x4 t = m;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t k = e + d;
            m[e] = k == 0 ? t.x : (k == 1 ? t.y : (k == 2 ? t.z : t.w));
        }
    }
    return m;
}

// MASKKIND: 0 no mask; 1 int32 entries, 2 one bit per key: the per-window mask of shifted-window
// attention, for windows of any size.  Both forms are
// applied to the registers once the row has been read back from LDS (the int32 entries load per
// block straight into the lane that needs them; a mask row is shared by `heads` rows and comes out
// of L1/L2), so the copy loop stays the one of the unmasked kernel.  What bounds it is still HBM,
// with the mask's lane-ops (two per score packed, four as int32) next.  Launches back to back in a
// graph, random masks, a bias table, Bit-exp: 524,288 rows of 8 x 8-token windows 31.5 us packed and
// 34.7 us as int32 entries, 29.6 us without a mask, 254 us in the three-pass kernel; 16 x 16 tokens
// (262,144 rows) 60.0 / 63.8 / 54.7 / 370 us.  At 49 and 144 tokens the compiled row lengths stay faster
// (589,824 rows of 144: 67.6 / 78.7 us against 85.9 / 91.9 us here).
//
// VARIANT is a template argument because every launch starts with a cold instruction cache: with a
// branch over the three exponentials 122,880 rows of 100 scores with a table took 16.3 us against
// 15.7 us (a launch of this kernel has one set of parameters, so nothing needs the branch).  In 32-bit
// lanes the branch costs between nothing and 4 % (122,880 x 100 15.1 us against 14.5, 30,000 x 401 16.2
// against 15.9, with a mask up to 2 %) and would save a tenth of the library's size.
//
// PRE: the requantization in front folded into Eq. 6 where the parameters allow it
// (SoftmaxDev::pre_rowconst, see softmax_rows_body): 153,984 rows of 401 scores 53.4 us (Bit-exp) and
// 53.6 us (Shiftmax), what they take without a requantization, against 54.6 and 53.9 us.
// (wg: this workgroup's index within the call; VARIANT < 0: by the parameters)
template <int K, int SLOTS, int MODE, int MASKKIND, int VARIANT, bool PRE>
IPTQ_DEV void softmax_rowsdyn_body(const DynArgs &A, uint32_t wg)
{
    constexpr int RPW = 64 / K;                       // rows per wavefront, a multiple of 4
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn_lds[];
    const SoftmaxDev &P = A.P;
    const int lane = threadIdx.x & 63;
    // (a scalar: the slab, its table offsets and every test on them then run on the scalar unit)
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t wpb = A.wpb;
    uint32_t slab = wg * wpb + (uint32_t)wv;
    if (A.share_q != 0) {
        const uint32_t g = mulhi_u32(wg, A.share_magic) >> A.share_sh;
        slab = g * (wpb * A.share_q) + (uint32_t)wv * A.share_q + (wg - g * A.share_q);
    }
    if (slab >= A.n_slabs) return;                    // no workgroup barrier below

    const int cols = A.cols;
    const int slab_el = RPW * cols;                   // multiple of 4
    const int in_chunks = slab_el >> 2;               // in (64 (SLOTS-2), 64 SLOTS]
    uint8_t *lds = dyn_lds + wv * A.wave_lds;
    uint8_t *lut = lds + A.wave_lds - kPostLutBytes;
    const int post_mode = A.post_mode;
    if (post_mode == PM_GENERAL) {                    // ordered before its use by the fences below
        const int p_max = 1 << (P.m_bits - P.p_shift);
        for (int p = lane; p <= p_max; p += 64) lut[p] = (uint8_t)post_dev<PM_GENERAL>((uint32_t)p, P);
    }
    const uint32_t row0 = min(slab * (uint32_t)RPW, A.last_row0);
    const int32_t *src1 = A.scores + (uint64_t)row0 * (uint32_t)cols;
    const int32_t *__restrict__ bias = A.bias;
    const bool partial = A.few_rows != 0;
    const int valid_el = (partial ? A.few_rows : RPW) * cols;

    // ---- the mask of this lane's blocks, in flight with the scores.  Packed form: the bits of
    // slot s start at key 4 (s K + j) - phi; one 4-byte load at the byte that holds that key
    // (moved inside the mask row where it would leave it) covers the bits of GROUP slots.  (8-byte
    // words take half the loads and two quarter-rate 64-bit shifts each: 204,800 rows of 20 x 20
    // tokens 102 us against 85 us.)
    constexpr int GROUP = K == 1 ? 6 : (K == 2 ? 3 : (K == 4 ? 2 : 1));
    constexpr int NG = (SLOTS + GROUP - 1) / GROUP;
    static_assert(4 * K * (GROUP - 1) + 4 + 7 <= 32, "the bits of a group of slots at any offset inside a byte");
    uint32_t mask_word[MASKKIND == 2 ? NG : 1];
    i32x4 mask_block[MASKKIND == 1 ? SLOTS : 1];
    if (MASKKIND != 0) {
        const int lr = lane / K, j = lane % K, phi = (lr * cols) & 3;    // as below
        // rows past the end of a partial slab take the last row's mask (never stored)
        const uint32_t row = row0 + (uint32_t)(partial ? min(lr, A.few_rows - 1) : lr);
        uint32_t rm = 0;
        if (P.mask_period_rows >= 2)
            rm = row - (mulhi_u32(row, P.mperiod_magic) >> P.mperiod_sh) * (uint32_t)P.mask_period_rows;
        const uint32_t w = P.group_rows >= 2 ? mulhi_u32(rm, P.group_magic) >> P.group_sh : rm;
        uint32_t q = rm - w * (uint32_t)P.group_rows;
        if (cols >= 2) q -= (mulhi_u32(q, A.cols_magic) >> A.cols_sh) * (uint32_t)cols;
        else q = 0;
        const uint32_t mrow = w * (uint32_t)cols + q;
        if (MASKKIND == 1) {
            const int32_t total = P.n_windows * cols * cols;     // below 2^30 (host)
            const int32_t first = (int32_t)(mrow * (uint32_t)cols) + 4 * j - phi;
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                mask_block[s] = (s == 0 || s >= SLOTS - 2)      // only there can a block leave the table
                    ? table_block_at(A.mask, first + 4 * s * K, total)
                    : load_i32x4_at(A.mask + (4 * s * K - 4), 4u * (uint32_t)(first + 4));   // first >= -3
        } else {
            const int32_t row_bytes = 8 * ((cols + 63) >> 6);
            const uint32_t row_at = mrow * (uint32_t)row_bytes;          // below 2^31 (host)
            const int32_t sh = 4 * j - phi;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int32_t p = 4 * K * GROUP * g + sh;
                if (K >= 8 && g >= 1 && g <= NG - 3) {
                    // inside the mask row for every lane (the blocks of slots 0 .. SLOTS-2 exist in
                    // every row): one address for all of these (sh >= -3: one byte is moved from
                    // the fixed offset to the unsigned one), one shift
                    mask_word[g] = load_u32_at(A.mask_bits, row_at + (uint32_t)((sh >> 3) + 1), 4 * K * g / 8 - 1) >> (sh & 7);
                } else {
                    const int32_t at = min(g == 0 ? max(p >> 3, 0) : p >> 3, row_bytes - 4);
                    const int32_t d = p - 8 * at;     // negative only for the first block of a row off the grid
                    const uint32_t v = load_u32_at(A.mask_bits, row_at + (uint32_t)at, 0);
                    mask_word[g] = v >> (d & 31);
                    if (g == 0) mask_word[g] = d < 0 ? v << (-d & 31) : mask_word[g];
                }
            }
        }
    }

    // ---- flat copy of the slab into LDS, bias added on the way.  Every load is issued before
    // the first LDS write and none sits behind a branch: in the last two passes the lanes
    // beyond the slab's last chunk load that chunk again and write it to its place again.
    // (with one lane per row a slab has 64 rows and the table may have as few as 32: two wraps)
    auto wrap = [](uint32_t o, uint32_t pe) -> uint32_t {
        if (o >= pe) o -= pe;
        if (K == 1 && o >= pe) o -= pe;
        return o;
    };
    auto add_bias = [](i32x4 v, const i32x4 bv) {
        v = add_table_chunk(v, bv);
        return v;
    };
    // With a table the scores are added with the saturating sum alone, which is the exact value
    // unless a score or an entry is INT32_MIN, and the smallest operand is tracked beside it (two
    // lane-ops per score instead of four); returns whether any lane met INT32_MIN, in which case
    // the caller copies the slab in again with the exact rule.
    // LINEAR: the slab's table rows lie one after the other like the slab itself, so a chunk of them sits at
    // the chunk's own offset from a scalar base and needs no address of its own (28 vector instructions per
    // wavefront less: 189,728 rows of 11 x 11 tokens with an int32 mask 29.4 -> 28.8 us, 248,430 of 13 x 13 with a
    // packed one 43.5 -> 42.5, 15,876 of 9 x 9 8.1 -> 7.85).
    auto copy_in = [&](auto bias_tag, auto straddle_tag, auto linear_tag) -> bool {
        constexpr bool BIAS = decltype(bias_tag)::value;
        constexpr bool LINEAR = decltype(linear_tag)::value;
        i32x4 lowest = {0, 0, 0, 0};
        // the additive table's end falls inside this slab and inside a chunk, which takes entries from both
        // ends of the table
        constexpr bool STRADDLE = decltype(straddle_tag)::value;
        i32x4 *lds4 = reinterpret_cast<i32x4 *>(lds);
        const int last = in_chunks - 1;
        auto chunk_of = [&](int i) {
            const int idx = i * 64 + lane;
            return i >= SLOTS - 2 ? min(idx, last) : idx;
        };
        uint32_t boff = 0;
        if (BIAS) boff = row_mod_period(row0, P) * (uint32_t)cols;
        const uint32_t pe = (uint32_t)P.bias_period_rows * (uint32_t)cols;
        i32x4 first4 = {0, 0, 0, 0};
        if (STRADDLE) first4 = load_i32x4(bias);
        auto bias_chunk = [&](int i) {
            if (LINEAR) return load_i32x4_at(bias + boff, 16u * (uint32_t)chunk_of(i));
            const uint32_t o = wrap(boff + 4u * (uint32_t)chunk_of(i), pe);
            return load_i32x4(bias + (STRADDLE ? min(o, pe - 4u) : o));
        };
        // With a table every load is in flight before the first is waited for, in the order of the chunks, so
        // that a chunk can be added up as it arrives (see softmax_rows_body): 62,720 rows of 196 scores 13.5 ->
        // 13.1 us, 100,352 of 256 22.9 -> 22.3, 93,600 of 25 5.75 -> 5.5, 524,288 of 64 with a packed mask 31.0 ->
        // 30.4.  Not beside an int32 mask, whose entries are in flight as well: there four table loads behind
        // all the scores' are faster (345,600 rows of 100 37.3 us against 38.1, 189,728 of 121 28.3 against 29.0).
        constexpr bool IN_ORDER = MASKKIND != 1;
        constexpr int AHEAD = IN_ORDER || SLOTS < 4 ? SLOTS : 4;
        i32x4 v[SLOTS], bv[BIAS ? AHEAD : 1];
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            v[i] = stream_load_i32x4(src1 + 4 * chunk_of(i));
            if (BIAS && IN_ORDER) {
                bv[BIAS ? i : 0] = bias_chunk(i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (BIAS && !IN_ORDER) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) bv[BIAS ? i : 0] = bias_chunk(i);
        }
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            if (BIAS) {
                i32x4 b = bv[BIAS ? i % AHEAD : 0];
                if (STRADDLE) b = bias_chunk_wrapped(b, wrap(boff + 4u * (uint32_t)chunk_of(i), pe), pe, first4);
                v[i] = add_tracking_lowest(v[i], b, lowest);
                if (i + AHEAD < SLOTS) bv[BIAS ? i % AHEAD : 0] = bias_chunk(i + AHEAD);
            }
            lds4[chunk_of(i)] = v[i];
        }
        wave_lds_fence();
        return BIAS && __builtin_amdgcn_ballot_w64(min(min(lowest.x, lowest.y), min(lowest.z, lowest.w)) == kI32Min) != 0;
    };
    // a partial slab (a call of fewer rows than a slab has), and a slab that holds an INT32_MIN operand:
    // guarded loads and the exact addition, chunk by chunk
    auto copy_in_partial = [&]() {
        i32x4 *lds4 = reinterpret_cast<i32x4 *>(lds);
        uint32_t boff = 0;
        if (bias != nullptr) boff = row_mod_period(row0, P) * (uint32_t)cols;
        const uint32_t pe = (uint32_t)P.bias_period_rows * (uint32_t)cols;
        for (int idx = lane; idx < in_chunks; idx += 64) {
            i32x4 v;
            if (4 * idx + 3 < valid_el) {
                v = stream_load_i32x4(src1 + 4 * idx);
            } else {
                v = (i32x4){0, 0, 0, 0};
                if (4 * idx < valid_el) v.x = src1[4 * idx];
                if (4 * idx + 1 < valid_el) v.y = src1[4 * idx + 1];
                if (4 * idx + 2 < valid_el) v.z = src1[4 * idx + 2];
            }
            if (bias != nullptr) {
                const uint32_t o = wrap(boff + 4u * (uint32_t)idx, pe);
                v = add_bias(v, bias_chunk_wrapping(bias, o, pe, load_i32x4(bias)));
            }
            lds4[idx] = v;
        }
        wave_lds_fence();
    };
    if (__builtin_expect(partial, 0)) copy_in_partial();
    else if (bias == nullptr) copy_in(std::false_type{}, std::false_type{}, std::false_type{});
    else {
        const uint32_t pe = (uint32_t)P.bias_period_rows * (uint32_t)cols;
        const uint32_t boff = row_mod_period(row0, P) * (uint32_t)cols;
        bool redo;
        if (boff + (uint32_t)slab_el <= pe) redo = copy_in(std::true_type{}, std::false_type{}, std::true_type{});
        else if (((boff | pe) & 3u) != 0) redo = copy_in(std::true_type{}, std::true_type{}, std::false_type{});
        else redo = copy_in(std::true_type{}, std::false_type{}, std::false_type{});
        if (__builtin_expect(redo, 0)) copy_in_partial();
    }

    // ---- this lane's blocks; elements outside the row become "minus infinity"
    const int lr = lane / K;                          // row inside the slab
    const int j = lane % K;                           // lane inside the row
    const int e_r = lr * cols;                        // first element of the row in the slab
    const int b_r = e_r >> 2;                         // its 16-byte block
    const int phi = e_r & 3;                          // and its offset inside that block
    const int nb = (phi + cols + 3) >> 2;             // blocks the row touches
    auto edge_slot = [](int s) { return s == 0 || s >= SLOTS - 2; };
    int32_t x[SLOTS][4];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int b = s * K + j;
        // a block beyond the row's last one (last slot only) is read from the last one and
        // masked entirely below: no lane-divergent branch around the LDS read
        const int bb = s == SLOTS - 1 ? min(b, nb - 1) : b;
        const i32x4 v = reinterpret_cast<const i32x4 *>(lds)[b_r + bb];
        x[s][0] = v.x; x[s][1] = v.y; x[s][2] = v.z; x[s][3] = v.w;
        if (edge_slot(s)) {
            const int c0 = 4 * b - phi;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((unsigned)(c0 + e) >= (unsigned)cols) x[s][e] = kI32Min;
        }
    }
    wave_lds_fence();                                 // the slab area is reused for the output

    // Most slabs lie in windows that the shift leaves whole: nothing of theirs is masked, and the lane-ops
    // are left out (9 x 9 tokens, 20 images, 36 windows, four heads 20.7 us packed against 21.9 with
    // them, 22.5 against 23.2 as int32 entries; 14 x 14 tokens 37.5 against 39.4 as int32 entries).
    bool any_masked = false;                          // wavefront-uniform
    if (MASKKIND != 0) {
        uint32_t any = 0;
        if (MASKKIND == 1) {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) any |= (uint32_t)(mask_block[s].x | mask_block[s].y | mask_block[s].z | mask_block[s].w);
        } else {
#pragma unroll
            for (int g = 0; g < NG; ++g) any |= mask_word[g];
        }
        any_masked = __builtin_amdgcn_ballot_w64(any != 0) != 0;
    }
    if (MASKKIND == 1 && any_masked) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[s][e] = add_table_entry(x[s][e], mask_block[s][e]);
    }
    if (MASKKIND == 2 && any_masked) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int pos = 4 * K * (s % GROUP) + e;          // compile-time position in the group's word
                const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int32_t)mask_word[s / GROUP], pos, 1);
                x[s][e] = select_bits_i32(m, kI32Min, x[s][e]);
            }
    }

    uint32_t w[SLOTS];                                // four probabilities per block, one per byte
    if constexpr (PRE) {
        int32_t mr = kI32Min;                         // the raw row maximum (the requantization is monotone)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) mr = max(mr, x[s][e]);
        mr = group_max_i32<K>(mr);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(pre_fold_low_row(mr, P)) != 0, 0)) {
            // The clamp of the differences cannot tell masked scores from live ones: they take the
            // (wrapping) value whose difference is the clamp, where the exponential is 0.  Nothing
            // else of the folded form depends on where the row lies.
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    x[s][e] = x[s][e] == kI32Min ? (int32_t)((uint32_t)mr - P.pre_dmax) : x[s][e];
        }
        softmax_slab_math<K, SLOTS, MODE, VARIANT, PM_NONE, LaneGroupSum<K>, true>(
            x, w, mr, 0, false, lut, P, LaneGroupSum<K>(), pre_fold_row_constant(mr, P));
    } else {
    // ---- fused requantization of the scores (after the bias, before the maximum)
    pre_requant_registers<SLOTS>(x, P);

    // ---- Eq. 6: row maximum
    int32_t mx = kI32Min;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = max(mx, x[s][e]);
    mx = group_max_i32<K>(mx);

    const int32_t D = P.d_clamp;
    const bool low_row = mx < kI32Min + D;            // see softmax_rows_kernel
    const int32_t lower = low_row ? kI32Min : mx - D;
    const bool any_low = __builtin_amdgcn_ballot_w64(low_row) != 0;

    if (VARIANT == 0 || (VARIANT < 0 && P.variant == 0))
        softmax_slab_math<K, SLOTS, MODE, 0, PM_NONE>(x, w, mx, lower, any_low, lut, P);
    else if (VARIANT == 1 || (VARIANT < 0 && P.variant == 1))
        softmax_slab_math<K, SLOTS, MODE, 1, PM_NONE>(x, w, mx, lower, any_low, lut, P);
    else
        softmax_slab_math<K, SLOTS, MODE, 2, PM_NONE>(x, w, mx, lower, any_low, lut, P);
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

    // ---- assemble the slab's bytes in LDS
    uint32_t *lds32 = reinterpret_cast<uint32_t *>(lds);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int b = s * K + j;
        if (!edge_slot(s)) {                          // every lane's block lies inside its row
            lds32[b_r + b] = w[s];
        } else if (b < nb) {
            const int c0 = 4 * b - phi;
            if (c0 >= 0 && c0 + 3 < cols) {
                lds32[b_r + b] = w[s];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((unsigned)(c0 + e) < (unsigned)cols)
                        lds[4 * (b_r + b) + e] = (uint8_t)(w[s] >> (8 * e));
            }
        }
    }
    wave_lds_fence();

    // ---- flat, fully coalesced store (byte stores at the end of a partial slab)
    uint8_t *dst8 = A.out + (uint64_t)row0 * (uint32_t)cols;
    auto copy_out = [&](auto tag) {
        constexpr bool PARTIAL = decltype(tag)::value;
        if ((slab_el & 15) == 0) {
            const int n16 = slab_el >> 4;
#pragma unroll
            for (int i = 0; i < (SLOTS + 3) / 4; ++i) {
                const int idx = i * 64 + lane;
                if (idx < n16) {
                    if (!PARTIAL || 16 * idx + 15 < valid_el) {
                        stream_store_bytes16(reinterpret_cast<const u32x4 *>(lds)[idx], dst8 + 16 * idx);
                    } else {
#pragma unroll 1
                        for (int b = 16 * idx; b < valid_el && b < 16 * idx + 16; ++b) dst8[b] = lds[b];
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                const int idx = i * 64 + lane;
                if (idx < in_chunks) {
                    if (!PARTIAL || 4 * idx + 3 < valid_el) {
                        stream_store_bytes4(lds32[idx], dst8 + 4 * idx);
                    } else {
#pragma unroll 1
                        for (int b = 4 * idx; b < valid_el && b < 4 * idx + 4; ++b) dst8[b] = lds[b];
                    }
                }
            }
        }
    };
    if (__builtin_expect(partial, 0)) copy_out(std::true_type{});
    else copy_out(std::false_type{});
}

// Wavefronts per SIMD that an unmasked kernel is held to.  Every form gets by with eight registers per block
// of a lane and about 20 more; since a table's loads are all in flight the scheduler, left to itself, takes up to 29
// beyond that for the second degree's arithmetic (6 to 8 blocks, also in a call without a table), which costs up
// to two wavefronts per SIMD (up to 7 blocks six are enough; seven at 6 blocks gain nothing, 400,000 rows of 81
// 27.5 us against 27.1): 150,528 rows of 196 scores of the second degree 26.3 us, 25.3 held to six, 120,000 of
// 401 43.0 and 41.2, 250,880 of 196 with a table 44.3 and 42.6; the first degree the same.
constexpr int rowsdyn_least_waves(int slots, int maskkind)
{
    return maskkind != 0 ? 1 : slots <= 7 ? 6 : 512 / (8 * slots + 24);
}

template <int K, int SLOTS, int MODE, int MASKKIND, int VARIANT, bool PRE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(rowsdyn_least_waves(SLOTS, MASKKIND))))
softmax_rowsdyn_kernel(DynArgs A)
{
    touch_kernel_arguments<MASKKIND == 0 ? offsetof(DynArgs, mask) : sizeof(DynArgs)>();
    softmax_rowsdyn_body<K, SLOTS, MODE, MASKKIND, VARIANT, PRE>(A, blockIdx.x);
}

// Several calls of one row length (the layers of a sweep) in one launch: packed arithmetic, no mask
// and no requantization in front; the variant is a wavefront-uniform branch.  Launched one by one such
// calls cost a launch each and its edges: 12 calls of 2303 x 145 scores and a GELU launch of 12 times 145 x 384
// values take 59 us call after call, 10.4 through this kernel; 5 of 1007 x 196 28.8 and 9.2; 2 of
// 13000 x 196 16.6 and 13.0.  Calls that each fill the chip gain their edges still: 2 of 100,000 x 196
// 36.7 and 34.2 (second degree 37.1 and 34.4), 2 of 200,000 x 64 with a table 28.3 and 24.4, 4 of
// 40,000 x 600 of the second degree 92.8 and 80.1.
struct DynBatch {
    BatchHead head;
    DynArgs item[kDynBatchMax];
};
static_assert(kDynBatchMax <= BatchHead::kMost && sizeof(DynBatch) <= 4096, "kernel arguments are limited to 4 KiB");
template <int K, int SLOTS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(rowsdyn_least_waves(SLOTS, 0))))
softmax_rowsdyn_batch_kernel(DynBatch B)
{
    const Problem p = problem_of(B.head, blockIdx.x);
    // (an item's 248 bytes start anywhere in a line, so that of 6 of the 14 the last line, the end of the plan's
    // constants, is not touched; with items of 256 bytes 421 batches of 2 to 14 problems take the same on average, 300
    // rows of 100 and 145 scores 2 % more)
    touch_kernel_arguments<offsetof(DynArgs, mask)>((uint32_t)offsetof(DynBatch, item) + p.index * (uint32_t)sizeof(DynArgs));
    softmax_rowsdyn_body<K, SLOTS, 2, 0, -1, false>(B.item[p.index], p.wg);
}

// mode: SoftmaxDev::packed
template <int K, int SLOTS>
static void rowsdyn_launch_ks(const DynArgs &A, int mode, dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
#define IPTQ_ROWSDYN_LAUNCH(MODE, MASKKIND)                                                       \
    do {                                                                                          \
        if (A.P.variant == 0) launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, MODE, MASKKIND, 0, false>), grid, block, lds, stream, A);      \
        else if (A.P.variant == 1) launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, MODE, MASKKIND, 1, false>), grid, block, lds, stream, A); \
        else launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, MODE, MASKKIND, 2, false>), grid, block, lds, stream, A);                       \
    } while (0)
    // pre_rowconst: packed arithmetic and a first-degree exponential
    if (A.P.pre_rowconst != 0 && A.mask == nullptr && A.mask_bits == nullptr) {
        if (mode == 2 && A.P.variant == 0) launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, 2, 0, 0, true>), grid, block, lds, stream, A);
        else if (mode == 2) launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, 2, 0, 1, true>), grid, block, lds, stream, A);
        else if (A.P.variant == 0) launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, 1, 0, 0, true>), grid, block, lds, stream, A);
        else launch_kernel((softmax_rowsdyn_kernel<K, SLOTS, 1, 0, 1, true>), grid, block, lds, stream, A);
        return;
    }
#define IPTQ_ROWSDYN_LAUNCH_MASK(MODE)                                                            \
    do {                                                                                          \
        if (A.mask != nullptr) IPTQ_ROWSDYN_LAUNCH(MODE, 1);                                      \
        else if (A.mask_bits != nullptr) IPTQ_ROWSDYN_LAUNCH(MODE, 2);                            \
        else IPTQ_ROWSDYN_LAUNCH(MODE, 0);                                                        \
    } while (0)
    if (mode == 0) IPTQ_ROWSDYN_LAUNCH_MASK(0);
    else if (mode == 1) IPTQ_ROWSDYN_LAUNCH_MASK(1);
    else IPTQ_ROWSDYN_LAUNCH_MASK(2);
#undef IPTQ_ROWSDYN_LAUNCH_MASK
#undef IPTQ_ROWSDYN_LAUNCH
}

// One launcher per group of layouts, each defined in its own translation unit so that the
// instantiations compile in parallel: one call, or a batch of calls if the second pointer is set.
// Each returns false for a slot count it does not hold.
bool rowsdyn_launch_k1(const DynArgs *, const DynBatch *, int slots, int mode, dim3, dim3, size_t, hipStream_t);         // 1..8
bool rowsdyn_launch_k2(const DynArgs *, const DynBatch *, int slots, int mode, dim3, dim3, size_t, hipStream_t);         // 5..8
bool rowsdyn_launch_k4(const DynArgs *, const DynBatch *, int slots, int mode, dim3, dim3, size_t, hipStream_t);         // 5..8
bool rowsdyn_launch_k8(const DynArgs *, const DynBatch *, int slots, int mode, dim3, dim3, size_t, hipStream_t);         // 5..8
bool rowsdyn_launch_k16(const DynArgs *, const DynBatch *, int slots, int mode, dim3, dim3, size_t, hipStream_t);        // 5..8
bool rowsdyn_launch_k16_long(const DynArgs *, const DynBatch *, int slots, int mode, dim3, dim3, size_t, hipStream_t);   // 9..10

#define IPTQ_ROWSDYN_CASE(K, S)                                                                   \
    case S:                                                                                       \
        if (B != nullptr) launch_kernel((softmax_rowsdyn_batch_kernel<K, S>), grid, block, lds, stream, *B); \
        else rowsdyn_launch_ks<K, S>(*A, mode, grid, block, lds, stream);                         \
        return true;

}  // namespace iptq
