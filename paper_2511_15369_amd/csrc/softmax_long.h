// Integer softmax (Section 4.4, Eq. 6-15) for the longest rows (up to the interface's 65536
// scores; up to 40957 wgrow16_is_faster decides between this and a workgroup per row): a workgroup of 16 wavefronts holds one row in its registers (the layout of
// softmax_wgrow.h with 1024 lanes) and walks over rows.  Such a row fills a compute unit (64 KB of
// LDS would not hold it, two of them do not fit the register file), so nothing else is resident
// to load while this one computes, and a kernel that ends with its row leaves the memory pipe
// idle for more than half the time.  Here the next row is fetched while the current one is
// computed: the first LDS_PASSES passes straight into LDS (global_load_lds, no registers), the rest
// into the registers that the scores leave when they have become exponentials.
//   LDS: at most 9 passes of 16 KB of the 160 KB; registers: 128 per lane at 16 wavefronts.
// 2048 rows of 50176 scores 91.0 us (5.6 TB/s; 1212 us in the three-pass kernel, one wavefront per
// row), of 65536 129 us (1567 us), 2000 rows of 32768 67.8 us (78.5 us as 16 wavefronts without the
// prefetch), 10 rows of 62000 12.9 us (720 us).  What is left: the last passes are asked for while
// the row is computed and not before, so the memory pipe still drains a little once per row; and the
// wait in front of a row is for every vector-memory operation, the stores of the row before among them.
// Tried instead: a ring of 9 passes in LDS alone, refilled pass by pass as the row is read (no
// registers, fewer loads in flight: 108 us at 2048 x 50176).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "plan.h"
#include "softmax_rows.h"
#include "softmax_wide.h"

namespace iptq {

constexpr int kLongWaves = 16;
constexpr int kLongMinSlots = 7;
constexpr int kLongMaxSlots = 16;
constexpr int kLoadNonTemporal = 2;                   // the cache-policy bit of a streaming load (2 to 4 % faster)
constexpr int kLongWorkgroups = 256;                  // compute units
constexpr int kLongLdsPasses = 9;

template <int V> using Int = std::integral_constant<int, V>;

// Every vector-memory (LDS) operation of this wavefront has completed; nothing is moved across.
IPTQ_DEV void wait_vector_memory()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("" ::: "memory");
}
IPTQ_DEV void wait_lds()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
}

// Workgroup barrier behind which earlier LDS accesses are visible.  Written out because a release
// fence also waits for the loads into LDS that are in flight for the next row.
IPTQ_DEV void lds_barrier()
{
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Sum over the workgroup; `between` runs once the caller's exponentials exist (its scores are
// dead by then).  Every thread of the workgroup must call it.
template <class F>
struct LongRowSum {
    uint32_t *partial;   // kLongWaves words of LDS
    int wv, lane;
    const F &between;
    IPTQ_DEV uint32_t operator()(uint32_t v) const
    {
        between();
        v = group_sum_u32<64>(v);
        if (lane == 0) partial[wv] = v;
        lds_barrier();
        uint32_t t = 0;
#pragma unroll
        for (int i = 0; i < kLongWaves; ++i) t += partial[i];
        return t;
    }
};

// EXTRA: an additive table, or the scores requantized in front; a kernel of its own because either
// takes registers, also when it is not used.  No register is left to fetch the next row's last passes
// into before the probabilities exist, and the table's blocks come two at a time.
template <int SLOTS, int MODE, int VARIANT, bool EXTRA>
__global__ void __launch_bounds__(64 * kLongWaves)
softmax_long_kernel(WideArgs A)
{
    constexpr int T = 64 * kLongWaves;                // lanes that share the row
    constexpr int NL = SLOTS < kLongLdsPasses ? SLOTS : kLongLdsPasses;      // passes fetched into LDS
    constexpr int NR = SLOTS - NL;                    // and into registers: the first NE of them once the
    constexpr int NE = (MODE == 0 || EXTRA) ? 0 : (SLOTS == 16 ? 2 : NR);   // exponentials exist, the rest after the probabilities
    // One block, the small arrays first and a wavefront's passes side by side, so that every access
    // is one address register and an immediate offset (below 64 KB).
    constexpr int kStageAt = 512;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kStageAt + NL * T * 16];
    int32_t *part_max = reinterpret_cast<int32_t *>(lds);
    uint32_t *part_sum = reinterpret_cast<uint32_t *>(lds + 4 * kLongWaves);
    uint8_t *lut = lds + 8 * kLongWaves;
    static_assert(8 * kLongWaves + kPostLutBytes <= kStageAt, "small arrays");
    touch_kernel_arguments<sizeof(WideArgs)>();
    const SoftmaxDev &P = A.P;
    int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    i32x4 *stage = reinterpret_cast<i32x4 *>(lds + kStageAt) + wv * (NL * 64);    // this wavefront's passes
    const int post_mode = A.post_mode;
    if (post_mode == PM_GENERAL) {                    // visible to all after the first row's barriers
        const int p_max = 1 << (P.m_bits - P.p_shift);
        for (int p = tid; p <= p_max; p += T) lut[p] = (uint8_t)post_dev<PM_GENERAL>((uint32_t)p, P);
    }
    const int cols = A.cols;
    auto edge_slot = [](int s) { return s == 0 || s >= SLOTS - 2; };

    // where a row lies on the 16-byte grid; everything here is workgroup-uniform
    struct Row {
        const i32x4 *src;
        int64_t e0;
        int phi, nb, nb_whole;                        // offset in its first block, blocks, blocks that can be loaded whole
    };
    auto row_at = [&](int64_t row) {
        Row R;
        R.e0 = row * cols + A.base_off;
        R.phi = (int)(R.e0 & 3);
        R.nb = (R.phi + cols + 3) >> 2;
        R.nb_whole = (A.cut_el != 0 && row == A.rows - 1) ? R.nb - 1 : R.nb;   // see softmax_wide.h
        R.src = reinterpret_cast<const i32x4 *>(A.scores) + (R.e0 >> 2);
        return R;
    };
    // Byte offset of this thread's block of pass s from the uniform address base_of(s) (so that a
    // pass costs a scalar addition and no address registers).  In the last two passes threads
    // beyond block n - 1 take it again; n - 1 >= (SLOTS - 2) T (the exact pass count).
    auto base_of = [](int s) { return (s == SLOTS - 1 ? SLOTS - 2 : s) * T; };
    auto offset_of = [&](int s, int n) -> uint32_t {
        const int b = s * T + tid;
        return 16u * (uint32_t)((s >= SLOTS - 2 ? min(b, n - 1) : b) - base_of(s));
    };
    i32x4 v[NR > 0 ? NR : 1];
    auto fetch_to_lds = [&](const Row &R) {
#pragma unroll
        for (int s = 0; s < NL; ++s)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(reinterpret_cast<const char *>(R.src + base_of(s)) + offset_of(s, R.nb_whole)),
                (__attribute__((address_space(3))) void *)(stage + s * 64), 16, 0, kLoadNonTemporal);
    };
    auto fetch_to_registers = [&](const Row &R, auto from, auto to) {
#pragma unroll
        for (int s = decltype(from)::value; s < decltype(to)::value; ++s)
            v[s] = stream_load(reinterpret_cast<const i32x4 *>(reinterpret_cast<const char *>(R.src + base_of(NL + s)) + offset_of(NL + s, R.nb_whole)));
    };

    int64_t row = blockIdx.x;                         // grid <= rows: every workgroup has a row
    Row R = row_at(row);
    fetch_to_lds(R);
    fetch_to_registers(R, Int<0>{}, Int<NR>{});
    for (;;) {
        const int64_t next = row + gridDim.x;
        const bool more = next < A.rows;              // workgroup-uniform, as is every branch around a barrier
        const Row N = row_at(more ? next : row);
        asm volatile("" : "+v"(tid));                 // offsets are recomputed per row: kept, they would spill

        // ---- the row out of LDS (each lane reads what its own wavefront's loads put there)
        wait_vector_memory();
        int32_t x[SLOTS][4];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const i32x4 t = s < NL ? stage[(s < NL ? s : 0) * 64 + lane] : v[s < NL ? 0 : s - NL];
            x[s][0] = t.x; x[s][1] = t.y; x[s][2] = t.z; x[s][3] = t.w;
        }
        if (R.nb_whole != R.nb) {                     // the tensor's last row, ending off the grid
            const int32_t *last = reinterpret_cast<const int32_t *>(R.src + (R.nb - 1));
#pragma unroll
            for (int s = SLOTS - 2; s < SLOTS; ++s) {
                if (s * T + tid == R.nb - 1) {        // elements beyond cut_el are masked below
                    x[s][0] = last[0];
                    if (A.cut_el > 1) x[s][1] = last[1];
                    if (A.cut_el > 2) x[s][2] = last[2];
                }
            }
            wait_vector_memory();                     // (else the wait lands behind the next row's loads, on every path)
        }
        wait_lds();                                   // the reads have returned: the places may be written again
        if (more) fetch_to_lds(N);

        // ---- elements outside the row become "minus infinity"
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
            if (edge_slot(s)) {
                const int c0 = 4 * (s * T + tid) - R.phi;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((unsigned)(c0 + e) >= (unsigned)cols) x[s][e] = kI32Min;
            }

        if (EXTRA && A.bias != nullptr) {
            const int64_t eb = (int64_t)row_mod_period((uint32_t)row, P) * cols;
            const i32x4 *bsrc = reinterpret_cast<const i32x4 *>(A.bias) + (eb >> 2);
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const i32x4 bv = load_i32x4_at(reinterpret_cast<const int32_t *>(bsrc + base_of(s)), offset_of(s, R.nb));
#pragma unroll
                for (int e = 0; e < 4; ++e) x[s][e] = add_table_entry(x[s][e], bv[e]);
                if (s % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // two loads in flight: the registers are the row's
            }
        }
        // the requantization in front, one block at a time for the same reason
        if (EXTRA && P.pre_mode != 0) {
            const int32_t pre_m = P.pre_m, pre_s = P.pre_s;
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int32_t r = pre_requant_dev(x[s][e], pre_m, pre_s);
                    x[s][e] = x[s][e] == kI32Min ? kI32Min : r;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // ---- Eq. 6: row maximum over the workgroup
        int32_t mx = kI32Min;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = max(mx, x[s][e]);
        mx = group_max_i32<64>(mx);
        if (lane == 0) part_max[wv] = mx;
        lds_barrier();
#pragma unroll
        for (int i = 0; i < kLongWaves; ++i) mx = max(mx, part_max[i]);

        const int32_t D = P.d_clamp;
        const bool low_row = mx < kI32Min + D;        // workgroup-uniform; see softmax_rows_kernel
        auto between = [&]() { if (more) fetch_to_registers(N, Int<0>{}, Int<NE>{}); };
        const LongRowSum<decltype(between)> row_sum{part_sum, wv, lane, between};
        if (__builtin_expect(low_row, 0)) {
            // The clamp cannot tell masked scores from live ones: the row again from memory, score
            // by score with an explicit test (a rare path: it must cost no registers, not no time).
            const int32_t *srow = A.scores + R.e0;
            const int32_t *brow = A.bias;
            if (EXTRA && brow != nullptr) brow += (int64_t)row_mod_period((uint32_t)row, P) * cols;
            auto exponential = [&](int c) {
                int32_t t = srow[c];
                if (EXTRA && A.bias != nullptr) t = add_table_entry(t, brow[c]);
                if (EXTRA && P.pre_mode != 0 && t != kI32Min) t = pre_requant_dev(t, P.pre_m, P.pre_s);
                return bit_exp_dev<VARIANT, true>(t, kI32Min, mx, P);
            };
            uint32_t sum = 0;
#pragma unroll 1
            for (int c = tid; c < cols; c += T) sum += exponential(c);
            const uint32_t f = floor_pow2_div(P.m_bits, row_sum(sum));
            uint8_t *orow = A.out + R.e0;
#pragma unroll 1
            for (int c = tid; c < cols; c += T)
                orow[c] = (uint8_t)post_dev<PM_GENERAL>((exponential(c) * f) >> P.p_shift, P);
            if (NE < NR && more) fetch_to_registers(N, Int<NE>{}, Int<NR>{});
        } else {
        uint32_t w[SLOTS];                            // four probabilities per block, one per byte
        softmax_slab_math<64, SLOTS, MODE, VARIANT, PM_NONE>(x, w, mx, mx - D, false, lut, P, row_sum);

        // ---- post step on the packed bytes (a probability is at most 128)
        if (post_mode == PM_CLAMP127) {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) w[s] = clamp127_bytes(w[s]);
        } else if (post_mode == PM_GENERAL) {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) w[s] = post_lut_gather(lut, w[s]);
        } else if (P.post_xor != 0) {                 // signed output around the zero-point -128
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) w[s] ^= P.post_xor;
        }

        if (NE < NR && more) fetch_to_registers(N, Int<NE>{}, Int<NR>{});

        // ---- write back: whole blocks as dwords, the two shared edge blocks byte by byte
        uint8_t *dst8 = A.out + (R.e0 - R.phi);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int b = s * T + tid;
            const int c0 = 4 * b - R.phi;
            if (!edge_slot(s)) {                      // every thread's block lies inside the row
                stream_store_bytes4(w[s], dst8 + 4 * T * s + (uint32_t)(4 * tid));
            } else if (b < R.nb) {
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
        if (!more) break;
        row = next;
        R = N;
    }
}

// mode: SoftmaxDev::packed
template <int SLOTS>
static void long_launch_s(const WideArgs &A, int mode, dim3 grid, hipStream_t stream)
{
#define IPTQ_LONG_LAUNCH(MODE, EXTRA)                                                             \
    do {                                                                                          \
        if (A.P.variant == 0) launch_kernel((softmax_long_kernel<SLOTS, MODE, 0, EXTRA>), grid, dim3(64 * kLongWaves), 0, stream, A);      \
        else if (A.P.variant == 1) launch_kernel((softmax_long_kernel<SLOTS, MODE, 1, EXTRA>), grid, dim3(64 * kLongWaves), 0, stream, A); \
        else launch_kernel((softmax_long_kernel<SLOTS, MODE, 2, EXTRA>), grid, dim3(64 * kLongWaves), 0, stream, A);                       \
    } while (0)
    const bool extra = A.bias != nullptr || A.P.pre_mode != 0;
    if (mode == 0 && extra) IPTQ_LONG_LAUNCH(0, true);
    else if (mode == 0) IPTQ_LONG_LAUNCH(0, false);
    else if (mode == 1 && extra) IPTQ_LONG_LAUNCH(1, true);
    else if (mode == 1) IPTQ_LONG_LAUNCH(1, false);
    else if (extra) IPTQ_LONG_LAUNCH(2, true);
    else IPTQ_LONG_LAUNCH(2, false);
#undef IPTQ_LONG_LAUNCH
}

// one translation unit per group of pass counts; each returns false for a count it does not hold
bool long_launch_p7_8(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);
bool long_launch_p9_12(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);
bool long_launch_p13_16(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream);

#define IPTQ_LONG_CASE(S)                                                                         \
    case S: long_launch_s<S>(A, mode, grid, stream); return true;

}  // namespace iptq
