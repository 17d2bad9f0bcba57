// Host side of the run-time-row-length slab kernel (softmax_rowsdyn.h): lane layout for a
// row length and the launch.
#include <hip/hip_runtime.h>

#include "softmax_rowsdyn.h"

namespace iptq {

// Lane layout for a row length: the fewest lanes per row that keep the blocks per lane at or
// below 8 (5 wavefronts per SIMD; measured equal or better than more blocks on fewer lanes),
// else 16 lanes per row with up to 10 blocks per lane (rows of up to about 635 scores).
// *slots is exactly ceil(most blocks a row can touch / lanes): the kernels rely on it.
// Returns false for longer rows: one wavefront per row serves those better (softmax_wide.h;
// measured 70-75 % against 66-69 % of the HBM roofline at 650 to 829 columns, 57-67 % against
// 69-75 % at 509 to 600).
bool rowsdyn_geometry(int32_t cols, int *lanes, int *slots)
{
    const int nb_max = (cols % 4 == 0) ? cols / 4 : ((cols % 2 == 0) ? (cols + 2 + 3) / 4 : (cols + 3 + 3) / 4);
    int k = 1;
    while (k < 16 && (nb_max + k - 1) / k > 8) k *= 2;
    const int n = (nb_max + k - 1) / k;
    if (n > 10) return false;
    *lanes = k;
    *slots = n;
    return true;
}

// Whether a short call is faster in the three-pass kernel: a masked one, or one beside a table that one
// wavefront per row does not take.  A call of a few thousand rows lasts as long as one wavefront takes from a
// cold start: here that grows with the code, which is unrolled over the blocks per lane, more so with an int32 mask
// and for odd row lengths; the three-pass kernel's code is short, and it pays per 64 scores of a row and per
// row.  Both times as linear models, in nanoseconds without what they share.  Of 5708 masked calls of 256 to
// 8192 rows of 9 to 256 scores, either mask, with and without a table, first and second degree, whole and ragged
// row counts, in a graph: the choice is at most 24 % and on average 0.7 % slower than the faster kernel (always
// this one: 71 % and 4.8 %); of 1172 beside a table alone 23 % and 1.2 %.  With fewer than three blocks per lane
// this kernel is always the faster one, beyond 256 scores nearly always.  704 rows of 64 scores with an int32 mask and a
// table 3.3 us in the three-pass kernel, 4.9 here, 6147 of 29 with a packed mask 5.0 and 3.8.  (A ragged row count has no term of
// its own: since its last slab is a whole one it takes what a whole one takes, 706 of 29 with an int32 mask and a table 5.5
// here, 704 5.1; charged for a partial one, 3075 x 100 went to the three-pass kernel, 5.1 us against 4.8, 258 x 196 6.0 against 4.1.)
bool rowsdyn_loses_short_call(int64_t rows, int32_t cols, bool has_bias, bool int_mask, bool bit_mask)
{
    int lanes = 0, slots = 0;
    if (rows > 8192 || cols > 256 || !rowsdyn_geometry(cols, &lanes, &slots) || slots < 3) return false;
    int64_t here = 960 + slots * (210 + (int_mask ? 70 : 0));
    if (cols % 2 != 0) here += 360;
    if (lanes == 1) here -= 440;
    const int64_t passes = (cols + 63) / 64;
    int64_t three_pass = 810 * passes + (int_mask || bit_mask ? 440 : 0);
    if (rows > 1024) three_pass += 170 * (passes + 1) * (rows - 1024) / 1024;
    return three_pass < here;
}

// The same against one wavefront per row, which takes unmasked calls (one pass up to 256 scores): how much
// longer this kernel's chain is, by its blocks and the steps of its reduction, against what the rows add
// there.  Rows that are whole 64-byte lines are 0.3 us faster there.  Fitted to 1120 calls of 3073 to 8192 rows of 9 to 256
// scores of the second degree, with and without a table, or with a table of 40 rows, in a graph: at most 18 % and on
// average 0.3 % slower than the faster kernel (always this one: 43 % and 7.4 %; by the model above, whose other side is three
// passes, 43 % and 5.9 %).  4096 rows of 256 scores of the second degree 4.3 us here, 3.2 there; 8192 of 25 3.7 and 4.6.
bool rowsdyn_loses_to_wavefronts(int64_t rows, int32_t cols)
{
    int lanes = 0, slots = 0;
    if (rows > 8192 || cols > 256 || !rowsdyn_geometry(cols, &lanes, &slots) || slots < 3) return false;
    int64_t longer = 210 * slots - 1130;
    for (int k = lanes; k > 1; k /= 2) longer += 190;
    if (cols % 16 == 0) longer += 350;
    return longer > 230 * (rows - 3072) / 1024;
}

static int64_t gcd_i64(int64_t a, int64_t b)
{
    while (b != 0) { const int64_t t = a % b; a = b; b = t; }
    return a;
}

// The kernel arguments of one call and its number of workgroups; false if this kernel does not serve it.
static bool rowsdyn_arguments(const SoftmaxCall &c, int32_t cols, int post_mode, int k, DynArgs *args, int64_t *wgs)
{
    DynArgs &A = *args;
    const int rpw = 64 / k;
    const bool has_bias = c.bias != nullptr;
    const bool aligned = ((reinterpret_cast<uintptr_t>(c.scores) | reinterpret_cast<uintptr_t>(c.bias)) & 3) == 0;
    // a slab wraps around the table once at most, twice with one lane per row (64 rows per slab)
    const bool bias_ok = !has_bias || ((int64_t)c.P.bias_period_rows * cols >= 4 &&
                                       (int64_t)c.P.bias_period_rows * cols < ((int64_t)1 << 31) &&
                                       c.P.bias_period_rows >= (k == 1 ? 32 : rpw));
    // int32 masks are loaded in blocks of four entries at 32-bit byte offsets
    const bool int_mask = c.mask != nullptr;
    const int64_t mask_el = int_mask ? (int64_t)c.P.n_windows * cols * cols : 0;
    if (int_mask && (mask_el < 4 || mask_el >= ((int64_t)1 << 30))) return false;
    if (c.mask_bits != nullptr && (int64_t)c.P.n_windows * cols * ((cols + 63) / 64) * 8 >= ((int64_t)1 << 31))
        return false;
    const int64_t n_slabs = (c.rows + rpw - 1) / rpw;
    if (!aligned || !bias_ok || n_slabs == 0) return false;
    A.scores = c.scores; A.bias = c.bias; A.out = c.out;
    A.n_slabs = (uint32_t)n_slabs;
    A.few_rows = c.rows < rpw ? (int32_t)c.rows : 0;
    A.last_row0 = A.few_rows != 0 ? 0u : (uint32_t)(c.rows - rpw);
    A.cols = cols; A.post_mode = post_mode;
    A.wave_lds = (int32_t)((((int64_t)rpw * cols * 4 + 15) & ~(int64_t)15) + kPostLutBytes);
    A.mask = c.mask; A.mask_bits = c.mask_bits;
    A.cols_magic = 0; A.cols_sh = 0;
    if ((c.mask != nullptr || c.mask_bits != nullptr) && cols >= 2 &&
        !make_magic_u32((uint32_t)cols, 31, &A.cols_magic, &A.cols_sh))
        return false;
    A.P = c.P;
    int wpb = 65536 / A.wave_lds;                     // wavefronts per workgroup: 1..4
    if (wpb > 4) wpb = 4;
    if (wpb < 1) return false;
    A.wpb = (uint32_t)wpb;
    int64_t &n_wgs = *wgs;
    n_wgs = (n_slabs + wpb - 1) / wpb;
    A.share_q = 0; A.share_magic = 0; A.share_sh = 0;
    auto share_every = [&](int64_t period) {          // wavefronts of a workgroup that many rows apart
        const int64_t q = period / gcd_i64(period, rpw);
        if (q < 2 || q >= 65536 || q * wpb > n_slabs ||
            !make_magic_u32((uint32_t)q, 31, &A.share_magic, &A.share_sh))
            return false;
        A.share_q = (uint32_t)q;
        n_wgs = (n_slabs + (int64_t)wpb * q - 1) / ((int64_t)wpb * q) * q;
        return true;
    };
    if (wpb > 1) {
        // an int32 mask is as large a stream through L1 as the scores: share it together with the
        // bias (least common multiple of both periods) where the call is long enough for that
        bool shared = false;
        if (int_mask) {
            const int64_t mp = c.P.mask_period_rows, bp = has_bias ? c.P.bias_period_rows : 1;
            shared = share_every(mp / gcd_i64(mp, bp) * bp);
        }
        if (!shared && has_bias) share_every(c.P.bias_period_rows);
    }
    return true;
}

static bool rowsdyn_launch(const DynArgs *A, const DynBatch *B, int k, int slots, int mode, dim3 grid, dim3 block,
                           size_t lds, hipStream_t stream)
{
    if (k == 1) return rowsdyn_launch_k1(A, B, slots, mode, grid, block, lds, stream);
    if (k == 2) return rowsdyn_launch_k2(A, B, slots, mode, grid, block, lds, stream);
    if (k == 4) return rowsdyn_launch_k4(A, B, slots, mode, grid, block, lds, stream);
    if (k == 8) return rowsdyn_launch_k8(A, B, slots, mode, grid, block, lds, stream);
    return slots <= 8 ? rowsdyn_launch_k16(A, B, slots, mode, grid, block, lds, stream)
                      : rowsdyn_launch_k16_long(A, B, slots, mode, grid, block, lds, stream);
}

// LDS to ask for in the longest launches: one workgroup per compute unit less than would fit, where three are
// left.  16 lanes per row, up to 8 blocks each, or 10 on the 16-byte grid: 130 / 190 million scores in rows of
// 401 107.8 / 157.4 us against 109.8 / 160.2, of 430 106.8 / 154.8 against 108.6 / 159.2, of 600 102.5 / 147.1 against
// 106.1 / 155.4 (95 million 76.2 and 78.2, 65 million the same).  9 blocks gain nothing (570 109.3 / 156.1 against
// 107.6 / 155.8), and with a table, a requantization in front or the second degree it is slower (600 162 against
// 152, 155 against 151, 151.6 against 151.2).
static size_t rowsdyn_lds(const DynArgs &A, int lanes, int slots, int64_t scores)
{
    const size_t own = (size_t)A.wave_lds * A.wpb;
    if (lanes != 16 || scores <= 110 * 1000 * 1000 || A.bias != nullptr || A.mask != nullptr || A.mask_bits != nullptr ||
        !plain_arithmetic(A.P) || !(slots <= 8 || (slots == 10 && A.cols % 4 == 0)))
        return own;
    const int fit = 160 * 1024 / (int)((own + 1279) / 1280 * 1280);       // handed out in units of 1280 bytes
    return fit >= 4 ? (size_t)(160 * 1024 / (fit - 1) / 1280 * 1280) : own;
}

// Every row of one call if the call qualifies; returns the number of rows served through
// *done (0: not served, nothing enqueued).
hipError_t softmax_rowsdyn_launch(const SoftmaxCall &c, int32_t cols, int post_mode, int64_t *done,
                                  hipStream_t stream)
{
    *done = 0;
    int k = 0, slots = 0;
    if (!rowsdyn_geometry(cols, &k, &slots)) return hipSuccess;
    DynArgs A;
    int64_t n_wgs = 0;
    if (!rowsdyn_arguments(c, cols, post_mode, k, &A, &n_wgs)) return hipSuccess;
    if (!rowsdyn_launch(&A, nullptr, k, slots, c.P.packed, dim3((unsigned)n_wgs), dim3(64 * A.wpb),
                        rowsdyn_lds(A, k, slots, c.rows * cols), stream))
        return hipSuccess;                            // no such layout: the caller's next kernel serves it
    *done = c.rows;
    return take_launch_status();
}

// The calls of a batch that one launch can serve together: packed arithmetic without a mask and
// without a requantization in front.  done[i] becomes the rows of every call that was served; fewer
// than two such calls are left alone, and so is what does not qualify.
hipError_t softmax_rowsdyn_launch_batch(const SoftmaxCall *calls, const int *post_modes, int n_calls, int32_t cols,
                                        int64_t *done, hipStream_t stream)
{
    int k = 0, slots = 0;
    if (!rowsdyn_geometry(cols, &k, &slots)) return hipSuccess;
    DynBatch B;
    int of[kDynBatchMax];                             // which call an item is
    int64_t total_wgs = 0;
    B.head.clear();
    auto flush = [&]() -> hipError_t {
        // (false: no such layout, the caller's next kernel serves these calls; wavefronts per workgroup and
        // their LDS are the same for every call of a row length)
        if (B.head.n_items >= 2 && rowsdyn_launch(nullptr, &B, k, slots, 2, dim3((unsigned)total_wgs), dim3(64 * B.item[0].wpb),
                                             (size_t)B.item[0].wave_lds * B.item[0].wpb, stream))
            for (int i = 0; i < B.head.n_items; ++i) done[of[i]] = calls[of[i]].rows;
        B.head.clear();
        total_wgs = 0;
        return take_launch_status();
    };
    for (int i = 0; i < n_calls; ++i) {
        const SoftmaxCall &c = calls[i];
        if (done[i] != 0 || c.mask != nullptr || c.mask_bits != nullptr || c.P.packed != 2 || c.P.pre_mode != 0 ||
            !(c.algo == IPTQ_ALGO_AUTO || c.algo == IPTQ_ALGO_DYNAMIC || c.algo == IPTQ_ALGO_SLAB))
            continue;
        DynArgs A;
        int64_t n_wgs = 0;
        if (!rowsdyn_arguments(c, cols, post_modes[i], k, &A, &n_wgs)) continue;
        // (a launch has fewer than 2^32 work-items)
        if (B.head.n_items == kDynBatchMax || (total_wgs + n_wgs) * 256 >= ((int64_t)1 << 32)) {
            const hipError_t e = flush();
            if (e != hipSuccess) return e;
        }
        const int at = B.head.add((uint32_t)total_wgs);
        B.item[at] = A;
        of[at] = i;
        total_wgs += n_wgs;
    }
    return flush();
}

}  // namespace iptq
