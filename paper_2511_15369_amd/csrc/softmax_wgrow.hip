// Host side of the one-workgroup-per-row softmax kernel (softmax_wgrow.h).
#include <hip/hip_runtime.h>

#include "softmax_wgrow.h"

namespace iptq {

// Wavefronts per workgroup and pass count for a row length (exactly the passes a row needs at its
// worst alignment: the kernels rely on it); false beyond 40957 scores (40960 where a multiple of four
// starts on the grid).  Up to 13 passes keep a lane within 128 registers, so two workgroups share a
// compute unit and one loads while the other computes (66-78 % of the HBM roofline).  Beyond 26621
// (26624) scores one workgroup of 16 wavefronts fills a compute unit; see wgrow16_is_faster.
bool wgrow_geometry(int32_t cols, int *waves, int *slots, bool off_grid)
{
    // off_grid: as for wide_geometry
    const int nb_max = (off_grid || cols % 2 != 0) ? (cols + 3 + 3) / 4 : ((cols % 4 == 0) ? cols / 4 : (cols + 2 + 3) / 4);
    int w = 4;
    if ((nb_max + 255) / 256 > 13) w = 8;
    if ((nb_max + 511) / 512 > 13) w = 16;
    const int n = (nb_max + 64 * w - 1) / (64 * w);
    if (n > (w == 16 ? 10 : 13)) return false;
    *waves = w;
    *slots = n;
    return true;
}

// Rows that fill a compute unit: 16 wavefronts and a workgroup per row here, or the kernel that
// walks over rows (softmax_long.h).  That one wins where it has a next row to fetch and the registers
// to fetch it into (2000 x 32768 scores 67.8 us against 78.5 here).  Up to one row per compute unit
// there is no next row, and its longer code only starts later (10 x 26628 scores 7.7 us against 7.4;
// from 257 rows on 15.0 against 15.8).  With a requantization in front nothing can be fetched before
// the arithmetic, and it breaks even between four and five rows per compute unit (33000 scores: 600 rows
// 33.4 us against 32.0, 1100 rows 54.7 against 54.3, 1200 rows 55.3 against 56.2, 1500 rows 65.5 against
// 67.8).  Beside an additive table it never does
// (2000 x 26628 82.7 us against 77.3, 1500 x 40956 87.9 against 82.4; with both 102.9 against 86.5).
// (The second-degree exponential has not been instantiated here: it goes to the walking kernel.)
bool wgrow16_is_faster(int64_t rows, bool has_bias, bool has_pre, int variant)
{
    if (variant == 2) return false;
    return has_bias || rows <= (has_pre ? 1152 : 256);
}

// Every row of one call if the call qualifies (same conditions as softmax_wide_launch).
hipError_t softmax_wgrow_launch(const SoftmaxCall &c, int32_t cols, int post_mode, int64_t *done,
                                hipStream_t stream)
{
    *done = 0;
    int waves = 0, slots = 0;
    // The tensor may start anywhere on the 4-byte grid (rows are addressed on the 16-byte grid
    // below it) and the output anywhere; the additive table is indexed block by block and needs
    // both tensors on the 16-byte grid.
    const uintptr_t sa = reinterpret_cast<uintptr_t>(c.scores);
    const int base_off = (int)((sa & 15) >> 2);
    if ((sa & 3) != 0) return hipSuccess;
    if (!wgrow_geometry(cols, &waves, &slots, base_off != 0)) return hipSuccess;
    if (waves == 16 && !wgrow16_is_faster(c.rows, c.bias != nullptr, c.P.pre_mode != 0, c.P.variant)) return hipSuccess;
    const bool has_bias = c.bias != nullptr;
    const bool bias_ok = !has_bias || (base_off == 0 && (reinterpret_cast<uintptr_t>(c.bias) & 15) == 0 &&
                                       ((int64_t)c.P.bias_period_rows * cols) % 4 == 0);
    if (!bias_ok) return hipSuccess;
    // A tensor that ends off the 16-byte grid: the kernel loads the last row's final block
    // element by element, which takes rows of at least 8 scores (a whole block before it).
    const int cut_el = (int)((base_off + c.rows * cols) & 3);
    if (c.rows <= 0 || (cut_el != 0 && cols < 8)) return hipSuccess;
    const int64_t rows = c.rows;
    WideArgs A;
    A.scores = c.scores - base_off; A.bias = c.bias; A.out = c.out - base_off; A.base_off = base_off; A.rows = rows; A.cols = cols; A.post_mode = post_mode; A.P = c.P;
    A.cut_el = cut_el;
    const dim3 grid((unsigned)rows);                  // one workgroup per row, exactly
    const int mode = c.P.packed;
    bool launched;
    if (waves == 4) launched = slots <= 9 ? wgrow_launch_w4_lo(A, slots, mode, grid, stream) : wgrow_launch_w4_hi(A, slots, mode, grid, stream);
    else if (waves == 8) launched = slots <= 10 ? wgrow_launch_w8_lo(A, slots, mode, grid, stream) : wgrow_launch_w8_hi(A, slots, mode, grid, stream);
    else launched = wgrow_launch_w16(A, slots, mode, grid, stream);
    if (!launched) return hipSuccess;
    *done = rows;
    return take_launch_status();
}

}  // namespace iptq
