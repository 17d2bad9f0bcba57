// Host side of the softmax of the longest rows (softmax_long.h).
#include <hip/hip_runtime.h>

#include "softmax_long.h"

namespace iptq {

// Passes of 1024 blocks a row of `cols` scores needs at its worst alignment (exactly: the kernels
// rely on it); false outside the compiled counts.
bool long_geometry(int32_t cols, int *slots, bool off_grid)
{
    // off_grid: as for wide_geometry
    const int nb_max = (off_grid || cols % 2 != 0) ? (cols + 3 + 3) / 4 : ((cols % 4 == 0) ? cols / 4 : (cols + 2 + 3) / 4);
    const int n = (nb_max + 64 * kLongWaves - 1) / (64 * kLongWaves);
    if (n < kLongMinSlots || n > kLongMaxSlots) return false;
    *slots = n;
    return true;
}

// Every row of one call if the call qualifies (same conditions as softmax_wide_launch).
hipError_t softmax_long_launch(const SoftmaxCall &c, int32_t cols, int post_mode, int64_t *done,
                               hipStream_t stream)
{
    *done = 0;
    int slots = 0;
    const uintptr_t sa = reinterpret_cast<uintptr_t>(c.scores);
    const int base_off = (int)((sa & 15) >> 2);
    if ((sa & 3) != 0 || c.rows <= 0) return hipSuccess;
    if (!long_geometry(cols, &slots, base_off != 0)) return hipSuccess;
    const bool has_bias = c.bias != nullptr;
    const bool bias_ok = !has_bias || (base_off == 0 && (reinterpret_cast<uintptr_t>(c.bias) & 15) == 0 &&
                                       ((int64_t)c.P.bias_period_rows * cols) % 4 == 0);
    if (!bias_ok) return hipSuccess;
    WideArgs A;
    A.scores = c.scores - base_off; A.bias = c.bias; A.out = c.out - base_off; A.base_off = base_off;
    A.rows = c.rows; A.cols = cols; A.post_mode = post_mode; A.P = c.P;
    A.cut_el = (int)((base_off + c.rows * cols) & 3);
    // one workgroup per compute unit, walking over the rows (any number of workgroups is correct)
    const int64_t wgs = c.rows < kLongWorkgroups ? c.rows : kLongWorkgroups;
    const dim3 grid((unsigned)wgs);
    const int mode = c.P.packed;
    const bool launched = slots <= 8 ? long_launch_p7_8(A, slots, mode, grid, stream)
                        : slots <= 12 ? long_launch_p9_12(A, slots, mode, grid, stream)
                                      : long_launch_p13_16(A, slots, mode, grid, stream);
    if (!launched) return hipSuccess;
    *done = c.rows;
    return take_launch_status();
}

}  // namespace iptq
