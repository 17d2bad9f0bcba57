// Softmax of the longest rows, one walking workgroup per row, 7 or 8 passes.
#include "softmax_long.h"

namespace iptq {
bool long_launch_p7_8(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream)
{
    switch (passes) {
    IPTQ_LONG_CASE(7)
    IPTQ_LONG_CASE(8)
    default: return false;
    }
}
}  // namespace iptq
