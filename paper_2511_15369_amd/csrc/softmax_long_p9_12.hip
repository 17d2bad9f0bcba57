// Softmax of the longest rows, one walking workgroup per row, 9 to 12 passes.
#include "softmax_long.h"

namespace iptq {
bool long_launch_p9_12(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream)
{
    switch (passes) {
    IPTQ_LONG_CASE(9)
    IPTQ_LONG_CASE(10)
    IPTQ_LONG_CASE(11)
    IPTQ_LONG_CASE(12)
    default: return false;
    }
}
}  // namespace iptq
