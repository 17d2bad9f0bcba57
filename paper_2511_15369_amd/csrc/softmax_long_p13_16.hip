// Softmax of the longest rows, one walking workgroup per row, 13 to 16 passes.
#include "softmax_long.h"

namespace iptq {
bool long_launch_p13_16(const WideArgs &A, int passes, int mode, dim3 grid, hipStream_t stream)
{
    switch (passes) {
    IPTQ_LONG_CASE(13)
    IPTQ_LONG_CASE(14)
    IPTQ_LONG_CASE(15)
    IPTQ_LONG_CASE(16)
    default: return false;
    }
}
}  // namespace iptq
