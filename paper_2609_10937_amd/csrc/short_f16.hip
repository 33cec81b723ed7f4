// The short-sequence kernel for dtype f16: every head dimension, 16 or 32 query
// rows per workgroup, one or two splits per wave.
#include "short_kernel.hpp"

namespace attn {

hipError_t launch_short_f16(const FwdParams& p, int d, int rows, hipStream_t s) {
  return launch_short_t<ATTN_F16>(p, d, rows, s);
}

}  // namespace attn
