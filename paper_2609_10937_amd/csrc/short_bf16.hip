// The short-sequence kernel for dtype bf16: every head dimension, 16 or 32 query
// rows per workgroup, one or two splits per wave.
#include "short_kernel.hpp"

namespace attn {

hipError_t launch_short_bf16(const FwdParams& p, int d, int rows, hipStream_t s) {
  return launch_short_t<ATTN_BF16>(p, d, rows, s);
}

}  // namespace attn
