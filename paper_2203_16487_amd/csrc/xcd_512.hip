// The per-XCD decoder's kernels, d = 512, cross-attention keys / values in bf16.
#include "xcd_core.h"

namespace sd {
namespace xcd {
template hipError_t pl_launch_both<false, 512>(hipStream_t, XcdArgs, int);
}  // namespace xcd
}  // namespace sd
