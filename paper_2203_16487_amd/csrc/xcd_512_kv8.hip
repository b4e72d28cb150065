// The per-XCD decoder's kernels, d = 512, cross-attention keys / values as E4M3 codes.
#include "xcd_core.h"

namespace sd {
namespace xcd {
template hipError_t pl_launch_both<true, 512>(hipStream_t, XcdArgs, int);
}  // namespace xcd
}  // namespace sd
