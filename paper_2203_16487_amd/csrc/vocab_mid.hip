// Vocabulary of 257 - 384 and 513 - 640 rows.  In a file of its own, that is in device code of its own: as kernels of gemm.hip these moved the others there
// (none of which they call or change), and every launch of a pass beyond them took 0.1 - 0.2 us more: verification of 128 x 11 rows, d = 1024,
// 874 / 882 us, an iteration of the loop of 128 sequences 1118 / 1128.
#include <algorithm>

#include "vocab_tiles.h"

namespace sd {

// 257 - 384 rows in two row tiles of 192, one block to a CU.  513 - 640: those behind the first 256, and of these a tile of 256 x 128 a CU ahead.
typedef GemmCfg<192, 256, 2, 2, 4> CfgVocabMid;
template <bool ARGMAX>
__global__ __launch_bounds__(CfgVocabMid::kThreads, 2) void vocab_mid_kernel(const bf16* __restrict__ A, const bf16* __restrict__ E, int M, int V, int K, int NT,
                                                                             const float* __restrict__ zd_row, float* __restrict__ part,
                                                                             float* __restrict__ logits) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  int mt, nt;
  if (!xcd_tile(blockIdx.x, 2, (V + 255) / 256, mt, nt)) return;
  if (M > 384) {
    if (nt * 256 + mt * 128 < V) vocab_tile<ARGMAX, CfgTall>(A, E, M, V, K, NT, 0, nt * 256 + mt * 128, zd_row, part, logits, smem);
    __syncthreads();
  }
  vocab_tile<ARGMAX, CfgVocabMid>(A, E, M, V, K, NT, (M > 384 ? 256 : 0) + mt * 192, nt * 256, zd_row, part, logits, smem);
}

template <bool ARGMAX>
static hipError_t launch_vocab_mid(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, const float* zd, float* part, float* logits) {
  constexpr int kBytes = std::max(CfgVocabMid::kSmemBytes, CfgTall::kSmemBytes);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(vocab_mid_kernel<ARGMAX>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  SD_LAUNCH_TIMED((vocab_mid_kernel<ARGMAX>), dim3(xcd_grid(2, (V + 255) / 256)), dim3(CfgVocabMid::kThreads), kBytes, st, A, E, M, V, K,
                  (V + 127) / 128, zd, part, logits);
  return hipGetLastError();
}

hipError_t vocab_mid(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, bool stats, const float* zd, float* part, float* logits) {
  return stats ? launch_vocab_mid<false>(st, A, E, M, V, K, zd, part, logits) : launch_vocab_mid<true>(st, A, E, M, V, K, nullptr, part, logits);
}

}  // namespace sd
