// What the vocabulary kernels of gemm.hip and vocab_mid.hip share: tiles dealt to the XCDs, a tile's product with the statistics of its rows.
#pragma once
#include <type_traits>

#include "gemm_core.h"
#include "kernels.h"

namespace sd {

// Workgroup ids are dealt round-robin to the 8 XCDs (id % 8), each with its own L2.  Tiles are
// numbered n-major (m fastest) and XCD x takes the contiguous run [x*per, (x+1)*per): the
// tiles that run together on one XCD then share a few weight column-panels and the
// activation rows, which stay in that XCD's L2.  Returns false for the padding blocks.
__device__ __forceinline__ bool xcd_tile(int id, int MT, int NT, int& mt, int& nt) {
  const int nb = MT * NT;
  const int per = (nb + 7) >> 3;
  const int t = (id & 7) * per + (id >> 3);
  if ((id >> 3) >= per || t >= nb) return false;
  nt = t / MT;
  mt = t - nt * MT;
  return true;
}
static inline int xcd_grid(int MT, int NT) { return 8 * ((MT * NT + 7) / 8); }

typedef GemmCfg<256, 128, 3, 4, 2> CfgTall;   // 144 KB LDS, eight waves: one block per CU

// The records of a finished tile of 256 rows; zd: the drafts' logits of the lane's rows (-inf on rows that score no draft: count unused); rec:
// [wave columns][256 rows].
template <bool ARGMAX, class Cfg>
__device__ __forceinline__ void vocab_records(const GemmAcc<Cfg>& acc, const float (&zd)[Cfg::kTM], f32x4* rec, int lane, int wave, int m0, int n0, int M,
                                              int V, int NT, float* __restrict__ part, float* __restrict__ logits) {
  static_assert((Cfg::kBM == 256 || Cfg::kBM == 192) && Cfg::kWN == 64 && (Cfg::kWavesN == 2 || Cfg::kWavesN == 4) && Cfg::kThreads == 512, "shape");
  const int tid = wave * 64 + lane, wy = wave / Cfg::kWavesN, wx = wave % Cfg::kWavesN, lcol = lane & 31, lhalf = lane >> 5;
  const int nw = n0 + wx * 64 + 4 * lhalf;        // first column of this lane
  // column of accumulator (j, r) relative to nw: ascending in (j, r), so ">" keeps the lowest index of a tie
  auto col = [](int j, int r) { return j * 32 + 8 * (r >> 2) + (r & 3); };
  constexpr float kLog2e = 1.44269504088896341f;
  auto scan = [&](auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    const int nvalid = V - nw;   // columns of this lane inside the matrix (FULL: all of them)
#pragma unroll
    for (int i = 0; i < Cfg::kTM; ++i) {
      float best = kNegInf;
      int bestc = 0x3fffffff, cnt = 0;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float v = acc.c[i][j][r];
          if (FULL || col(j, r) < nvalid) {
            if (v > best) { best = v; bestc = col(j, r); }
            if (!ARGMAX) cnt += (v > zd[i]) ? 1 : 0;
          }
        }
      float se = 0.f;
      if (!ARGMAX) {
        const float nb2 = -best * kLog2e;   // exp(v - best) = 2^(v log2e - best log2e)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (FULL || col(j, r) < nvalid) se += __builtin_amdgcn_exp2f(__builtin_fmaf(acc.c[i][j][r], kLog2e, nb2));
        if (!(best > kNegInf)) se = 0.f;    // no valid column (or all -inf): nothing to sum
      }
      const int besti = nw + bestc;
      // the other lane half holds the interleaved groups of 4 columns of the same row
      const float obest = __shfl_xor(best, 32, 64);
      const int obesti = __shfl_xor(besti, 32, 64);
      const float ose = __shfl_xor(se, 32, 64);
      const int ocnt = __shfl_xor(cnt, 32, 64);
      const float nb = fmaxf(best, obest);
      float tot = 0.f;
      if (best > kNegInf) tot += se * __expf(best - nb);
      if (obest > kNegInf) tot += ose * __expf(obest - nb);
      const int nbi = (obest > best || (obest == best && obesti < besti)) ? obesti : besti;
      if (lhalf == 0)
        rec[wx * 256 + wy * Cfg::kWM + i * 32 + lcol] = f32x4{nb, __int_as_float(nbi), tot, __int_as_float(cnt + ocnt)};
    }
  };
  if (n0 + Cfg::kBN <= V) scan(std::true_type{});
  else scan(std::false_type{});
  if (logits) {
#pragma unroll
    for (int i = 0; i < Cfg::kTM; ++i) {
      const int m = m0 + wy * Cfg::kWM + i * 32 + lcol;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int n = nw + j * 32 + 8 * (r >> 2) + (r & 3);
          if (m < M && n < V) logits[(size_t)m * V + n] = acc.c[i][j][r];
        }
    }
  }
  lds_barrier();
  // thread (row, 128-column tile): waves 2t and 2t+1 of the row, lower columns first
  const int row = tid & 255, ct = tid >> 8;
  const int m = m0 + row, nt128 = n0 / 128 + ct;
  if (ct < Cfg::kBN / 128 && (Cfg::kBM == 256 || row < Cfg::kBM) && m < M && nt128 < NT) {
    const f32x4 a = rec[(2 * ct) * 256 + row], b = rec[(2 * ct + 1) * 256 + row];
    const float nb = fmaxf(a[0], b[0]);
    float tot = 0.f;
    if (a[0] > kNegInf) tot += a[2] * __expf(a[0] - nb);
    if (b[0] > kNegInf) tot += b[2] * __expf(b[0] - nb);
    const bool tb = b[0] > a[0];   // equal maxima: the lower columns (a) win
    f32x4 out = {nb, tb ? b[1] : a[1], tot, __int_as_float(__float_as_int(a[3]) + __float_as_int(b[3]))};
    *reinterpret_cast<f32x4*>(part + ((size_t)m * NT + nt128) * kPartF) = out;
  }
}

// A tile of 256 rows x 128 columns, or 192 x 256.
template <bool ARGMAX, class Cfg>
__device__ __forceinline__ void vocab_tile(const bf16* __restrict__ A, const bf16* __restrict__ E, int M, int V, int K, int NT, int m0, int n0,
                                           const float* __restrict__ zd_row, float* __restrict__ part, float* __restrict__ logits, bf16* smem) {
  const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float zd[Cfg::kTM];   // (requested ahead of the products)
#pragma unroll
  for (int i = 0; i < Cfg::kTM; ++i) zd[i] = zd_row ? zd_row[min(m0 + wave / Cfg::kWavesN * Cfg::kWM + i * 32 + (lane & 31), M - 1)] : kNegInf;
  GemmAcc<Cfg> acc;
  gemm_mainloop<Cfg, true>(A, K, E, K, M, V, 0, K / Cfg::GK, m0, n0, smem, acc);
  vocab_records<ARGMAX>(acc, zd, reinterpret_cast<f32x4*>(smem), lane, wave, m0, n0, M, V, NT, part, logits);
}

// 257 - 384 and 513 - 640 rows (vocab_mid.hip); stats: of the logits, else arg-max alone (zd null)
hipError_t vocab_mid(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, bool stats, const float* zd, float* part, float* logits);

}  // namespace sd
