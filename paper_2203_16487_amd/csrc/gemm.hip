// MFMA GEMM kernels of the decoder / encoder blocks and the fused vocabulary kernel.
#include "gemm_core.h"
#include "kernels.h"
#include "vocab_tiles.h"
#include <type_traits>

namespace sd {

static thread_local KernelTimer* g_kernel_timer = nullptr;
void set_kernel_timer(KernelTimer* t) { g_kernel_timer = t; }
KernelTimer* kernel_timer() { return g_kernel_timer; }

// xcd_tile for many row tiles: groups of 8 row tiles, inside a group n-major, so that what runs together on an XCD shares
// both a few weight panels and a few row panels (one long n-major run streams all rows past each weight panel: 32768 x 3072
// x 1024 on 128 x 128 tiles 276 us, grouped 247; on 256 x 256 231, grouped 212).
__device__ __forceinline__ bool xcd_tile_grouped(int id, int MT, int NT, int& mt, int& nt) {
  constexpr int G = 8;
  const int nb = MT * NT;
  const int per = (nb + 7) >> 3;
  const int t = (id & 7) * per + (id >> 3);
  if ((id >> 3) >= per || t >= nb) return false;
  const int g = t / (G * NT), r = t - g * G * NT, rows = min(G, MT - g * G);
  nt = r / rows;
  mt = g * G + r - nt * rows;
  return true;
}

// fp32 staging tile in LDS, [BM][BN]; rows r and r+4 come from the two lane halves of one
// MFMA register, so bit 5 of the column is flipped for every other group of 4 rows.
template <int BN>
__device__ __forceinline__ int cs_off(int row, int col) {
  return row * BN + (col ^ (((row >> 2) & 1) << 5));
}

// ----------------------------------------------------------------------------- epilogues
// An epilogue handles 8 consecutive columns [n, n+8) of row m (n % 8 == 0, inside the matrix)
// in two steps: fetch() issues every global read the chunk needs (bias, residual, row
// bookkeeping), store() consumes them.  The kernel calls fetch() for all chunks of a thread
// before the first store(), so the reads of a tile cost one memory round trip in total.
struct EpiF32 {
  const bf16* __restrict__ bias;
  const float* resid;   // may alias out
  float* out;
  int ldo;
  struct Pre { bf16x8 b; f32x4 r0, r1; };
  __device__ __forceinline__ Pre fetch(int m, int n) const {
    Pre p;
    p.b = *reinterpret_cast<const bf16x8*>(bias + n);
    const size_t o = (size_t)m * ldo + n;
    if (resid) { p.r0 = *reinterpret_cast<const f32x4*>(resid + o); p.r1 = *reinterpret_cast<const f32x4*>(resid + o + 4); }
    else { p.r0 = f32x4{0.f, 0.f, 0.f, 0.f}; p.r1 = p.r0; }
    return p;
  }
  __device__ __forceinline__ void store(int m, int n, const float (&v)[8], const Pre& p) const {
    f32x4 w0, w1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w0[i] = v[i] + (float)p.b[i] + p.r0[i];
      w1[i] = v[4 + i] + (float)p.b[4 + i] + p.r1[i];
    }
    const size_t o = (size_t)m * ldo + n;
    *reinterpret_cast<f32x4*>(out + o) = w0;
    *reinterpret_cast<f32x4*>(out + o + 4) = w1;
  }
};

__device__ __forceinline__ bf16x8 pack_bias(const float (&v)[8], const bf16x8& b, bool relu) {
  bf16x8 o;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float t = v[i] + (float)b[i];
    if (relu) t = fmaxf(t, 0.f);
    o[i] = (bf16)t;
  }
  return o;
}

struct EpiBf16 {
  const bf16* __restrict__ bias;
  bf16* __restrict__ out;
  int ldo;
  int relu;
  struct Pre { bf16x8 b; };
  __device__ __forceinline__ Pre fetch(int m, int n) const {
    return Pre{*reinterpret_cast<const bf16x8*>(bias + n)};
  }
  __device__ __forceinline__ void store(int m, int n, const float (&v)[8], const Pre& p) const {
    *reinterpret_cast<bf16x8*>(out + (size_t)m * ldo + n) = pack_bias(v, p.b, relu != 0);
  }
};

// Decoder self-attention projection: columns [0,d) are queries, [d,2d) keys, [2d,3d) values.
// Keys and values go straight into the cache rows of the token they belong to: this is the
// "append" of the KV cache, fused into the projection.  Both caches are [B][H][Lcap][64].
struct EpiQkvAppend {
  const bf16* __restrict__ bias;
  bf16* __restrict__ q;
  bf16* __restrict__ kc;
  bf16* __restrict__ vc;
  const int* __restrict__ row_b;
  const int* __restrict__ row_pos;
  int d, H, Lcap;
  struct Pre { bf16x8 b; int sb, pos; };
  __device__ __forceinline__ Pre fetch(int m, int n) const {
    return Pre{*reinterpret_cast<const bf16x8*>(bias + n), row_b[m], row_pos[m]};
  }
  __device__ __forceinline__ void store(int m, int n, const float (&v)[8], const Pre& p) const {
    const bf16x8 o = pack_bias(v, p.b, false);
    const int part = n / d, c = n - part * d;
    if (part == 0) {
      *reinterpret_cast<bf16x8*>(q + (size_t)m * d + c) = o;
      return;
    }
    if (p.sb < 0) return;
    const int h = c >> 6, e = c & 63;
    bf16* cache = (part == 1) ? kc : vc;
    *reinterpret_cast<bf16x8*>(cache + (((size_t)p.sb * H + h) * Lcap + p.pos) * kHeadDim + e) = o;
  }
};

template <class Cfg, class Epi>
__global__ __launch_bounds__(Cfg::kThreads) void gemm_kernel(const bf16* __restrict__ A, int lda,
                                                             const bf16* __restrict__ W, int ldw,
                                                             int M, int N, int K, int MT, int NT,
                                                             Epi epi, const int* __restrict__ m_real) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  static_assert(Cfg::kSmemBytes >= Cfg::kBM * Cfg::kBN * 4, "staging tile must fit in the ring");
  int mt, nt;
  if (!xcd_tile(blockIdx.x, MT, NT, mt, nt)) return;
  const int m0 = mt * Cfg::kBM, n0 = nt * Cfg::kBN;
  if (m_real) {   // only the leading *m_real rows hold data (same value for the whole grid)
    M = min(M, *m_real);
    if (m0 >= M) return;
  }
  constexpr int CPR = Cfg::kBN / 8;                          // 8-column chunks per row
  constexpr int ITER = Cfg::kBM * CPR / Cfg::kThreads;       // chunks per thread
  static_assert(Cfg::kBM * CPR % Cfg::kThreads == 0, "tile / thread count");
  // what the epilogue reads from memory is requested before the K loop and arrives under it
  typename Epi::Pre pre[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int idx = it * Cfg::kThreads + threadIdx.x;
    const int r = idx / CPR, c = (idx - r * CPR) * 8;
    pre[it] = epi.fetch(min(m0 + r, M - 1), min(n0 + c, N - 8));
  }
  GemmAcc<Cfg> acc;
  gemm_mainloop<Cfg>(A, lda, W, ldw, M, N, 0, K / Cfg::GK, m0, n0, smem, acc);
  float* cs = reinterpret_cast<float*>(smem);
  gemm_foreach<Cfg>(acc, 0, 0, [&](int r, int c, float v) { cs[cs_off<Cfg::kBN>(r, c)] = v; });
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int idx = it * Cfg::kThreads + threadIdx.x;
    const int r = idx / CPR, c = (idx - r * CPR) * 8;
    const int m = m0 + r, n = n0 + c;
    if (m < M && n < N) {
      const float* src = cs + cs_off<Cfg::kBN>(r, c);
      f32x4 a = *reinterpret_cast<const f32x4*>(src), b = *reinterpret_cast<const f32x4*>(src + 4);
      const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      epi.store(m, n, v, pre[it]);
    }
  }
}

typedef GemmCfg<128, 128, 2> CfgWide;      // 64 KB LDS: two blocks per CU
typedef GemmCfg<64, 64, 4> CfgSmall;       // 64 KB LDS; many tiles for narrow outputs

template <class Cfg, class Epi>
static hipError_t launch_cfg(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K,
                             const Epi& epi, const int* m_real) {
  // (initialisation of a function-local static is thread-safe)
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_kernel<Cfg, Epi>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kSmemBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + Cfg::kBM - 1) / Cfg::kBM, NT = (N + Cfg::kBN - 1) / Cfg::kBN;
  SD_LAUNCH_TIMED((gemm_kernel<Cfg, Epi>), dim3(xcd_grid(MT, NT)), dim3(Cfg::kThreads), Cfg::kSmemBytes, st,
                     A, lda, W, K, M, N, K, MT, NT, epi, m_real);
  return hipGetLastError();
}

template <class Epi>
static hipError_t launch(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K,
                         const Epi& epi, const int* m_real = nullptr) {
  if (M <= 0 || N <= 0) return hipSuccess;
  // enough 128x128 tiles to give every CU one?  else take 64x64 tiles
  const long wide_tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  // (a K of 512 is eight stages: a launch is then mostly its tiles' fixed costs, and the small tiles' are smaller)
  if (wide_tiles >= 200 && K > 512) return launch_cfg<CfgWide>(st, A, lda, W, M, N, K, epi, m_real);
  return launch_cfg<CfgSmall>(st, A, lda, W, M, N, K, epi, m_real);
}

hipError_t gemm_f32(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K,
                    const bf16* bias, const float* resid, float* out, int ldo, const int* m_real) {
  return launch(st, A, lda, W, M, N, K, EpiF32{bias, resid, out, ldo}, m_real);
}
hipError_t gemm_bf16(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K,
                     const bf16* bias, bf16* out, int ldo, bool relu, const int* m_real) {
  return launch(st, A, lda, W, M, N, K, EpiBf16{bias, out, ldo, relu ? 1 : 0}, m_real);
}
hipError_t gemm_qkv_append(hipStream_t st, const bf16* A, const bf16* W, int M, int d, int K,
                           const bf16* bias, bf16* q_out, bf16* kc, bf16* vc, const int* row_b,
                           const int* row_pos, int H, int Lcap, const int* m_real) {
  return launch(st, A, K, W, M, 3 * d, K, EpiQkvAppend{bias, q_out, kc, vc, row_b, row_pos, d, H, Lcap}, m_real);
}
// ----------------------------------------------------------------------------- LayerNorm folded into the GEMMs
// Post-LN blocks: x' = LN(y), y = x + sublayer(x).  Instead of a pass of its own over y, the
// normalisation is split between the GEMM that produces y and the GEMMs that consume x':
//   producer (EpiLnSum)   writes y (fp32), bf16(y * g) and, for every 64- (or 32-) column chunk of every row,
//                         the pair {sum, sum of squared deviations from the chunk mean};
//   consumer (EpiLn*)     multiplies bf16(y * g) by the unchanged weights and finishes
//                         LN(y) W^T + b = rstd * (acc - mean * cs) + bf,
//                         cs[n] = sum_k g[k] W[n][k],  bf[n] = b[n] + sum_k beta[k] W[n][k]
//                         (both fp32, derived once per model by ln_fold);
//   the residual x' that the next producer adds is recomputed there from y, mean, rstd, g, beta.
// bf16(y * g) rounds y with its mean, LayerNorm before the rounding would have taken it out: the operand's relative error is
// sqrt(1 + (mean / standard deviation)^2) times as large.  What shifts every row alike, the mean of the shift beta and of the bias
// b, is therefore left out of y (LayerNorm does not see it), and so is the mean of the embedded rows (embed_row).  What remains
// is what gains and the columns of a matrix have in common, which has no gradient through a LayerNorm.  Error of logits and encoder
// memories against 64 bits, 6 + 6 layers, d = 512 and 1024, as LayerNorm before the rounding leaves it / so: 1.85 - 2.4e-3 / the
// same for weights as initialised, biases of 2, gains of 1 +- 0.3 (with the biases' means left in y: 2.2 - 3.4e-3 at biases of 2);
// 1.9 / 1.8e-3 at shifts of 2; 2.35 / 2.40e-3 for matrices whose columns are all off by 4 standard deviations.
// mean and rstd of a row come from its chunk pairs, merged with the parallel-variance formula;
// eps = 1e-5 and the biased variance, as in layer_norm.  Epilogues run with every wave of the
// chip at the same point and nothing to overlap with, so they are written for few instructions:
// per row {rstd, -mean * rstd}, per column folded constants, fused multiply-adds.
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Sums over aligned groups of 2, 4 or 8 neighbouring lanes with DPP moves (no LDS round trip).
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(LANES == 2 || LANES == 4 || LANES == 8 || LANES == 16 || LANES == 32, "group size");
  v += dpp_f<kDppSwap1>(v);
  if (LANES >= 4) v += dpp_f<kDppSwap2>(v);
  if (LANES >= 8) v += dpp_f<kDppHalfMirror>(v);
  if (LANES >= 16) v += dpp_f<kDppMirror>(v);
  if (LANES >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// V consecutive columns (V = 2, 4 or 8; addresses aligned to V elements) as whole words
template <int V>
__device__ __forceinline__ void load_cols(const float* p, float (&o)[V]) { __builtin_memcpy(o, __builtin_assume_aligned(p, V == 2 ? 8 : 16), V * 4); }
template <int V>
__device__ __forceinline__ void store_cols(float* p, const float (&v)[V]) { __builtin_memcpy(__builtin_assume_aligned(p, V == 2 ? 8 : 16), v, V * 4); }
// (As a vector from the start: a copy of the array may be stored in pieces, as it was in the QKV projection, in 8, 4 and 2 bytes:
// 1408 x 3072 x 1024 on 256 x 128 tiles 21.8 us, now 20.6.)
template <int V>
__device__ __forceinline__ void store_cols(bf16* p, const bf16 (&v)[V]) {
  typedef bf16 vec __attribute__((ext_vector_type(V)));
  vec t;
#pragma unroll
  for (int i = 0; i < V; ++i) t[i] = v[i];
  *reinterpret_cast<vec*>(p) = t;
}

// Chunk pairs of a row lie together, [M][pitch] pairs with pitch = chunks rounded up to even, so a thread fetches two
// pairs per 16-byte load.  A chunk is 64 columns, or 32 where the kernel that formed the sums has tiles of 32 columns
// (few rows): wider chunks are fewer bytes for every consumer (256 rows x 32 pairs are 64 KB per 256 x 128 tile).
__host__ __device__ __forceinline__ int ln_pitch(int chunks) { return (chunks + 1) & ~1; }

// Mean and rstd of one row from its chunk pairs (the parallel-variance formula): TPR neighbouring threads hold pairs
// 2q, 2q+1 for q = j + i * TPR in p; the first of them writes {rstd, -mean * rstd} ({1, 0} for identity: nothing to
// normalise).
template <int TPR, int NL>
__device__ __forceinline__ void ln_row_stats(const f32x4 (&p)[NL], int j, int d, int chunks, bool identity, bool writer,
                                             float* out) {
  const float inv_d = __builtin_amdgcn_rcpf((float)d);   // exact for powers of two
  const float cw = d == 32 * chunks ? 32.f : 64.f, inv_cw = d == 32 * chunks ? 1.f / 32 : 1.f / 64;   // chunk width
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if (2 * i * TPR >= chunks) continue;
    const int c = 2 * (j + i * TPR);
    s += (c < chunks ? p[i][0] : 0.f) + (c + 1 < chunks ? p[i][2] : 0.f);
  }
  s = group_sum<TPR>(s);
  const float mean = s * inv_d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if (2 * i * TPR >= chunks) continue;
    const int c = 2 * (j + i * TPR);
    const float d0 = p[i][0] * inv_cw - mean, d1 = p[i][2] * inv_cw - mean;
    q += (c < chunks ? p[i][1] + cw * d0 * d0 : 0.f) + (c + 1 < chunks ? p[i][3] + cw * d1 * d1 : 0.f);
  }
  q = group_sum<TPR>(q);
  if (writer && j == 0) {
    const float rstd = identity ? 1.f : fast_rsqrt(q * inv_d + 1e-5f);
    out[0] = rstd;
    out[1] = identity ? 0.f : -mean * rstd;
  }
}

// PAIRS: most chunks of a row.
template <class Cfg, int PAIRS>
struct LnRows {
  static constexpr int TPR = Cfg::kThreads / Cfg::kBM;   // threads that share one tile row
  static constexpr int NL = PAIRS / 2 / TPR;             // 16-byte loads per thread
  static_assert(TPR == 2 || TPR == 4, "threads per row");
  f32x4 p[NL];                                           // pairs 2q, 2q+1 for q = j + i * TPR
  // Loads sit behind conditions on kernel arguments only (no lane takes a branch of its own).
  __device__ __forceinline__ void request(const f32x2* part, int chunks, int m0, int M) {
    const int r = threadIdx.x / TPR, j = threadIdx.x % TPR;
    const f32x4* src = reinterpret_cast<const f32x4*>(part + (size_t)min(m0 + r, M - 1) * ln_pitch(chunks));
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      p[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (2 * i * TPR < chunks) p[i] = src[min(j + i * TPR, ln_pitch(chunks) / 2 - 1)];
    }
  }
  // rowstat [BM][2] in LDS
  __device__ __forceinline__ void finish(int d, int chunks, bool identity, float* rowstat) const {
    ln_row_stats<TPR, NL>(p, threadIdx.x % TPR, d, chunks, identity, true, rowstat + 2 * (threadIdx.x / TPR));
  }
};

// Producer.  x holds the previous sum y_prev (or the plain residual when has_prev is 0) and
// receives the new sum in place.  Column vectors (LnSumVecs, fp32 [3][d]):
//   0: gain of the LayerNorm pending on x (1 without one)
//   1: its shift (0 without one) + this GEMM's bias, less the mean of both over the columns
//   2: gain of the LayerNorm that follows
// An epilogue handles V consecutive columns of one row; CW / V neighbouring lanes hold one chunk of CW columns.
struct EpiLnSum {
  static constexpr int kVec = 3;
  const float* __restrict__ vecs;
  const f32x2* ln_in;              // chunk pairs of y_prev
  f32x2* ln_out;                   // chunk pairs of the new sum
  float* x;
  bf16* __restrict__ xg;           // bf16(y * next gain)
  int ld, chunks;                  // d; chunks of y_prev
  int has_prev;                    // 0: x is the residual itself
  __device__ __forceinline__ int d_ln() const { return ld; }
  __device__ __forceinline__ const float* vec(int i) const { return vecs + i * ld; }
  __device__ __forceinline__ bool identity() const { return has_prev == 0; }
  template <int V> struct Pre { float r[V]; };
  template <int V>
  __device__ __forceinline__ void fetch(int m, int n, Pre<V>& p) const { load_cols<V>(x + (size_t)m * ld + n, p.r); }
  // called by every lane (live = inside the matrix): the chunk sums cross lanes
  template <int V, int CW>
  __device__ __forceinline__ void store(int m, int n, bool live, const float (&v)[V], const Pre<V>& p,
                                        float rstd, float nmr, const float (&cv)[kVec][V]) const {
    float y[V], s = 0.f, ss = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      y[i] = v[i] + __builtin_fmaf(__builtin_fmaf(p.r[i], rstd, nmr), cv[0][i], cv[1][i]);
      s += y[i];
      ss = __builtin_fmaf(y[i], y[i], ss);
    }
    s = group_sum<CW / V>(s);
    ss = group_sum<CW / V>(ss);
    if (!live) return;
    const size_t o = (size_t)m * ld + n;
    store_cols<V>(x + o, y);
    bf16 g[V];
#pragma unroll
    for (int i = 0; i < V; ++i) g[i] = (bf16)(y[i] * cv[2][i]);
    store_cols<V>(xg + o, g);
    // squared deviations from the chunk mean = sum y^2 - (sum y)^2 / CW, never below 0
    if (n % CW == 0) ln_out[(size_t)m * ln_pitch(ld / CW) + n / CW] = f32x2{s, fmaxf(ss - s * s * (1.0f / CW), 0.f)};
  }
  // gemm_tile_kernel: four columns of a row, 16 neighbouring lanes the row's chunk of 64; keep: the lane that writes the chunk's pair
  __device__ __forceinline__ void tile_line(int m, int n, bool live, const f32x4& a, const f32x4& p, const f32x4 (&cv)[kVec], float rstd,
                                            float nmr, bool keep, f32x2& pair) const {
    f32x4 y;
    bf16x4 g;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[e] = a[e] + __builtin_fmaf(__builtin_fmaf(p[e], rstd, nmr), cv[0][e], cv[1][e]);
      g[e] = (bf16)(y[e] * cv[2][e]);
    }
    const float s = group_sum<16>((y[0] + y[1]) + (y[2] + y[3]));
    const float ss = group_sum<16>(__builtin_fmaf(y[0], y[0], y[1] * y[1]) + __builtin_fmaf(y[2], y[2], y[3] * y[3]));
    pair = f32x2{keep ? s : pair[0], keep ? fmaxf(ss - s * s * (1.0f / 64), 0.f) : pair[1]};
    if (!live) return;
    const size_t o = (size_t)m * ld + n;
    *reinterpret_cast<f32x4*>(x + o) = y;
    *reinterpret_cast<bf16x4*>(xg + o) = g;
  }
  __device__ __forceinline__ void tile_pair(int m, int n, const f32x2& pair) const { ln_out[(size_t)m * ln_pitch(ld / 64) + n / 64] = pair; }
};

// rstd * (acc - mean * cs) + bf on V columns: cv[0] = cs, cv[1] = bf
template <int V>
__device__ __forceinline__ void ln_finish(const float (&v)[V], float rstd, float nmr, const float (&cv)[2][V],
                                          bool relu, bf16 (&o)[V]) {
#pragma unroll
  for (int i = 0; i < V; ++i) {
    float t = __builtin_fmaf(v[i], rstd, __builtin_fmaf(nmr, cv[0][i], cv[1][i]));
    if (relu) t = fmaxf(t, 0.f);
    o[i] = (bf16)t;
  }
}

// The same on a lane's 16 columns of a 32-column block: columns 8 half .. + 7 and 16 + 8 half .. + 7 of the block.
__device__ __forceinline__ void ln_finish_block(const f32x16& a, float rstd, float nmr, const f32x4 (&cv)[2][4], float floor,
                                                bf16x8 (&o)[2]) {
  bf16x4 g[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      g[q][e] = (bf16)fmaxf(__builtin_fmaf(a[4 * q + e], rstd, __builtin_fmaf(nmr, cv[0][q][e], cv[1][q][e])), floor);
    }
  o[0] = join_halves(g[0], g[1]);
  o[1] = join_halves(g[2], g[3]);
}

struct EpiLnBf16 {
  static constexpr int kVec = 2;
  const float* __restrict__ cs;
  const float* __restrict__ bf;
  const f32x2* ln_in;
  bf16* __restrict__ out;
  int ldo, d, chunks, relu;
  int has_prev;                    // 0: A holds the input itself, no LayerNorm pending on it
  __device__ __forceinline__ int d_ln() const { return d; }
  __device__ __forceinline__ const float* vec(int i) const { return i == 0 ? cs : bf; }
  __device__ __forceinline__ bool identity() const { return has_prev == 0; }
  template <int V> struct Pre {};
  template <int V>
  __device__ __forceinline__ void fetch(int, int, Pre<V>&) const {}
  template <int V, int CW>
  __device__ __forceinline__ void store(int m, int n, bool live, const float (&v)[V], const Pre<V>&,
                                        float rstd, float nmr, const float (&cv)[kVec][V]) const {
    bf16 o[V];
    ln_finish<V>(v, rstd, nmr, cv, relu != 0, o);
    if (live) store_cols<V>(out + (size_t)m * ldo + n, o);
  }
  __device__ __forceinline__ bool tile_relu() const { return relu != 0; }
  static constexpr bool kStoresAll = true;   // every row inside the matrix is stored
  struct TileRow { __device__ __forceinline__ TileRow of(int) const { return {}; } };
  __device__ __forceinline__ void tile_row(int, TileRow&) const {}
  // columns nb + c .. + 7 of row m + r (m, nb: the same for the whole wave)
  __device__ __forceinline__ void tile_store(int m, int r, int nb, int c, const bf16x8& v, const TileRow&) const {
    *reinterpret_cast<bf16x8*>(reinterpret_cast<char*>(out + (size_t)m * ldo + nb) + (unsigned)(r * ldo + c) * 2u) = v;
  }
};

// Decoder self-attention projection: columns [0,d) are queries, [d,2d) keys, [2d,3d) values.
// Keys and values go straight into the cache rows of the token they belong to: this is the
// "append" of the KV cache, fused into the projection.  Both caches are [B][H][Lcap][64].
struct EpiLnQkvAppend {
  static constexpr int kVec = 2;
  const float* __restrict__ cs;
  const float* __restrict__ bf;
  const f32x2* ln_in;
  int chunks;
  int has_prev;                    // 0: A holds the input itself (embeddings), no LayerNorm pending on it
  bf16* __restrict__ q;
  bf16* __restrict__ kc;
  bf16* __restrict__ vc;
  const int* __restrict__ row_b;
  const int* __restrict__ row_pos;
  int d, H, Lcap;
  __device__ __forceinline__ int d_ln() const { return d; }
  __device__ __forceinline__ const float* vec(int i) const { return i == 0 ? cs : bf; }
  __device__ __forceinline__ bool identity() const { return has_prev == 0; }
  template <int V> struct Pre { int sb, pos; };
  template <int V>
  __device__ __forceinline__ void fetch(int m, int, Pre<V>& p) const { p.sb = row_b[m]; p.pos = row_pos[m]; }
  template <int V, int CW>
  __device__ __forceinline__ void store(int m, int n, bool live, const float (&v)[V], const Pre<V>& p,
                                        float rstd, float nmr, const float (&cv)[kVec][V]) const {
    if (!live) return;
    bf16 o[V];
    ln_finish<V>(v, rstd, nmr, cv, false, o);
    const int part = n / d, cc = n - part * d;
    if (part == 0) {
      store_cols<V>(q + (size_t)m * d + cc, o);
      return;
    }
    if (p.sb < 0) return;
    const int h = cc >> 6, e = cc & 63;
    bf16* cache = (part == 1) ? kc : vc;
    store_cols<V>(cache + (((size_t)p.sb * H + h) * Lcap + p.pos) * kHeadDim + e, o);
  }
  __device__ __forceinline__ bool tile_relu() const { return false; }
  static constexpr bool kStoresAll = false;
  struct TileRow : Pre<8> {   // of(l): lane l's
    __device__ __forceinline__ TileRow of(int l) const {
      TileRow t;
      t.sb = __shfl(this->sb, l, 64);
      t.pos = __shfl(this->pos, l, 64);
      return t;
    }
  };
  __device__ __forceinline__ void tile_row(int m, TileRow& t) const { fetch<8>(m, 0, t); }
  __device__ __forceinline__ void tile_store(int m, int r, int nb, int c, const bf16x8& v, const TileRow& t) const {
    const int part = nb / d, h = (nb - part * d) >> 6;   // (a wave's 64 columns are one head's)
    if (part != 0 && t.sb < 0) return;
    bf16* dst = part == 0 ? q + (size_t)m * d + h * kHeadDim + (unsigned)(r * d)
                          : (part == 1 ? kc : vc) + (((size_t)t.sb * H + h) * Lcap + t.pos) * kHeadDim;
    *reinterpret_cast<bf16x8*>(dst + c) = v;
  }
};

template <int VEC>
constexpr int ln_smem_bytes() { return CfgSmall::kSmemBytes + (2 * CfgSmall::kBM + VEC * CfgSmall::kBN) * 4; }

// PAIRS: 32 chunks of 64 columns are the most there can be (d <= 2048); with 32 columns, for d > 1024, up to 64.  They are held in
// registers through the main loop, so the kernel that has room for 64 is for those rows only.
template <class Epi, int PAIRS>
__global__ __launch_bounds__(CfgSmall::kThreads) void gemm_ln_kernel(const bf16* __restrict__ A, int lda,
                                                                const bf16* __restrict__ W, int ldw,
                                                                int M, int N, int K, int MT, int NT,
                                                                Epi epi, const int* __restrict__ m_real) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  typedef CfgSmall Cfg;
  static_assert(Cfg::kSmemBytes >= Cfg::kBM * Cfg::kBN * 4, "staging tile must fit in the ring");
  static_assert(Cfg::kThreads >= Epi::kVec * Cfg::kBN / 4, "one thread per 4 entries of the column vectors");
  float* rowstat = reinterpret_cast<float*>(reinterpret_cast<char*>(smem) + Cfg::kSmemBytes);   // [BM][2]
  float* colv = rowstat + 2 * Cfg::kBM;                                                          // [kVec][BN]
  int mt, nt;
  if (!xcd_tile(blockIdx.x, MT, NT, mt, nt)) return;
  const int m0 = mt * Cfg::kBM, n0 = nt * Cfg::kBN;
  if (m_real) {   // only the leading *m_real rows hold data (same value for the whole grid)
    M = min(M, *m_real);
    if (m0 >= M) return;
  }
  constexpr int CPR = Cfg::kBN / 8;                    // 8-column pieces per tile row
  constexpr int RPI = Cfg::kThreads / CPR;             // tile rows covered by one pass of the block
  constexpr int ITER = Cfg::kBM / RPI;
  static_assert(Cfg::kThreads % CPR == 0 && Cfg::kBM % RPI == 0, "tile / thread count");
  // a thread keeps its 8 columns in every pass: what depends on the column alone is computed once
  const int tr = threadIdx.x / CPR, tc = (threadIdx.x % CPR) * 8;
  const int n = n0 + tc;
  // everything the epilogue reads is requested here and arrives under the K loop
  LnRows<Cfg, PAIRS> rows;
  rows.request(epi.ln_in, epi.chunks, m0, M);
  constexpr int QPV = Cfg::kBN / 4;   // 16-byte pieces per column vector of the tile
  const bool vec_thread = threadIdx.x < Epi::kVec * QPV;
  f32x4 cvec = {0.f, 0.f, 0.f, 0.f};
  if (vec_thread) cvec = *reinterpret_cast<const f32x4*>(epi.vec(threadIdx.x / QPV) + min(n0 + (int)(threadIdx.x % QPV) * 4, N - 4));
  typename Epi::template Pre<8> pre[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) epi.template fetch<8>(min(m0 + it * RPI + tr, M - 1), min(n, N - 8), pre[it]);
  GemmAcc<Cfg> acc;
  gemm_mainloop<Cfg>(A, lda, W, ldw, M, N, 0, K / Cfg::GK, m0, n0, smem, acc);
  float* cs = reinterpret_cast<float*>(smem);
  gemm_foreach<Cfg>(acc, 0, 0, [&](int r, int c, float v) { cs[cs_off<Cfg::kBN>(r, c)] = v; });
  rows.finish(epi.d_ln(), epi.chunks, epi.identity(), rowstat);
  if (vec_thread) *reinterpret_cast<f32x4*>(colv + threadIdx.x * 4) = cvec;
  __syncthreads();
  float cv[Epi::kVec][8];
#pragma unroll
  for (int i = 0; i < Epi::kVec; ++i) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(colv + i * Cfg::kBN + tc);
    const f32x4 b = *reinterpret_cast<const f32x4*>(colv + i * Cfg::kBN + tc + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { cv[i][e] = a[e]; cv[i][4 + e] = b[e]; }
  }
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int r = it * RPI + tr, m = m0 + r;
    const float* src = cs + cs_off<Cfg::kBN>(r, tc);
    const f32x4 a = *reinterpret_cast<const f32x4*>(src), b = *reinterpret_cast<const f32x4*>(src + 4);
    const f32x2 st = *reinterpret_cast<const f32x2*>(rowstat + 2 * r);
    const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    epi.template store<8, 64>(m, n, m < M && n < N, v, pre[it], st[0], st[1], cv);
  }
}

template <int PAIRS = 32, class Epi>
static hipError_t launch_ln_small(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K,
                                const Epi& epi, const int* m_real) {
  if constexpr (PAIRS < 64) {
    if (epi.chunks > PAIRS) return launch_ln_small<64>(st, A, lda, W, M, N, K, epi, m_real);
  }
  typedef CfgSmall Cfg;
  constexpr int kBytes = ln_smem_bytes<Epi::kVec>();
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_ln_kernel<Epi, PAIRS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + Cfg::kBM - 1) / Cfg::kBM, NT = (N + Cfg::kBN - 1) / Cfg::kBN;
  SD_LAUNCH_TIMED((gemm_ln_kernel<Epi, PAIRS>), dim3(xcd_grid(MT, NT)), dim3(Cfg::kThreads), kBytes, st,
                     A, lda, W, K, M, N, K, MT, NT, epi, m_real);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- large tiles
// Many rows (encoder, prefill, full batches).  The product is formed transposed (gemm_mainloop<.., SWAP>), so a lane owns 16
// columns of one row per 32-column block, four groups of four (8 q + 4 (lane / 32) .. + 3), and a wave's 64 columns are one chunk
// of a row's statistics.  The epilogue has the whole ring to itself: a wave turns its row tiles through 16 KB of it, without barriers,
// into whole lines.  Outputs are finished in the accumulators, then 8 lanes store a row's 128 bytes; sums are finished by 16
// lanes a row, which read and write its 256 bytes of fp32.  Straight from the accumulators a store touches 32 rows, 32 bytes of each:
// 32768 x 1024 x 1024 + sum 134.8 us, now 107.5; x 4096 + 280 / 255; outputs 32768 x 4096 x 1024 279 / 265 (of which the stores are some
// 27 us, 268 MB; without any 197 for the product alone), 16384 x 3072 x 1024 99.0 / 96.5.
//   256 x 256 (8 waves, one block per CU): a third fewer LDS reads and half the L2 traffic per product of
//   128 x 128 (4 waves, two blocks per CU: one block's epilogue runs under the other's products);
//   256 x 128 and 128 x 128 with a deep ring, one block per CU, for outputs of one round of them.
// (Outputs of more than one round of 256 x 256 tiles: gemm_stream_kernel.)
typedef GemmCfg<256, 256, 2, 2, 4> CfgSquare;
typedef GemmCfg<128, 128, 4> CfgDeep;   // 128 KB LDS: one block per CU

template <class Cfg, int VEC>
constexpr int tile_smem_bytes() { return Cfg::kSmemBytes + (2 * Cfg::kBM + VEC * Cfg::kBN) * 4; }

// the tile at (m0, n0); smem: tile_smem_bytes
template <class Cfg, class Epi>
__device__ __forceinline__ void gemm_tile(const bf16* __restrict__ A, int lda, const bf16* __restrict__ W, int ldw, int M, int N, int K,
                                          int m0, int n0, const Epi& epi, bf16* smem) {
  static_assert(Cfg::kWN == 64, "a wave's columns are one statistics chunk");
  static_assert(Cfg::kThreads >= Epi::kVec * Cfg::kBN / 4, "one thread per 4 entries of the column vectors");
  constexpr int TM = Cfg::kTM, TN = Cfg::kTN, BN = Cfg::kBN;
  float* rowstat = reinterpret_cast<float*>(reinterpret_cast<char*>(smem) + Cfg::kSmemBytes);   // [BM][2]
  float* colv = rowstat + 2 * Cfg::kBM;                                                          // [kVec][BN]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lrow = lane & 31, half = lane >> 5;
  const int wm = (wave / Cfg::kWavesN) * Cfg::kWM, wn = (wave % Cfg::kWavesN) * Cfg::kWN;
  GemmAcc<Cfg> acc;
  // The rows' statistics and the column vectors: requested ahead of the operands and finished behind the products where registers can hold
  // them meanwhile (1408 x 3072 x 1024 on 256 x 128 21.2 us, now 20.7; sums of 7168 x 1024 39.1 / 38.3; with the residual requested there
  // as well, ahead of the operands, 38.8); by the 256 x 256 tiles ahead of the loop.
  constexpr bool HELD = Cfg::kBM * BN < 65536;
  constexpr int QPV = BN / 4;   // 16-byte pieces per column vector of the tile
  const int t = threadIdx.x;
  LnRows<Cfg, 32> rows;
  f32x4 cvec = {0.f, 0.f, 0.f, 0.f};
  auto request = [&] {
    rows.request(epi.ln_in, epi.chunks, m0, M);
    if (t < Epi::kVec * QPV) cvec = *reinterpret_cast<const f32x4*>(epi.vec(t / QPV) + min(n0 + (t % QPV) * 4, N - 4));
  };
  auto finish = [&] {
    if (t < Epi::kVec * QPV) *reinterpret_cast<f32x4*>(colv + t * 4) = cvec;
    rows.finish(epi.d_ln(), epi.chunks, epi.identity(), rowstat);
  };
  if constexpr (HELD) {
    request();
    gemm_mainloop<Cfg, true>(A, lda, W, ldw, M, N, 0, K / Cfg::GK, m0, n0, smem, acc);
    finish();
    lds_barrier();
  } else {
    gemm_mainloop<Cfg, true>(A, lda, W, ldw, M, N, 0, K / Cfg::GK, m0, n0, smem, acc, [&] {
      request();
      finish();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // visible after the main loop's first barrier
    });
  }
  // Through 16 KB of the ring a wave, a row tile of 32 x 64 at a time, two in turn (LDS accesses of a wave are in order).
  constexpr int OWN = Cfg::kSmemBytes / Cfg::kWaves;
  static_assert(OWN >= 16384, "two fp32 row tiles");
  char* own = reinterpret_cast<char*>(smem) + wave * OWN;
  const int nb = n0 + wn;
  if constexpr (Epi::kVec == 3) {
    // sums: lane l finishes columns 4 (l % 16) .. + 3 of rows 4 p + l / 16, p = 0 .. 7
    const int r4 = lane >> 4, c4 = lane & 15;
    f32x4 cv[3], res[TM][8];
#pragma unroll
    for (int v = 0; v < 3; ++v) cv[v] = *reinterpret_cast<const f32x4*>(colv + v * BN + wn + c4 * 4);
    auto fetch = [&](int i) {
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int r = i * 32 + p * 4;
        res[i][p] = *reinterpret_cast<const f32x4*>(epi.x + (size_t)min(m0 + wm + r + r4, M - 1) * epi.ld + min(nb + c4 * 4, N - 4));
      }
    };
    fetch(0);
    fetch(1);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float* buf = reinterpret_cast<float*>(own + (i & 1) * 8192);
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16& a = acc.c[i][j];
          *reinterpret_cast<f32x4*>(buf + lrow * 64 + (((j * 8 + 2 * q + half) ^ (lrow & 15)) << 2)) = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (i + 2 < TM) fetch(i + 2);
      f32x2 pair = {0.f, 0.f};
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const int r = i * 32 + p * 4;
        const f32x4 a = *reinterpret_cast<const f32x4*>(buf + (p * 4 + r4) * 64 + ((c4 ^ (((p & 3) << 2) + r4)) << 2));
        const f32x2 st = *reinterpret_cast<const f32x2*>(rowstat + 2 * (wm + r + r4));
        epi.tile_line(m0 + wm + r + r4, nb + c4 * 4, m0 + wm + r + r4 < M && nb < N, a, res[i][p], cv, st[0], st[1], c4 == p, pair);
      }
      const int m = m0 + wm + i * 32 + c4 * 4 + r4;
      if (c4 < 8 && m < M && nb < N) epi.tile_pair(m, nb, pair);
    }
  } else {
    // outputs: a lane finishes its accumulators and stores 8 columns of rows 8 p + l / 8, p = 0 .. 3
    f32x4 cv[TN][2][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int q = 0; q < 4; ++q) cv[j][v][q] = *reinterpret_cast<const f32x4*>(colv + v * BN + wn + j * 32 + 8 * q + 4 * half);
    typename Epi::TileRow tr[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) epi.tile_row(min(m0 + wm + i * 32 + lrow, M - 1), tr[i]);
    const float floor = epi.tile_relu() ? 0.f : __builtin_nanf("");   // (fmaxf of a number and NaN is the number)
    const int r8 = lane >> 3, c8 = (lane & 7) * 8;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      bf16* buf = reinterpret_cast<bf16*>(own + (i & 1) * 4096);
      const f32x2 st = *reinterpret_cast<const f32x2*>(rowstat + 2 * (wm + i * 32 + lrow));
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        bf16x8 o[2];
        ln_finish_block(acc.c[i][j], st[0], st[1], cv[j], floor, o);
#pragma unroll
        for (int q = 0; q < 2; ++q) *reinterpret_cast<bf16x8*>(buf + lrow * 64 + (((j * 4 + q * 2 + half) ^ (lrow & 7)) << 3)) = o[q];
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(buf + (p * 8 + r8) * 64 + (c8 ^ (r8 << 3)));
        const typename Epi::TileRow t = tr[i].of(p * 8 + r8);
        if (m0 + wm + i * 32 + p * 8 + r8 < M && nb + c8 < N) epi.tile_store(m0 + wm + i * 32 + p * 8, r8, nb, c8, v, t);
      }
    }
  }
}

template <class Cfg, class Epi>
__global__ __launch_bounds__(Cfg::kThreads, 2) void gemm_tile_kernel(const bf16* __restrict__ A, int lda,
                                                                     const bf16* __restrict__ W, int ldw, int M, int N, int K,
                                                                     int NT, Epi epi, const int* __restrict__ m_real) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  if (m_real) M = min(M, *m_real);   // only the leading *m_real rows hold data (same value for the whole grid)
  int mt, nt;
  if (!xcd_tile_grouped(blockIdx.x, (M + Cfg::kBM - 1) / Cfg::kBM, NT, mt, nt)) return;
  gemm_tile<Cfg, Epi>(A, lda, W, ldw, M, N, K, mt * Cfg::kBM, nt * Cfg::kBN, epi, smem);
}

template <class Cfg, class Epi>
static hipError_t launch_tile(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K, const Epi& epi,
                              const int* m_real) {
  constexpr int kBytes = tile_smem_bytes<Cfg, Epi::kVec>();
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_tile_kernel<Cfg, Epi>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + Cfg::kBM - 1) / Cfg::kBM, NT = (N + Cfg::kBN - 1) / Cfg::kBN;
  SD_LAUNCH_TIMED((gemm_tile_kernel<Cfg, Epi>), dim3(xcd_grid(MT, NT)), dim3(Cfg::kThreads), kBytes, st, A, lda, W, K, M, N, K,
                  NT, epi, m_real);
  return hipGetLastError();
}

// Outputs of more than one round of 256 x 256 tiles: a block per CU takes one tile after the other (gemm_mainloop_square).  The ring stays
// the products': a wave turns 16 rows x 64 columns at a time through 2 KB of its own, and the column vectors (and the rows' statistics, where the
// row tile changes) of the next tile have a place beside those of this one.
// As blocks of a tile each, every round began with a memory round trip (operands, the rows' statistics) and ended with the stores of all
// CUs at once, which a block has to see through before its LDS is free: 34 us a round at K = 1024, 22 at 512; now 30 and 19, of which the
// products' rate on real data (1.42 PFLOP/s, see gemm_mainloop_square) asks for 24 and 12.  us, launches in place: 32768 x 4096 x 1024 277,
// now 241; x 3072 205 / 182; 32768 x 2048 x 512 88 / 77; x 1536 (on 128 x 128 tiles before) 79 / 64; 9216 of 16384 rows x 3072 x 1024 75 / 59.
template <class Epi>
struct StreamTiles {
  typedef CfgSquare Cfg;
  static constexpr bool kStream = true;
  static constexpr int kStores = Epi::kStoresAll ? 4 * Cfg::kTM : 0;
  static constexpr int kPairs = 16;   // chunks of a row at most
  static constexpr int kOwn = 16 * 64 * 2, kVecBytes = Epi::kVec * Cfg::kBN * 4, kStatBytes = 2 * Cfg::kBM * 4;
  static constexpr int kBytes = Cfg::kSmemBytes + Cfg::kWaves * kOwn + 2 * (kVecBytes + kStatBytes);
  static_assert(kBytes <= 160 * 1024, "LDS of a CU");
  const Epi& epi;
  GemmAcc<Cfg>& acc;
  char* smem;
  int M, N, MT, NT;
  int m0, n0, m1, n1, at, flip, rflip;   // this tile, the next one; which of the XCD's run; halves of vectors and statistics in use
  bool more;
  int end;                               // of the XCD's run: where tiles of half the width begin
  __device__ __forceinline__ float* rowstat(int f) const { return reinterpret_cast<float*>(smem + Cfg::kSmemBytes + Cfg::kWaves * kOwn + f * kStatBytes); }
  __device__ __forceinline__ float* colv(int f) const { return reinterpret_cast<float*>(smem + Cfg::kSmemBytes + Cfg::kWaves * kOwn + 2 * kStatBytes + f * kVecBytes); }
  // tile `at` of the XCD's run
  __device__ __forceinline__ bool tile(int at, int& m, int& n) const {
    int mt, nt;
    if (!xcd_tile_grouped((blockIdx.x & 7) + 8 * at, MT, NT, mt, nt)) return false;
    m = mt * Cfg::kBM;
    n = nt * Cfg::kBN;
    return true;
  }
  __device__ __forceinline__ bool next(int& m, int& n) {
    at += gridDim.x >> 3;
    m1 = m0;
    n1 = n0;
    more = at < end && tile(at, m1, n1);
    m = m1;
    n = n1;
    return more;
  }
  // the first waves' requests of the column vectors, 256 columns each
  __device__ __forceinline__ void vectors(int wave, int lane, int n, int f) const {
    if (wave < Epi::kVec)
      dma16(reinterpret_cast<const bf16*>(epi.vec(wave)), (unsigned)min(n + lane * 4, N - 4) * 4u,
            __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(colv(f) + wave * Cfg::kBN)));
  }
  __device__ __forceinline__ void statistics(int m, int f) const {
    int chunks = epi.chunks;
    asm volatile("" : "+s"(chunks));   // (as fresh_lane)
    LnRows<Cfg, kPairs> rows;
    rows.request(epi.ln_in, chunks, m, M);
    rows.finish(epi.d_ln(), chunks, epi.identity(), rowstat(f));
  }
  __device__ __forceinline__ bool done() {
    constexpr int TM = Cfg::kTM, TN = Cfg::kTN, BN = Cfg::kBN;
    const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lrow = lane & 31, half = lane >> 5;
    const int wm = (wave / Cfg::kWavesN) * Cfg::kWM, wn = (wave % Cfg::kWavesN) * Cfg::kWN, nb = n0 + wn;
    const float *stat = rowstat(rflip), *cvs = colv(flip);
    if (more) {   // (ahead of the stores: loads and stores are answered in order)
      vectors(wave, lane, n1, flip ^ 1);
      if (m1 != m0) statistics(m1, rflip ^= 1);
    }
    bf16* buf = reinterpret_cast<bf16*>(smem + Cfg::kSmemBytes + wave * kOwn);
    f32x4 cv[TN][2][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int q = 0; q < 4; ++q) cv[j][v][q] = *reinterpret_cast<const f32x4*>(cvs + v * BN + wn + j * 32 + 8 * q + 4 * half);
    typename Epi::TileRow tr[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) epi.tile_row(min(m0 + wm + i * 32 + lrow, M - 1), tr[i]);
    const float floor = epi.tile_relu() ? 0.f : __builtin_nanf("");   // (fmaxf of a number and NaN is the number)
    const int r8 = lane >> 3, c8 = (lane & 7) * 8;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const f32x2 st = *reinterpret_cast<const f32x2*>(stat + 2 * (wm + i * 32 + lrow));
      bf16x8 o[TN][2];
#pragma unroll
      for (int j = 0; j < TN; ++j) ln_finish_block(acc.c[i][j], st[0], st[1], cv[j], floor, o[j]);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if ((lrow >> 4) == h) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<bf16x8*>(buf + (lrow & 15) * 64 + (((j * 4 + q * 2 + half) ^ (lrow & 7)) << 3)) = o[j][q];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int r = i * 32 + h * 16 + p * 8;
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(buf + (p * 8 + r8) * 64 + (c8 ^ (r8 << 3)));
          const typename Epi::TileRow t = tr[i].of(h * 16 + p * 8 + r8);
          if (m0 + wm + r + r8 < M && nb + c8 < N) epi.tile_store(m0 + wm + r, r8, nb, c8, v, t);
        }
      }
    }
    const bool all = Epi::kStoresAll && m0 + Cfg::kBM <= M && n0 + BN <= N;
    m0 = m1;
    n0 = n1;
    flip ^= 1;
    return all;
  }
};

// The XCD's run of `tiles` tiles, its whole rounds up to `end` and, where the round behind them is at most half full, the number of its
// tiles, which are computed as two of half the width; 0 if it is not.
__device__ __forceinline__ int half_round(int tiles, int& end) {
  const int per = (tiles + 7) >> 3, run = min(per, tiles - (int)(blockIdx.x & 7) * per), cus = gridDim.x >> 3, left = run % cus;
  const bool halves = run > cus && left != 0 && 2 * left <= cus;
  end = halves ? run - left : run;
  return halves ? left : 0;
}

template <class Epi>
__global__ __launch_bounds__(CfgSquare::kThreads, 2) void gemm_stream_kernel(const bf16* __restrict__ A, int lda,
                                                                             const bf16* __restrict__ W, int ldw, int M, int N, int K,
                                                                             int NT, Epi epi, const int* __restrict__ m_real) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  typedef CfgSquare Cfg;
  if (m_real) M = min(M, *m_real);   // only the leading *m_real rows hold data (same value for the whole grid)
  GemmAcc<Cfg> acc;
  StreamTiles<Epi> t{epi, acc, reinterpret_cast<char*>(smem), M, N, (M + Cfg::kBM - 1) / Cfg::kBM, NT, 0, 0, 0, 0, (int)blockIdx.x >> 3, 0, 0, false, 0};
  if (!t.tile(t.at, t.m0, t.n0)) return;
  const int left = half_round(t.MT * NT, t.end);
  gemm_mainloop_square<Cfg>(A, lda, W, ldw, M, N, 0, K / Cfg::GK, t.m0, t.n0, smem, acc, [&] {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    t.vectors(wave, threadIdx.x & 63, t.n0, 0);
    t.statistics(t.m0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // visible after the main loop's barriers
  }, t);
  // a last round at most half full: tiles of 256 x 128, for twice as many CUs (7168 x 3072 x 1024, 336 tiles: 61.7 us, now 56.0; 9216 of 16384
  // rows x 2048 x 512, 288 tiles, 37.7 / 34.4)
  const int i = (int)blockIdx.x >> 3;
  if (i >= 2 * left || !t.tile(t.end + (i >> 1), t.m0, t.n0)) return;
  t.n0 += (i & 1) * 128;
  if (t.n0 >= N) return;
  __syncthreads();   // the ring is everybody's again
  gemm_tile<CfgTall, Epi>(A, lda, W, ldw, M, N, K, t.m0, t.n0, epi, smem);
}

template <class Epi>
static hipError_t launch_stream(hipStream_t st, const bf16* A, int lda, const bf16* W, int M, int N, int K, const Epi& epi, const int* m_real) {
  constexpr int kBytes = std::max(StreamTiles<Epi>::kBytes, tile_smem_bytes<CfgTall, Epi::kVec>());
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_stream_kernel<Epi>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + 255) / 256, NT = (N + 255) / 256;
  SD_LAUNCH_TIMED((gemm_stream_kernel<Epi>), dim3(std::min(xcd_grid(MT, NT), 256)), dim3(CfgSquare::kThreads), kBytes, st, A, lda, W, K, M, N,
                  K, NT, epi, m_real);
  return hipGetLastError();
}

// 256 x 256 tiles or 128 x 128 ones?  Time of a full round of blocks (256 and 512) as measured over K = 512 .. 4096, us:
// 10.5 + 1.73 and 3.6 + 1.12 per 64 columns of K; 8.2 + 1.38 where a block takes tile after tile (stream); a last round costs nearly a full one
// on one block per CU, and on two the better part of one as soon as some CU has a second block.  (Sums of K = 512 take twice as long on both.
// A streamed last round that is at most half full is computed as tiles of half the width, gemm_stream_kernel, and costs 0.65 of one.)
// Of twelve row counts from 352 to 32768 and nine (N, K) of the two models, the choice was at most 3 % slower than the better of the two
// wherever it is made.  Charging that last round in full kept 11264 and 16384 rows of 1536 and 2048 x 512 on 128 x 128 tiles: encoding
// 128 sources of 128 tokens with a 512-wide encoder of 12 layers 2150 us, now 2064; 128 of 16 .. 128 tokens 1517 / 1475; 88 of 128 tokens 1682
// / 1697, of 16 .. 128 1252 / 1177; with a 1024-wide encoder level.  Where M only bounds the rows in use (bound), the sum over half, three quarters and all of it decides.
static float square_minus_wide(int M, int N, int K, bool stream) {
  const float kt = K / 64.f;
  const long sq = (long)((M + 255) / 256) * ((N + 255) / 256), wd = (long)((M + 127) / 128) * ((N + 127) / 128);
  const float round = stream && sq > 256 ? 8.2f + 1.38f * kt : 10.5f + 1.73f * kt;
  const long last = sq % 256;
  const float rounds = (float)(sq / 256) + (last == 0 ? 0.f : stream && sq > 256 && last <= 128 ? 0.65f : 1.f);
  const float t_sq = rounds * (sq < 256 ? 0.8f : 1.f) * round;
  const long rem = wd % 512;
  const float t_wd = ((float)(wd / 512) + (rem == 0 ? 0.f : rem <= 256 ? 0.6f : 1.f)) * (3.6f + 1.12f * kt);
  return t_sq - t_wd;
}
static bool square_tiles(int M, int N, int K, bool bound, bool stream = false) {
  float t = square_minus_wide(M, N, K, stream);
  if (bound) t += square_minus_wide(M / 2, N, K, stream) + square_minus_wide((int)(M * 3L / 4), N, K, stream);
  return t < 0.f;
}

// ----------------------------------------------------------------------------- cross-attention keys / values
// Keys and values of the encoder memory for up to kCrossLayers decoder layers in one launch (the layers share the memory's
// rows): xk [layer][B][H][Scap][64], xv [layer][B][H][Scap/8][64][8].  The finished tile passes through LDS as bf16.  Keys
// leave as whole rows of a head.  A block of 8 keys of the values is 1 KB of memory: a wave turns 8 tile rows x 64 columns
// with two transposing reads and stores it at once, wherever in the tile the sequence's blocks begin (single values, as
// before, only for blocks cut by the tile's edge).
// 32768 rows, d = 1024: 288 us a layer with values stored one by one; six layers now 815 us, 136 a layer.
template <class Cfg>
__global__ __launch_bounds__(Cfg::kThreads, 2) void cross_kv_kernel(const bf16* __restrict__ A, CrossKvArgs a, int M, int d,
                                                                    int NT, const int* __restrict__ m_real) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  constexpr int BM = Cfg::kBM, BN = Cfg::kBN, TM = Cfg::kTM, TN = Cfg::kTN, P = BN + 8;
  static_assert(BM * P * 2 <= Cfg::kSmemBytes + Cfg::kTailBytes, "bf16 tile in the ring");
  if (m_real) M = min(M, *m_real);
  int mt, ntl;
  if (!xcd_tile_grouped(blockIdx.x, (M + BM - 1) / BM, NT * a.layers, mt, ntl)) return;
  const int layer = ntl / NT, nt = ntl - layer * NT, m0 = mt * BM, n0 = nt * BN, N = 2 * d;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lrow = lane & 31, half = lane >> 5;
  const int wm = (wave / Cfg::kWavesN) * Cfg::kWM, wn = (wave % Cfg::kWavesN) * Cfg::kWN;
  const bf16* bias = a.b[layer];
  GemmAcc<Cfg> acc;
  gemm_mainloop<Cfg, true>(A, d, a.w[layer], d, M, N, 0, d / Cfg::GK, m0, n0, smem, acc);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    bf16x4 bv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bv[q] = *reinterpret_cast<const bf16x4*>(bias + min(n0 + wn + j * 32, N - 32) + 8 * q + 4 * half);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      bf16x4 g[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) g[q][e] = (bf16)(acc.c[i][j][4 * q + e] + (float)bv[q][e]);
      bf16* dst = smem + (wm + i * 32 + lrow) * P + wn + j * 32 + 8 * half;
      *reinterpret_cast<bf16x8*>(dst) = join_halves(g[0], g[1]);
      *reinterpret_cast<bf16x8*>(dst + 16) = join_halves(g[2], g[3]);
    }
  }
  __syncthreads();
  // a wave takes RPW rows of one 64-column strip (one head's keys or values)
  constexpr int STRIPS = BN / 64, RW = Cfg::kWaves / STRIPS, RPW = BM / RW, STEP = RPW < 64 ? RPW : 64;
  const int c0 = (wave % STRIPS) * 64, r0 = (wave / STRIPS) * RPW;
  const int part = (n0 + c0) / d, h = (n0 + c0 - part * d) >> 6, H = d >> 6;
  if (n0 + c0 >= N) return;
  bf16* out = (part == 0 ? a.xk : a.xv) + a.layer_stride * layer;
  for (int base = r0; base < r0 + RPW; base += STEP) {
    SrcRows::At at{-1, 0};   // of row base + lane
    if (lane < STEP && m0 + base + lane < M) at = a.rows.at(m0 + base + lane);
    if (part == 0) {
#pragma unroll
      for (int it = 0; it < STEP / 8; ++it) {
        const int r = it * 8 + (lane >> 3), b = __shfl(at.b, r, 64), s = __shfl(at.s, r, 64);
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(smem + (base + r) * P + c0 + (lane & 7) * 8);
        if (b >= 0) *reinterpret_cast<bf16x8*>(out + (((size_t)b * H + h) * a.Scap + s) * kHeadDim + (lane & 7) * 8) = v;
      }
      continue;
    }
    const bool head = at.b >= 0 && ((at.s & 7) == 0 || base + lane == 0);
    unsigned long long heads = __builtin_amdgcn_ballot_w64(head);
    while (heads) {
      const int l = __builtin_ctzll(heads), r = base + l;
      heads &= heads - 1;
      const int b = __builtin_amdgcn_readlane(at.b, l), s = __builtin_amdgcn_readlane(at.s, l), o = s & 7;
      bf16* dst = out + ((size_t)b * H + h) * a.Scap * kHeadDim + vt_off(s & ~7, lane);
      if (o == 0 && r + 8 <= BM) {   // whole (rows beyond the sequence's end fill key slots nobody reads)
        const bf16* src = smem + (r + ((lane >> 2) & 3)) * P + c0 + 16 * (lane >> 4) + 4 * (lane & 3);
        s16x4 v[2] = {lds_tr16(src), lds_tr16(src + 4 * P)};
        bf16x8 w;
        __builtin_memcpy(&w, v, 16);
        *reinterpret_cast<bf16x8*>(dst) = w;
      } else {
        for (int i = 0; i < 8 - o && r + i < BM && m0 + r + i < M; ++i) {
          if (a.rows.at(m0 + r + i).b != b) break;
          dst[o + i] = smem[(r + i) * P + c0 + lane];
        }
      }
    }
  }
}

template <class Cfg>
static hipError_t launch_cross_kv(hipStream_t st, const bf16* A, const CrossKvArgs& a, int M, int d, const int* m_real) {
  constexpr int kBytes = Cfg::kSmemBytes + Cfg::kTailBytes;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(cross_kv_kernel<Cfg>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + Cfg::kBM - 1) / Cfg::kBM, NT = (2 * d + Cfg::kBN - 1) / Cfg::kBN;
  SD_LAUNCH_TIMED((cross_kv_kernel<Cfg>), dim3(xcd_grid(MT, NT * a.layers)), dim3(Cfg::kThreads), kBytes, st, A, a, M, d, NT,
                  m_real);
  return hipGetLastError();
}

hipError_t gemm_cross_kv(hipStream_t st, const bf16* A, const CrossKvArgs& a, int M, int d, const int* m_real) {
  if (M <= 0 || a.layers <= 0) return hipSuccess;
  const long wide = (long)((M + 127) / 128) * ((2 * d + 127) / 128) * a.layers;
  if (wide < 200) return launch_cross_kv<CfgSmall>(st, A, a, M, d, m_real);
  if (wide >= 512 && square_tiles(M, 2 * d * a.layers, d, m_real != nullptr)) return launch_cross_kv<CfgSquare>(st, A, a, M, d, m_real);
  return launch_cross_kv<CfgWide>(st, A, a, M, d, m_real);
}

// ----------------------------------------------------------------------------- K split inside the block
// With a few hundred rows or fewer, 64 x 64 tiles whose four waves share one ring leave most CUs without a block and
// make the others walk K alone, one barrier per 64 columns.  Here the waves of a block split K: each takes every
// NW-th 64-column slab, moves its slab of the whole tile's rows into an LDS ring of its own (whole 128-byte lines,
// global -> LDS) and multiplies it without ever meeting the other waves, so that a block keeps all of its LDS in
// flight and no wave waits for another's requests.  The NW partial tiles are summed through LDS in wave order
// (bit-reproducible); LPR neighbouring lanes finish one row, V columns each, and reduce its LayerNorm statistics.
// W8: W holds E4M3 codes, one byte each, with a scale per output column (applied to the finished sum): a slab of a W row is 64
// bytes, and a fragment becomes a bf16 operand in registers.
template <int BM, int BN, int NW, int STAGES>
struct KsplitCfg {
  static constexpr int kBM = BM, kBN = BN, kWaves = NW, kThreads = 64 * NW, kStages = STAGES;
  static constexpr int kStageElems = (BM + BN) * 64;
  static constexpr int kIPW = (BM + BN) / 8;                       // requests per wave and stage
  static constexpr int kRingBytes = NW * STAGES * kStageElems * 2;
  // rows' statistics: behind the rings, or where these take all of the LDS, in what a wave's partial tile leaves of its own
  static constexpr bool kStatInRing = kRingBytes + BM * 8 > 160 * 1024;
  static constexpr int kSmemBytes = kRingBytes + (kStatInRing ? 0 : BM * 8);
  static constexpr int kV = BN / 16, kLPR = 16;                    // columns per lane, lanes per row in the epilogue
  static constexpr int kRowsPerPass = kThreads / kLPR < BM ? kThreads / kLPR : BM;
  static constexpr int kIter = BM / kRowsPerPass;
  static constexpr int kTPR = kThreads / BM >= 16 ? 16 : kThreads / BM >= 8 ? 8 : kThreads / BM >= 4 ? 4 : 2;   // statistics: threads per row
  static constexpr int kWaveRows = 64 / kTPR, kWaveF = STAGES * kStageElems / 2;   // rows whose statistics a wave forms; floats of a ring
  __device__ __forceinline__ static int stat_off(int r) { return kStatInRing ? r / kWaveRows * kWaveF + BM * BN + r % kWaveRows * 2 : kRingBytes / 4 + r * 2; }
  static_assert(BM * BN * 4 + (kStatInRing ? kWaveRows * 8 : 0) <= STAGES * kStageElems * 2, "a wave's partial tile fits its ring");
  static_assert((BN == 32 || BN == 64) && BM % 16 == 0 && BM % kRowsPerPass == 0, "tile shape");
  static_assert(kSmemBytes <= 160 * 1024, "LDS of a CU");
  // partial tile in LDS: [BM][BN] floats, 16-byte chunk c of row r at chunk c ^ (r mod chunks)
  __device__ __forceinline__ static int red_off(int r, int c) { return r * BN + ((((c >> 2) ^ r) & (BN / 4 - 1)) << 2) + (c & 3); }
};

template <class Cfg, class Epi, bool W8>
__global__ __launch_bounds__(Cfg::kThreads) void gemm_ksplit_kernel(const bf16* __restrict__ A, int lda,
                                                                    const void* __restrict__ Wv, int ldw, int M, int N,
                                                                    int K, int MT, int NT, Epi epi,
                                                                    const int* __restrict__ m_real,
                                                                    const float* __restrict__ wscale) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  // (offsets into W are in bf16 units throughout: half as many for codes)
  const bf16* __restrict__ W = static_cast<const bf16*>(Wv);
  constexpr int BM = Cfg::kBM, BN = Cfg::kBN, NW = Cfg::kWaves, S = Cfg::kStages, IPW = W8 ? BM / 8 + BN / 16 : Cfg::kIPW;
  constexpr int FA = BM / 16, FB = BN / 16, V = Cfg::kV, LPR = Cfg::kLPR, ITER = Cfg::kIter, RPP = Cfg::kRowsPerPass;
  int mt, nt;
  if (!xcd_tile(blockIdx.x, MT, NT, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * BN;
  const int mr = m_real ? *m_real : M;   // arrives with the first operands (rows below M may all be read)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 15, g = lane >> 4;
  const int slabs = K >> 6, cnt = (slabs - wave + NW - 1) / NW;   // this wave's slabs: wave, wave + NW, ...
  // request i of a stage moves tile rows 8i .. 8i + 7 (A rows, then W rows), lane -> row 8i + lane/8; the swizzled
  // chunk depends on i by its parity alone
  unsigned voff[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    if (W8 && i * 8 >= BM) {   // 16 rows of 64 codes
      const int row = (i - BM / 8) * 16 + (lane >> 2), chunk = (lane & 3) ^ ((row >> 2) & 3);
      voff[i] = (unsigned)min(row, N - 1 - n0) * (unsigned)ldw + chunk * 16;
      continue;
    }
    const int row = i * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
    voff[i] = i * 8 < BM ? (unsigned)min(row, M - 1 - m0) * (unsigned)(lda * 2) + chunk * 16
                         : (unsigned)min(row - BM, N - 1 - n0) * (unsigned)(ldw * 2) + chunk * 16;
  }
  constexpr int WS = W8 ? 32 : 64;   // a slab of a W row
  const bf16 *abase = A + (size_t)m0 * lda + wave * 64, *wbase = W + (size_t)n0 * ldw / (64 / WS) + wave * WS;
  const bf16* ring = smem + wave * (S * Cfg::kStageElems);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(const_cast<bf16*>(ring)));
  auto request = [&](int t, int slot) {
    const bf16 *as = abase + t * (NW * 64), *ws = wbase + t * (NW * WS);
    const unsigned l = lds0 + slot * (Cfg::kStageElems * 2);
#pragma unroll
    for (int i = 0; i < IPW; ++i) dma16(i * 8 < BM ? as : ws, voff[i], l + i * 1024);
  };
#pragma unroll
  for (int t = 0; t < S; ++t)
    if (t < cnt) request(t, t);
  // what the epilogue reads travels behind the first operands
  constexpr int TPR = Cfg::kTPR, NL = 32 / TPR;   // 16-byte loads of two chunk pairs per thread (d <= 2048)
  const int sr = min(tid / TPR, BM - 1), sj = tid % TPR;
  f32x4 pr[NL];
  {
    const f32x4* src = reinterpret_cast<const f32x4*>(epi.ln_in + (size_t)min(m0 + sr, M - 1) * ln_pitch(epi.chunks));
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      pr[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (2 * i * TPR < epi.chunks) pr[i] = src[min(sj + i * TPR, ln_pitch(epi.chunks) / 2 - 1)];
    }
  }
  const int r0 = (tid / LPR) % RPP, j0 = tid % LPR, n = n0 + j0 * V;
  const int nc = min(n, N - V);
  typename Epi::template Pre<V> pre[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) epi.template fetch<V>(min(m0 + it * RPP + r0, M - 1), nc, pre[it]);
  float cv[Epi::kVec][V];
#pragma unroll
  for (int i = 0; i < Epi::kVec; ++i) load_cols<V>(epi.vec(i) + nc, cv[i]);
  float wsc[V];
  if constexpr (W8) load_cols<V>(wscale + nc, wsc);
  __builtin_amdgcn_sched_barrier(0);
  f32x4 acc[FA][FB];
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int slot = 0;
  for (int t = 0; t < cnt; ++t) {
    wait_vm_stages<IPW, S - 1>(min(cnt - 1 - t, S - 1));   // (the younger epilogue requests only make this stricter)
    asm volatile("" ::: "memory");
    const bf16* st = ring + slot * Cfg::kStageElems;
    bf16x8 fa[2][FA], fb[2][FB];
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) {
#pragma unroll
      for (int j = 0; j < FB; ++j) {
        if constexpr (W8)
          fb[ss][j] = e4m3x8_to_bf16(*reinterpret_cast<const fp8x8*>(st + BM * 64 + lds_off<32>(j * 16 + lq, ss * 2 + (g >> 1)) + (g & 1) * 4));
        else
          fb[ss][j] = *reinterpret_cast<const bf16x8*>(st + lds_off<64>(BM + j * 16 + lq, ss * 4 + g));
      }
#pragma unroll
      for (int i = 0; i < FA; ++i) fa[ss][i] = *reinterpret_cast<const bf16x8*>(st + lds_off<64>(i * 16 + lq, ss * 4 + g));
    }
    auto mma = [&](int ss) {
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ss][j], fa[ss][i], acc[i][j], 0, 0, 0);
    };
    mma(0);
    if (t + S < cnt) {   // once the slot's rows are in registers it may be filled again
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      request(t + S, slot);
    }
    mma(1);
    slot = slot + 1 == S ? 0 : slot + 1;
  }
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; j += 2) mfma_settle(acc[i][j], acc[i][j + 1]);
  if (m0 >= mr) return;                  // (same for the whole block)
  M = min(M, mr);
  // D[n][m]: this lane holds row i*16 + lq, columns j*16 + 4g .. + 3; the wave's own ring takes its partial tile
  float* red = reinterpret_cast<float*>(smem);
  constexpr int kWaveF = Cfg::kWaveF;
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j)
      *reinterpret_cast<f32x4*>(red + wave * kWaveF + Cfg::red_off(i * 16 + lq, j * 16 + 4 * g)) = acc[i][j];
  ln_row_stats<TPR, NL>(pr, sj, epi.d_ln(), epi.chunks, epi.identity(), tid < BM * TPR, red + Cfg::stat_off(sr));
  lds_barrier();
  if (RPP * LPR < Cfg::kThreads && tid >= RPP * LPR) return;
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int r = it * RPP + r0, m = m0 + r;
    float v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      float t[V];
      load_cols<V>(red + w * kWaveF + Cfg::red_off(r, j0 * V), t);
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] += t[e];
    }
    if constexpr (W8) {
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] *= wsc[e];
    }
    const f32x2 rs = *reinterpret_cast<const f32x2*>(red + Cfg::stat_off(r));
    epi.template store<V, BN>(m, n, m < M && n < N, v, pre[it], rs[0], rs[1], cv);
  }
}

template <class Cfg, class Epi, bool W8 = false>
static hipError_t launch_ksplit(hipStream_t st, const bf16* A, int lda, const void* W, int M, int N, int K,
                                const Epi& epi, const int* m_real, const float* wscale = nullptr) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_ksplit_kernel<Cfg, Epi, W8>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kSmemBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + Cfg::kBM - 1) / Cfg::kBM, NT = (N + Cfg::kBN - 1) / Cfg::kBN;
  SD_LAUNCH_TIMED((gemm_ksplit_kernel<Cfg, Epi, W8>), dim3(xcd_grid(MT, NT)), dim3(Cfg::kThreads), Cfg::kSmemBytes, st, A, lda,
                  W, K, M, N, K, MT, NT, epi, m_real, wscale);
  return hipGetLastError();
}

static bool one_round(int M, int N, int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) <= 256; }

template <class Epi>
static hipError_t launch_ln(hipStream_t st, const bf16* A, int lda, const SkWeight& w, int M, int N, int K,
                            const Epi& epi, const int* m_real) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (w.scale) {   // codes: passes of a few rows only
    if (!one_round(M, N, 16, 32)) return hipErrorInvalidValue;
    return launch_ksplit<KsplitCfg<16, 32, 8, 3>, Epi, true>(st, A, lda, w.p, M, N, K, epi, m_real, w.scale);
  }
  const bf16* W = static_cast<const bf16*>(w.p);
  // K split inside the block wherever its tiles give every CU at most one block (a second round costs more than it
  // saves): the smallest tile that does.  Launches back to back, 64 x 64 ring -> K split, us: sums of N = K = 512, M = 77: 5.6 ->
  // 5.2; N = 1024, M = 128: K = 1024 7.0 -> 5.2, K = 4096 15.9 -> 7.2; M = 352: K = 1024 7.3 -> 5.9, K = 4096 16.2 -> 11.2;
  // output N = 4096, K = 1024, M = 128: 6.7 -> 5.9.
  if (one_round(M, N, 16, 32)) return launch_ksplit<KsplitCfg<16, 32, 8, 3>>(st, A, lda, W, M, N, K, epi, m_real);
  if (one_round(M, N, 32, 32)) return launch_ksplit<KsplitCfg<32, 32, 8, 2>>(st, A, lda, W, M, N, K, epi, m_real);
  if (one_round(M, N, 32, 64)) return launch_ksplit<KsplitCfg<32, 64, 8, 1>>(st, A, lda, W, M, N, K, epi, m_real);
  if (one_round(M, N, 48, 64)) return launch_ksplit<KsplitCfg<48, 64, 4, 2>>(st, A, lda, W, M, N, K, epi, m_real);
  // a long K pays for a larger tile where the ring's tiles are more than one to a CU (FFN2 of the big model at 1408 rows: 64 x 64 ring
  // 28.0 us, with three waves 24.2; but at 1024 rows 19.2 and 22.9); at K <= 2048 the ring is level or better, and so it is where M is only a
  // bound on the rows in use.  Four waves, one to a SIMD, whose rings take all of the LDS: a verify pass of 128 x 11 rows 885 us with three, now 876 (x 1024 x
  // 1024 so as well, in place of the 64 x 64 ring: 890).  The four partial sums, of other slabs than the three, are added in another order: statistics of a
  // pass of 1408 rows move by 7e-5 - 1.6e-4 (2-norm, relative), as far as they are from those in 64 bits (8.5e-5 - 1.8e-4 with three, 8.2e-5 - 1.8e-4
  // with four).  What a CU takes in bounds it, some 64 B/ns: fragments of a slab read under the products of the one
  // before it were slower (886).
  if constexpr (Epi::kVec == 3) {
    if (K >= 4096 && !m_real && !one_round(M, N, 64, 64) && one_round(M, N, 96, 64)) return launch_ksplit<KsplitCfg<96, 64, 4, 2>>(st, A, lda, W, M, N, K, epi, m_real);
  }
  // From 512 tiles of 128 x 128 on: two of them a CU, or 256 x 256.  Below: 256 x 128 while those are at most one to a CU, 128 x 128 with a
  // ring of four, one to a CU, while these are, and 64 x 64, two to a CU, while those are.  us on 64 x 64 / 128 x 128 ring of four /
  // 256 x 128 / 128 x 128 two to a CU (x N x K, "+" a sum; of 128 x 128 tiles):
  //   2048 x 1024 x 1024 (128) 10.8 / 12.7 / 17.1 / 12.5;  1408 x 1536 x 512 (132) 9.7 / 8.7 / 10.5 / 9.1;  1024 x 3072 x 1024 (192)
  //   14.0 / 12.4 / 15.9 / 13.7;  4096 x 1024 x 1024 (256) 24.0 / 14.0 / 17.3 / 14.0;  2816 x 1024 x 4096 + (176) 56.3 / 35.2 / 48.5 / 49.3
  //   2816 x 1536 x 512 (264) 13.9 / 16.4 / 11.6 / 12.9;  9216 x 512 x 512 + (288) 24.4 / 22.9 / 17.6 / 18.4;  7168 x 1024 x 4096 + (448)
  //   147 / 72.2 / 62.5 / 66.0;  16384 x 512 x 512 (512) 26.6 / 20.1 / 16.1 / 15.1
  // (512 of a sum, where 256 x 128 is exactly one round: that.  x 512 x 2048 and x 512 x 512, mean, against 128 x 128: 9216 of 16384 rows
  // in use 28.7 / 31.6, all of a bound 35.3 / 36.8, 16384 without one 31.0 / 32.1)
  const long wide_tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  if (epi.chunks > 32) return launch_ln_small(st, A, lda, W, M, N, K, epi, m_real);   // (sums of so many rows come in fewer chunks)
  if (wide_tiles > 512 || (wide_tiles == 512 && !(Epi::kVec == 3 && one_round(M, N, 256, 128)))) {
    bool stream = false;
    if constexpr (Epi::kVec == 2) stream = K % 128 == 0 && K >= 256 && epi.chunks <= StreamTiles<Epi>::kPairs && !one_round(M, N, 256, 256);
    if (square_tiles(M, N, K, m_real != nullptr, stream)) {
      if constexpr (Epi::kVec == 2) {
        if (stream) return launch_stream(st, A, lda, W, M, N, K, epi, m_real);
      }
      return launch_tile<CfgSquare>(st, A, lda, W, M, N, K, epi, m_real);
    }
    return launch_tile<CfgWide>(st, A, lda, W, M, N, K, epi, m_real);
  }
  if (wide_tiles > 256) {
    if (one_round(M, N, 256, 128)) return launch_tile<CfgTall>(st, A, lda, W, M, N, K, epi, m_real);
    return launch_tile<CfgWide>(st, A, lda, W, M, N, K, epi, m_real);
  }
  if (wide_tiles > 128) return launch_tile<CfgDeep>(st, A, lda, W, M, N, K, epi, m_real);
  return launch_ln_small(st, A, lda, W, M, N, K, epi, m_real);
}

int ln_sum_chunks(int M, int d) { return one_round(M, d, 32, 32) ? d / 32 : d / 64; }
hipError_t gemm_ln_sum(hipStream_t st, const bf16* A, int lda, const SkWeight& W, int M, int d, int K,
                       const float* vecs, LnPairs ln_in, float* x, bf16* xg, float* ln_out, const int* m_real) {
  return launch_ln(st, A, lda, W, M, d, K,
                   EpiLnSum{vecs, reinterpret_cast<const f32x2*>(ln_in.p), reinterpret_cast<f32x2*>(ln_out), x, xg, d,
                            ln_in.chunks > 0 ? ln_in.chunks : d / 64, ln_in.chunks > 0}, m_real);
}
hipError_t gemm_ln_bf16(hipStream_t st, const bf16* A, const SkWeight& W, int M, int N, int d, const LnFold& f,
                        LnPairs ln_in, bf16* out, int ldo, bool relu, const int* m_real) {
  return launch_ln(st, A, d, W, M, N, d,
                   EpiLnBf16{f.cs, f.bf, reinterpret_cast<const f32x2*>(ln_in.p), out, ldo, d,
                             ln_in.chunks > 0 ? ln_in.chunks : d / 64, relu ? 1 : 0, ln_in.chunks > 0}, m_real);
}
hipError_t gemm_ln_qkv_append(hipStream_t st, const bf16* A, const SkWeight& W, int M, int d, const LnFold& f,
                              LnPairs ln_in, bf16* q_out, bf16* kc, bf16* vc, const int* row_b,
                              const int* row_pos, int H, int Lcap, const int* m_real) {
  return launch_ln(st, A, d, W, M, 3 * d, d,
                   EpiLnQkvAppend{f.cs, f.bf, reinterpret_cast<const f32x2*>(ln_in.p),
                                  ln_in.chunks > 0 ? ln_in.chunks : d / 64, ln_in.chunks > 0, q_out,
                                  kc, vc, row_b, row_pos, d, H, Lcap}, m_real);
}

// cs[n] = sum_k g[k] W[n][k],  bf[n] = b[n] + sum_k beta[k] W[n][k]; one wave per column n
__global__ __launch_bounds__(256) void ln_fold_kernel(const bf16* __restrict__ W, const bf16* __restrict__ g,
                                                      const bf16* __restrict__ beta, const bf16* __restrict__ b,
                                                      int N, int K, float* __restrict__ cs, float* __restrict__ bf) {
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= N) return;
  const bf16* w = W + (size_t)n * K;
  if (!g) {   // no LayerNorm in front: the plain bias
    if (lane == 0) { cs[n] = 0.f; bf[n] = (float)b[n]; }
    return;
  }
  float s = 0.f, t = 0.f;
  for (int k = lane; k < K; k += 64) {
    const float wk = (float)w[k];
    s += (float)g[k] * wk;
    t += (float)beta[k] * wk;
  }
  s = wave_sum(s);
  t = wave_sum(t);
  if (lane == 0) { cs[n] = s; bf[n] = (float)b[n] + t; }
}
hipError_t ln_fold(hipStream_t st, const bf16* W, const bf16* g, const bf16* beta, const bf16* b, int N, int K,
                   const LnFold& out) {
  hipLaunchKernelGGL(ln_fold_kernel, dim3((N + 3) / 4), dim3(256), 0, st, W, g, beta, b, N, K,
                     const_cast<float*>(out.cs), const_cast<float*>(out.bf));
  return hipGetLastError();
}

// The same for a matrix stored as codes: value = scale[n] * decode(code[n][k]).
__global__ __launch_bounds__(256) void ln_fold8_kernel(const fp8* __restrict__ W, const float* __restrict__ scale,
                                                       const bf16* __restrict__ g, const bf16* __restrict__ beta,
                                                       const bf16* __restrict__ b, int N, int K, float* __restrict__ cs,
                                                       float* __restrict__ bf) {
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= N) return;
  float s = 0.f, t = 0.f;
  if (g)
    for (int k = lane * 8; k < K; k += 512) {
      const bf16x8 w = e4m3x8_to_bf16(*reinterpret_cast<const fp8x8*>(W + (size_t)n * K + k));
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        s += (float)g[k + i] * (float)w[i];
        t += (float)beta[k + i] * (float)w[i];
      }
    }
  s = wave_sum(s) * scale[n];
  t = wave_sum(t) * scale[n];
  if (lane == 0) { cs[n] = s; bf[n] = (float)b[n] + t; }
}
hipError_t ln_fold8(hipStream_t st, const SkWeight& W, const bf16* g, const bf16* beta, const bf16* b, int N, int K,
                    const LnFold& out) {
  hipLaunchKernelGGL(ln_fold8_kernel, dim3((N + 3) / 4), dim3(256), 0, st, static_cast<const fp8*>(W.p), W.scale, g, beta, b, N,
                     K, const_cast<float*>(out.cs), const_cast<float*>(out.bf));
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void ln_sum_vecs_kernel(const bf16* __restrict__ bias, const bf16* __restrict__ gp,
                                                          const bf16* __restrict__ bp, const bf16* __restrict__ gn, int d,
                                                          float* __restrict__ out) {
  __shared__ float red[4];
  float s = 0.f;
  for (int n = threadIdx.x; n < d; n += 256) s += (float)bias[n] + (bp ? (float)bp[n] : 0.f);
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  const float mean = (red[0] + red[1] + red[2] + red[3]) / (float)d;
  for (int n = threadIdx.x; n < d; n += 256) {
    out[n] = gp ? (float)gp[n] : 1.f;
    out[d + n] = (float)bias[n] + (bp ? (float)bp[n] : 0.f) - mean;
    out[2 * d + n] = (float)gn[n];
  }
}
hipError_t ln_sum_vecs(hipStream_t st, const bf16* bias, const bf16* g_prev, const bf16* b_prev, const bf16* g_next,
                       int d, float* out) {
  hipLaunchKernelGGL(ln_sum_vecs_kernel, dim3(1), dim3(256), 0, st, bias, g_prev, b_prev, g_next, d, out);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- vocabulary
// Rank test without a sort (paper Eq. 8): the draft is inside the top beta iff fewer than
// beta logits are strictly larger than its own.  Its logit z_d is needed before the big
// product is scanned, so a tiny pre-pass computes it -- with the SAME instruction sequence
// (MFMA 32x32x16, k blocks of 16 in ascending order, same operand roles) that produces that
// very element in the main kernel.  The two values are therefore bit-identical and the
// count is exactly the count over the row the main kernel sees.
//
// One wave = 32 rows: D[i][j] = x_i . E[draft_j]; the diagonal is kept.
template <bool SWAP>
__global__ __launch_bounds__(64) void draft_logit_kernel(const bf16* __restrict__ A, const bf16* __restrict__ E,
                                                         int M, int V, int K, const int* __restrict__ row_draft,
                                                         float* __restrict__ zd_out) {
  const int lane = threadIdx.x, lrow = lane & 31, lhalf = lane >> 5;
  const int r = blockIdx.x * 32 + lrow;
  const int rr = min(r, M - 1);
  const int t = row_draft[rr];
  const bool has = (r < M) && t >= 0 && t < V;
  const bf16* ap = A + (size_t)rr * K + lhalf * 8;
  const bf16* bp = E + (size_t)(has ? t : 0) * K + lhalf * 8;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  // operands of 16 k-blocks are requested together (one memory round trip per 256 columns of K
  // instead of one per block); the accumulation order stays k-ascending
  constexpr int U = 16;
  const int nkb = K / 16;
  for (int kb0 = 0; kb0 < nkb; kb0 += U) {
    bf16x8 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kb = min(kb0 + u, nkb - 1);
      a[u] = *reinterpret_cast<const bf16x8*>(ap + kb * 16);
      b[u] = *reinterpret_cast<const bf16x8*>(bp + kb * 16);
    }
    if (kb0 + U <= nkb) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        acc = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[u], a[u], acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u], b[u], acc, 0, 0, 0);
    } else {
      for (int u = 0; u < nkb - kb0; ++u) {
        bf16x8 au = a[0], bu = b[0];
#pragma unroll
        for (int v = 1; v < U; ++v) if (v == u) { au = a[v]; bu = b[v]; }
        acc = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bu, au, acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(au, bu, acc, 0, 0, 0);
      }
    }
  }
  mfma_settle(acc);
  // element (i, j): j = lane%32, i = 8*(reg/4) + 4*(lane/32) + reg%4; the diagonal j = i sits in
  // the lane half (j/4)%2, register 4*(j/8) + j%4
  if (lhalf == ((lrow >> 2) & 1) && r < M) {
    const int reg = 4 * (lrow >> 3) + (lrow & 3);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) if (i == reg) v = acc[i];
    zd_out[r] = has ? v : kNegInf;
  }
}

// The last LayerNorm and the draft logits of 16 rows in one launch: a wave normalises two rows, x in place and bf16 rows to memory and
// LDS, and the first one forms the products, in the same order and with the same instruction as above.  A chain of a few memory round
// trips and K / 16 dependent products; all loads are issued ahead of it (with the products' operands read from memory as they go,
// 14 us at 1024).  In two launches, ln_kernel and the kernel above, 2.7 - 4.8 + 4.2 - 7.2 us; here 4.7 us (352 rows of 512),
// 7.3 - 8.8 us (352 - 1408 rows of 1024).
template <int PER, bool SWAP>
__global__ __launch_bounds__(512) void ln_draft_kernel(float* __restrict__ x, const bf16* __restrict__ g, const bf16* __restrict__ b,
                                                       bf16* __restrict__ xb, const bf16* __restrict__ E, int M, int V,
                                                       const int* __restrict__ row_draft, float* __restrict__ zd_out) {
  constexpr int K = 64 * PER, P = K + 8, PIECES = K / 8, NE = 16 * PIECES / 512;   // (rows padded by 16 bytes: reads of 16 rows meet all banks)
  __shared__ __attribute__((aligned(16))) bf16 rows[16 * P], emb[16 * P];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lrow = lane & 31, lhalf = lane >> 5;
  const int r0 = blockIdx.x * 16, r = r0 + (lrow & 15);
  bf16x8 e[NE];   // the drafts' embedding rows, all at once, under the LayerNorm
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int p = threadIdx.x + i * 512, t = row_draft[min(r0 + p / PIECES, M - 1)];
    e[i] = *reinterpret_cast<const bf16x8*>(E + (size_t)(t >= 0 && t < V ? t : 0) * K + p % PIECES * 8);
  }
  float y[2][PER];
#pragma unroll
  for (int i = 0; i < 2; ++i) ln_row<PER>(x + (size_t)min(r0 + wave * 2 + i, M - 1) * K, g, b, lane, y[i]);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = r0 + wave * 2 + i;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (m < M) {
        x[(size_t)m * K + j * 64 + lane] = y[i][j];
        xb[(size_t)m * K + j * 64 + lane] = (bf16)y[i][j];
      }
      rows[(wave * 2 + i) * P + j * 64 + lane] = (bf16)y[i][j];
    }
  }
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int p = threadIdx.x + i * 512;
    *reinterpret_cast<bf16x8*>(emb + p / PIECES * P + p % PIECES * 8) = e[i];
  }
  lds_barrier();
  if (wave != 0) return;
  const int t = row_draft[min(r, M - 1)];
  const bool has = r < M && t >= 0 && t < V;
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll 8
  for (int k = 0; k < K / 16; ++k) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(rows + (lrow & 15) * P + k * 16 + lhalf * 8);
    const bf16x8 c = *reinterpret_cast<const bf16x8*>(emb + (lrow & 15) * P + k * 16 + lhalf * 8);
    acc = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(c, a, acc, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, c, acc, 0, 0, 0);
  }
  mfma_settle(acc);
  if (lrow < 16 && lhalf == ((lrow >> 2) & 1) && r < M) {   // the diagonal, as above
    const int reg = 4 * (lrow >> 3) + (lrow & 3);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) if (i == reg) v = acc[i];
    zd_out[r] = has ? v : kNegInf;
  }
}

// One block = 128 rows x 128 vocabulary columns.  After the K loop the fp32 tile goes through
// LDS so that two threads own one row (64 columns each); each scans its columns once for
// max / arg-max / number of logits above the draft's and once for the sum of exponentials, the
// two halves are merged with lane shuffles, and one 16-byte partial record per (row, tile) is
// written.  Logits never reach memory unless the caller asks for them.
typedef GemmCfg<128, 128, 2> CfgVocab;       // two blocks per CU
typedef CfgDeep CfgVocabDeep;                // where there is one to a CU at most, nothing hides its loads but its own ring: 128 KB LDS

// Staging tile of the vocabulary kernel: [128 rows][32 chunks of 4 columns], chunk ch of row r
// at chunk (ch & 16) + ((ch & 15) ^ (r & 15) ^ ((ch >> 4) << 3)): the 16 lanes that read one
// 16-byte chunk each in the same cycle (8 rows x 2 halves) then cover all 64 banks.
__device__ __forceinline__ int vs_off(int row, int ch) {
  return row * 128 + (((ch & 16) + ((ch & 15) ^ (row & 15) ^ ((ch >> 4) << 3))) << 2);
}

// ARGMAX: rows that score no draft and whose log-sum-exp nobody reads (the drafter's slots):
// only max / arg-max are formed; the record's sum is 0 and its count 0.
template <bool ARGMAX, class Cfg>
__global__ __launch_bounds__(Cfg::kThreads) void vocab_kernel(const bf16* __restrict__ A,
                                                                   const bf16* __restrict__ E, int M,
                                                                   int V, int K, int MT, int NT,
                                                                   const float* __restrict__ zd_row,
                                                                   float* __restrict__ part,
                                                                   float* __restrict__ logits) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  int mt, nt;
  if (!xcd_tile(blockIdx.x, MT, NT, mt, nt)) return;
  const int m0 = mt * 128, n0 = nt * 128;
  GemmAcc<Cfg> acc;
  gemm_mainloop<Cfg>(A, K, E, K, M, V, 0, K / Cfg::GK, m0, n0, smem, acc);
  float* cs = reinterpret_cast<float*>(smem);  // [128][128] fp32 = 64 KB
  gemm_foreach<Cfg>(acc, 0, 0, [&](int r, int c, float v) { cs[vs_off(r, c >> 2) + (c & 3)] = v; });
  __syncthreads();

  const int tid = threadIdx.x;
  const int row = tid >> 1, half = tid & 1;
  const int m = m0 + row;
  const float zd = (zd_row && m < M) ? zd_row[m] : kNegInf;   // -inf on rows that score no draft: count unused
  float best = kNegInf;
  int besti = 0x7fffffff, cnt = 0;
  const bool full = n0 + 128 <= V;
  // thread (row, half) owns columns [half*64, half*64 + 64) of its row: 16 reads of 4 columns
  f32x4 vals[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) vals[i] = *reinterpret_cast<const f32x4*>(cs + vs_off(row, half * 16 + i));
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = n0 + half * 64 + i * 4 + e;   // ascending: ">" keeps the lowest index of a tie
      const float v = vals[i][e];
      if (full || n < V) {
        if (v > best) { best = v; besti = n; }
        if (!ARGMAX) cnt += (v > zd) ? 1 : 0;
      }
    }
  float se = 0.f;
  if (!ARGMAX) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (full || n0 + half * 64 + i * 4 + e < V) se += __expf(vals[i][e] - best);
  }
  // merge the two halves of the row (lanes tid and tid^1)
  const float obest = __shfl_xor(best, 1, 64);
  const int obesti = __shfl_xor(besti, 1, 64);
  const float ose = __shfl_xor(se, 1, 64);
  const int ocnt = __shfl_xor(cnt, 1, 64);
  const float nb = fmaxf(best, obest);
  float tot = 0.f;
  if (best > kNegInf) tot += se * __expf(best - nb);
  if (obest > kNegInf) tot += ose * __expf(obest - nb);
  const int nbi = (obest > best || (obest == best && obesti < besti)) ? obesti : besti;
  if (half == 0 && m < M) {
    f32x4 rec = {nb, __int_as_float(nbi), tot, __int_as_float(cnt + ocnt)};
    *reinterpret_cast<f32x4*>(part + ((size_t)m * NT + nt) * kPartF) = rec;
  }
  if (logits) {
    for (int idx = tid; idx < 128 * 128; idx += Cfg::kThreads) {
      int r = idx >> 7, c = idx & 127;
      if (m0 + r < M && n0 + c < V) logits[(size_t)(m0 + r) * V + n0 + c] = cs[vs_off(r, c >> 2) + (c & 3)];
    }
  }
}

// Many rows (the batched verify and draft passes): one block = 256 rows x 256 vocabulary columns,
// 8 waves (2 along rows x 4 along the vocabulary), which halves what the operand tiles pull through
// L2 per output.  The product is formed transposed (gemm_mainloop<.., SWAP>): a lane then owns 32
// columns of each of its 4 rows, so a row's statistics are a serial scan of the lane's own
// accumulators -- no staging of the fp32 tile through LDS -- followed by one exchange between the lane
// halves and a merge of the two waves that share a 128-column tile through 16 KB of LDS.  The
// partial records keep the 128-column granularity of the kernel above.
// Beyond 256 tiles a block takes one after the other (STREAM, see gemm_mainloop_square): the next one's first operands arrive under the scan.
// Launches in the translation loop, a block a tile / so: 1408 rows, d = 1024 97.6 / 95.2 us, 1280 rows, d = 512, 50.2 / 47.4 (three rounds
// each; the scan, a quarter-rate exponential and six instructions per logit, is 4 us of a round, with nothing beside it).
typedef GemmCfg<256, 256, 2, 2, 4> CfgVocab256;

template <bool ARGMAX, bool STREAM>
struct VocabTiles {
  typedef CfgVocab256 Cfg;
  static constexpr bool kStream = STREAM;
  static constexpr int kStores = 0;   // (one record a lane, or logits beside it: not counted on)
  static constexpr int kBytes = Cfg::kSmemBytes + 4 * 256 * 16 + 2 * 256 * 4;
  GemmAcc<Cfg>& acc;
  char* smem;
  int M, V, MT, NT256, NT;
  const float* __restrict__ zd_row;
  float* __restrict__ part;
  float* __restrict__ logits;
  int m0, n0, m1, n1, at, flip;   // this tile, the next one; which of the XCD's run; half of zd in use
  int end;                        // of the XCD's run: where tiles of half the width begin
  __device__ __forceinline__ float* zd_rows(int f) const { return reinterpret_cast<float*>(smem + Cfg::kSmemBytes + 4 * 256 * 16) + f * 256; }
  __device__ __forceinline__ bool tile(int at, int& m, int& n) const {
    int mt, nt;
    if (!xcd_tile((blockIdx.x & 7) + 8 * at, MT, NT256, mt, nt)) return false;
    m = mt * 256;
    n = nt * 256;
    return true;
  }
  // the first wave's request of the drafts' logits of 256 rows (of rows beyond M: not used)
  __device__ __forceinline__ void drafts(int m, int f) const {
    if (zd_row && threadIdx.x < 64)
      dma16(reinterpret_cast<const bf16*>(zd_row), (unsigned)min(m + (int)threadIdx.x * 4, (M - 1) & ~3) * 4u,
            __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(zd_rows(f))));
  }
  __device__ __forceinline__ bool next(int& m, int& n) {
    at += gridDim.x >> 3;
    m1 = m0;
    n1 = n0;
    const bool more = at < end && tile(at, m1, n1);
    if (more) drafts(m1, flip ^ 1);
    m = m1;
    n = n1;
    return more;
  }
  __device__ __forceinline__ bool done() {
    finish();
    m0 = m1;
    n0 = n1;
    flip ^= 1;
    return false;
  }
  __device__ __forceinline__ void finish() const;
};

template <bool ARGMAX, bool STREAM>
__device__ __forceinline__ void VocabTiles<ARGMAX, STREAM>::finish() const {
  const int lane = fresh_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float zd[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) zd[i] = zd_row ? zd_rows(flip)[(wave >> 2) * 128 + i * 32 + (lane & 31)] : kNegInf;
  vocab_records<ARGMAX>(acc, zd, reinterpret_cast<f32x4*>(smem + Cfg::kSmemBytes), lane, wave, m0, n0, M, V, NT, part, logits);
}

// 129 - 256 rows: one block to a CU, where the vocabulary is one round of them.
template <bool ARGMAX>
__global__ __launch_bounds__(CfgTall::kThreads, 2) void vocab_tall_kernel(const bf16* __restrict__ A, const bf16* __restrict__ E, int M, int V, int K, int NT,
                                                                          const float* __restrict__ zd_row, float* __restrict__ part,
                                                                          float* __restrict__ logits) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  int mt, nt;
  if (!xcd_tile(blockIdx.x, 1, NT, mt, nt)) return;
  vocab_tile<ARGMAX, CfgTall>(A, E, M, V, K, NT, 0, nt * 128, zd_row, part, logits, smem);
}

template <bool ARGMAX, bool STREAM>
__global__ __launch_bounds__(CfgVocab256::kThreads, 2) void vocab256_kernel(const bf16* __restrict__ A,
                                                                            const bf16* __restrict__ E, int M, int V,
                                                                            int K, int MT, int NT256, int NT,
                                                                            const float* __restrict__ zd_row,
                                                                            float* __restrict__ part,
                                                                            float* __restrict__ logits) {
  extern __shared__ __attribute__((aligned(1024))) bf16 smem[];
  GemmAcc<CfgVocab256> acc;
  VocabTiles<ARGMAX, STREAM> t{acc, reinterpret_cast<char*>(smem), M, V, MT, NT256, NT, zd_row, part, logits, 0, 0, 0, 0, (int)blockIdx.x >> 3, 0, 0};
  if (!t.tile(t.at, t.m0, t.n0)) return;
  auto hook = [&] { t.drafts(t.m0, 0); };
  if constexpr (STREAM) {
    const int left = half_round(MT * NT256, t.end);
    gemm_mainloop_square<CfgVocab256>(A, K, E, K, M, V, 0, K / CfgVocab256::GK, t.m0, t.n0, smem, acc, hook, t);
    // a last round at most half full: tiles of 256 x 128, as in gemm_stream_kernel (384 tiles, 704 rows, K = 1024: 58.3 us, now 52.8; 640 of K
    // = 512, arg-max alone, 32.8 / 30.3; 378 tiles of statistics, 572 rows of 512, 36.9 / 32.8)
    const int i = (int)blockIdx.x >> 3;
    if (i >= 2 * left || !t.tile(t.end + (i >> 1), t.m0, t.n0)) return;
    t.n0 += (i & 1) * 128;
    if (t.n0 >= V) return;
    __syncthreads();   // the ring and the records are everybody's again
    vocab_tile<ARGMAX, CfgTall>(A, E, M, V, K, NT, t.m0, t.n0, zd_row, part, logits, smem);
  } else {
    gemm_mainloop_square<CfgVocab256>(A, K, E, K, M, V, 0, K / CfgVocab256::GK, t.m0, t.n0, smem, acc, hook);
    t.finish();
  }
}
template <bool ARGMAX, bool STREAM>
static hipError_t launch_vocab256(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, const float* zd, float* part, float* logits) {
  constexpr int kBytes = STREAM ? std::max(VocabTiles<ARGMAX, STREAM>::kBytes, CfgTall::kSmemBytes) : VocabTiles<ARGMAX, STREAM>::kBytes;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(vocab256_kernel<ARGMAX, STREAM>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  const int MT = (M + 255) / 256, NT = (V + 255) / 256, grid = xcd_grid(MT, NT);
  SD_LAUNCH_TIMED((vocab256_kernel<ARGMAX, STREAM>), dim3(STREAM ? std::min(grid, 256) : grid), dim3(CfgVocab256::kThreads), kBytes, st, A, E, M, V, K,
                  MT, NT, (V + 127) / 128, zd, part, logits);
  return hipGetLastError();
}

template <bool ARGMAX>
static hipError_t launch_vocab_tall(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, const float* zd, float* part, float* logits) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(vocab_tall_kernel<ARGMAX>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, CfgTall::kSmemBytes);
  if (attr != hipSuccess) return attr;
  const int NT = (V + 127) / 128;
  SD_LAUNCH_TIMED((vocab_tall_kernel<ARGMAX>), dim3(xcd_grid(1, NT)), dim3(CfgTall::kThreads), CfgTall::kSmemBytes, st, A, E, M, V, K, NT, zd, part, logits);
  return hipGetLastError();
}

int vocab_tile_cols(int) { return CfgVocab::kBN; }

template <bool ARGMAX, class Cfg>
static hipError_t launch_vocab(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, int MT, int NT, const float* zd, float* part,
                               float* logits) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(vocab_kernel<ARGMAX, Cfg>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kSmemBytes);
  if (attr != hipSuccess) return attr;
  SD_LAUNCH_TIMED((vocab_kernel<ARGMAX, Cfg>), dim3(xcd_grid(MT, NT)), dim3(Cfg::kThreads), Cfg::kSmemBytes, st, A, E, M, V, K, MT, NT, zd, part,
                  logits);
  return hipGetLastError();
}

template <bool SWAP>
static hipError_t launch_draft_logits(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K, const int* row_draft, float* zd_row,
                                      const VocabLn* ln) {
  if (ln && row_draft && (K == 512 || K == 1024)) {
    if (K == 512) hipLaunchKernelGGL((ln_draft_kernel<8, SWAP>), dim3((M + 15) / 16), dim3(512), 0, st, ln->x, ln->g, ln->b, ln->xb, E, M, V, row_draft, zd_row);
    else hipLaunchKernelGGL((ln_draft_kernel<16, SWAP>), dim3((M + 15) / 16), dim3(512), 0, st, ln->x, ln->g, ln->b, ln->xb, E, M, V, row_draft, zd_row);
    return hipGetLastError();
  }
  if (ln) {
    const hipError_t e = layer_norm(st, ln->x, ln->g, ln->b, ln->xb, M, K);
    if (e != hipSuccess) return e;
  }
  // without row_draft no row scores a draft (drafter pass): every count is taken against -inf, unused
  if (row_draft) hipLaunchKernelGGL(draft_logit_kernel<SWAP>, dim3((M + 31) / 32), dim3(64), 0, st, A, E, M, V, K, row_draft, zd_row);
  return hipGetLastError();
}

hipError_t vocab_stats(hipStream_t st, const bf16* A, const bf16* E, int M, int V, int K,
                       const int* row_draft, float* zd_row, float* part, float* logits, bool force_wide, const VocabLn* ln) {
  if (M <= 0) return hipSuccess;
  const bool stats = row_draft || logits;
  const int MT = (M + 127) / 128, NT = (V + 127) / 128;
  // 256 x 256 tiles once they give every CU one (the batched passes); their product is formed with
  // the operand roles swapped, and the draft logits follow suit.  V = 32768, d = 1024, a launch on 128 x 128 / 256 x 256 tiles: 132 rows
  // (128 of the larger tiles) 25.6 / 32.3 us, 352 (256) 44.8 / 34.7 (d = 512
  // 25.3 / 20.9), 704 (384) 68.6 / 52.8.
  const int MT256 = (M + 255) / 256, NT256 = (V + 255) / 256;
  // ... or where those of 128 x 128, two to a CU, are one round and some of a second, up to three quarters of it.  Whole verify passes on 128 x 128 / 256 x 256,
  // us, tiles of 128 x 128: 506 rows, d = 512, 440 of them 207.8 / 209.2, 532 219.3 / 210.2, 752 222.6 / 215.5, 1004 226.3 / 225.4; d = 1024 438.4 / 438.7,
  // 455.9 / 439.1, 461.2 / 445.1, 465.6 / 468.4; 704 rows, d = 512, 474 236.3 / 233.3, 660 247.5 / 234.6, 942 249.8 / 246.8; d = 1024 485.5 / 487.4,
  // 506.5 / 488.2, 508.4 / 509.7.
  const long tiles = (long)MT * NT;
  const bool big = force_wide || (long)MT256 * NT256 >= 256 || (M > 256 && tiles > 512 && tiles <= 896);
  // 129 - 256 rows of a short K, one round of 256 x 128: a launch on 128 x 128 tiles (two to a CU) / so, K = 512: 143 rows 15.7 / 12.4 us, 240 of
  // a drafter 15.0 / 12.0, 253 16.0 / 13.2.  At K = 1024 a launch by itself is faster, too (209 rows 28.5 / 23.4), but whole passes are not
  // (209 rows 353.8 / 355.4, 253 356.5 / 360): in those E comes from memory, 16 stages of it one behind the other.
  const bool tall = !big && MT == 2 && NT <= 256 && K <= 512;
  // 257 - 384 rows, one round of 192 x 256: two row tiles of 256 would be a third empty.  Whole verify passes of 352 rows on 128 x 128 tiles / so, us, by
  // vocabulary: d = 512, 14000 166.0 / 167.3, 17000 168.0 / 169.0, 20000 168.5 / 170.1, 22000 176.1 / 168.0, 28000 182.2 / 172.8, 32003 182.8 / 177.2; d = 1024
  // 349.6 / 352.5, 352.0 / 354.5, 357.9 / 354.6, 366.3 / 354.5, 372.3 / 358.5, 373.6 / 364.3; of 32768, on 256 x 256 tiles before, d = 512 185.0 / 183.2.
  // 513 - 640 rows, one round of these behind one of 256 x 128, where 256 x 256 would be one and a half: a drafter's 640 with the pass around them 127.5 / 123.4;
  // whole verify passes, d = 512, 528 rows 225.2 / 221.4, 638 244.5 / 240.8; d = 1024 459.6 / 456.3, 501.0 / 497.0.  (770 rows as two rounds of 192 x 256, and the last
  // 384 rows of 825, 1056 and 1408 as one: level or up to 3 % slower.)
  const bool mid = 2 * NT256 <= 256 && ((MT == 3 && (force_wide || tiles > 512)) || (MT == 5 && 3 * NT256 > 256));
  const hipError_t e = big || tall || mid ? launch_draft_logits<true>(st, A, E, M, V, K, row_draft, zd_row, ln)
                                   : launch_draft_logits<false>(st, A, E, M, V, K, row_draft, zd_row, ln);
  if (e != hipSuccess) return e;
  const float* zd = row_draft ? zd_row : nullptr;
  if (tall) return stats ? launch_vocab_tall<false>(st, A, E, M, V, K, zd, part, logits) : launch_vocab_tall<true>(st, A, E, M, V, K, nullptr, part, logits);
  if (mid) return vocab_mid(st, A, E, M, V, K, stats, zd, part, logits);
  if (big) {
    const bool stream = K % 128 == 0 && K >= 256 && (long)MT256 * NT256 > 256;
    if (stats) return stream ? launch_vocab256<false, true>(st, A, E, M, V, K, zd, part, logits) : launch_vocab256<false, false>(st, A, E, M, V, K, zd, part, logits);
    return stream ? launch_vocab256<true, true>(st, A, E, M, V, K, nullptr, part, logits) : launch_vocab256<true, false>(st, A, E, M, V, K, nullptr, part, logits);
  }
  const bool deep = tiles <= 256;   // V = 32768, d = 1024, 128 rows (256 blocks): short ring 24.2 us, deep 21.1; more blocks share CUs
  if (stats) return deep ? launch_vocab<false, CfgVocabDeep>(st, A, E, M, V, K, MT, NT, zd, part, logits) : launch_vocab<false, CfgVocab>(st, A, E, M, V, K, MT, NT, zd, part, logits);
  return deep ? launch_vocab<true, CfgVocabDeep>(st, A, E, M, V, K, MT, NT, nullptr, part, logits) : launch_vocab<true, CfgVocab>(st, A, E, M, V, K, MT, NT, nullptr, part, logits);
}

}  // namespace sd
