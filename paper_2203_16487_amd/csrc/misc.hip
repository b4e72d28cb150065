// Small kernels around the GEMMs: embedding, LayerNorm, row assembly, the acceptance test
// (paper Sec. 3.2, Eq. 8-10), commit (Sec. 2, Eq. 3) and state / cache marshalling.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sd {

static inline dim3 blocks_for(long n, int t) { return dim3((unsigned)((n + t - 1) / t)); }

// ----------------------------------------------------------------------------- positions
// PE(p, 2i) = sin(p / 10000^(2i/d)), PE(p, 2i+1) = cos(same), evaluated in fp64.
__global__ void pos_table_kernel(float* pe, int n_pos, int d) {
  long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)n_pos * d) return;
  int p = (int)(idx / d), c = (int)(idx % d);
  int i = c >> 1;
  double ang = (double)p / pow(10000.0, 2.0 * (double)i / (double)d);
  pe[idx] = (float)((c & 1) ? cos(ang) : sin(ang));
}
hipError_t build_pos_table(hipStream_t st, float* pe, int n_pos, int d) {
  long n = (long)n_pos * d;
  hipLaunchKernelGGL(pos_table_kernel, blocks_for(n, 256), dim3(256), 0, st, pe, n_pos, d);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- embedding
// xb[r] = E[tok[r]] * sqrt(d) + PE[pos[r]] in bf16, and x[r] the same in fp32 less the row's mean: x only ever enters residual
// sums that a LayerNorm follows, and sums that lie about zero lose nothing when they are rounded before it (LnFold, gemm.hip).
// (The positions alone would put a row off by half its standard deviation.)
// 128 threads per row (this one is number t), 8 columns per thread and step (d % 64 == 0, d <= 2048); red: two floats of LDS.
// Meets a barrier: every thread of the block calls it, `live` or not.
__device__ __forceinline__ void embed_row(const bf16* __restrict__ e, const float* __restrict__ p,
                                          float* __restrict__ xr, bf16* __restrict__ xbr, int d, float scale,
                                          int t, float* red, bool live = true) {
  f32x4 v[2][2];
  float s = 0.f;
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const int c = t * 8 + st * 1024;
    if (!live || c >= d) continue;
    const bf16x8 ev = *reinterpret_cast<const bf16x8*>(e + c);
    const f32x4 p0 = *reinterpret_cast<const f32x4*>(p + c), p1 = *reinterpret_cast<const f32x4*>(p + c + 4);
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[st][0][i] = (float)ev[i] * scale + p0[i];
      v[st][1][i] = (float)ev[4 + i] * scale + p1[i];
      o[i] = (bf16)v[st][0][i];
      o[4 + i] = (bf16)v[st][1][i];
      s += v[st][0][i] + v[st][1][i];
    }
    *reinterpret_cast<bf16x8*>(xbr + c) = o;
  }
  s = wave_sum(s);
  if ((t & 63) == 0) red[t >> 6] = s;
  __syncthreads();
  const float mean = (red[0] + red[1]) / (float)d;
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const int c = t * 8 + st * 1024;
    if (!live || c >= d) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[st][h][i] -= mean;
      *reinterpret_cast<f32x4*>(xr + c + 4 * h) = v[st][h];
    }
  }
}
__global__ __launch_bounds__(128) void embed_kernel(const int* __restrict__ tok, const int* __restrict__ pos,
                                                    const bf16* __restrict__ E, const float* __restrict__ pe,
                                                    float* __restrict__ x, bf16* __restrict__ xb, int R, int d,
                                                    float scale) {
  __shared__ float red[2];
  const int r = blockIdx.x;
  if (r >= R) return;
  embed_row(E + (size_t)tok[r] * d, pe + (size_t)pos[r] * d, x + (size_t)r * d, xb + (size_t)r * d, d, scale, threadIdx.x, red);
}
hipError_t embed_rows(hipStream_t st, const int* tok, const int* pos, const bf16* E,
                      const float* pe, float* x, bf16* xb, int R, int d) {
  if (R <= 0) return hipSuccess;
  hipLaunchKernelGGL(embed_kernel, dim3(R), dim3(128), 0, st, tok, pos, E, pe, x, xb, R, d,
                     sqrtf((float)d));
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- LayerNorm
// One wave per row; mean and biased variance as two reductions over registers; eps 1e-5.
template <int PER>   // d = 64 * PER
__global__ __launch_bounds__(256) void ln_kernel(float* __restrict__ x, const bf16* __restrict__ g,
                                                 const bf16* __restrict__ bta, bf16* __restrict__ xb,
                                                 int R, const int* __restrict__ m_real, int keep_x) {
  constexpr int d = 64 * PER;
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= R || (m_real && r >= *m_real)) return;
  float* xr = x + (size_t)r * d;
  float y[PER];
  ln_row<PER>(xr, g, bta, lane, y);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (keep_x) xr[i * 64 + lane] = y[i];
    xb[(size_t)r * d + i * 64 + lane] = (bf16)y[i];
  }
}
// The same on the drafter's mask-slot rows only: output row o = b*k + s is the LayerNorm of row
// b*T + new_rows[b] + s of x, written (bf16 only) to the dense [B*k][d] operand of the
// vocabulary kernel.
template <int PER>
__global__ __launch_bounds__(256) void ln_slots_kernel(const float* __restrict__ x, const bf16* __restrict__ g,
                                                       const bf16* __restrict__ bta, bf16* __restrict__ dst,
                                                       const int* __restrict__ new_rows,
                                                       const int* __restrict__ row_start, int B, int T, int k) {
  constexpr int d = 64 * PER;
  const int lane = threadIdx.x & 63;
  const int o = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (o >= B * k) return;
  const int b = o / k, sl = o - b * k;
  const float* xr = x + (size_t)((row_start ? row_start[b] : b * T) + new_rows[b] + sl) * d;
  float v[PER], gg[PER], bb[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = xr[i * 64 + lane];
#pragma unroll
  for (int i = 0; i < PER; ++i) { gg[i] = (float)g[i * 64 + lane]; bb[i] = (float)bta[i * 64 + lane]; }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) s += v[i];
  const float mean = wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) { float t = v[i] - mean; q += t * t; }
  const float rstd = fast_rsqrt(wave_sum(q) / (float)d + 1e-5f);
#pragma unroll
  for (int i = 0; i < PER; ++i)
    dst[(size_t)o * d + i * 64 + lane] = (bf16)((v[i] - mean) * rstd * gg[i] + bb[i]);
}
template <int PER>
static hipError_t ln_slots_launch(hipStream_t st, const float* x, const bf16* g, const bf16* b, bf16* dst,
                                  const int* new_rows, const int* row_start, int B, int T, int k) {
  hipLaunchKernelGGL(ln_slots_kernel<PER>, dim3((B * k + 3) / 4), dim3(256), 0, st, x, g, b, dst, new_rows, row_start,
                     B, T, k);
  return hipGetLastError();
}
hipError_t layer_norm_slots(hipStream_t st, const float* x, const bf16* g, const bf16* b, bf16* dst,
                            const int* new_rows, const int* row_start, int B, int T, int k, int d) {
  if (B <= 0 || k <= 0) return hipSuccess;
  switch (d / 64) {
#define SD_LN_CASE(P) case P: return ln_slots_launch<P>(st, x, g, b, dst, new_rows, row_start, B, T, k);
    SD_LN_CASE(1) SD_LN_CASE(2) SD_LN_CASE(3) SD_LN_CASE(4) SD_LN_CASE(5) SD_LN_CASE(6) SD_LN_CASE(7) SD_LN_CASE(8)
    SD_LN_CASE(9) SD_LN_CASE(10) SD_LN_CASE(11) SD_LN_CASE(12) SD_LN_CASE(13) SD_LN_CASE(14) SD_LN_CASE(15)
    SD_LN_CASE(16) SD_LN_CASE(17) SD_LN_CASE(18) SD_LN_CASE(19) SD_LN_CASE(20) SD_LN_CASE(21) SD_LN_CASE(22)
    SD_LN_CASE(23) SD_LN_CASE(24) SD_LN_CASE(25) SD_LN_CASE(26) SD_LN_CASE(27) SD_LN_CASE(28) SD_LN_CASE(29)
    SD_LN_CASE(30) SD_LN_CASE(31) SD_LN_CASE(32)
#undef SD_LN_CASE
    default: return hipErrorInvalidValue;
  }
}

template <int PER>
static hipError_t ln_launch(hipStream_t st, float* x, const bf16* g, const bf16* b, bf16* xb, int R, const int* m_real,
                            bool keep_x) {
  hipLaunchKernelGGL(ln_kernel<PER>, dim3((R + 3) / 4), dim3(256), 0, st, x, g, b, xb, R, m_real, keep_x ? 1 : 0);
  return hipGetLastError();
}
hipError_t layer_norm(hipStream_t st, float* x, const bf16* g, const bf16* b, bf16* xb, int R, int d, const int* m_real,
                      bool keep_x) {
  if (R <= 0) return hipSuccess;
  switch (d / 64) {   // d = 64 * heads, heads <= 32
#define SD_LN_CASE(P) case P: return ln_launch<P>(st, x, g, b, xb, R, m_real, keep_x);
    SD_LN_CASE(1) SD_LN_CASE(2) SD_LN_CASE(3) SD_LN_CASE(4) SD_LN_CASE(5) SD_LN_CASE(6) SD_LN_CASE(7) SD_LN_CASE(8)
    SD_LN_CASE(9) SD_LN_CASE(10) SD_LN_CASE(11) SD_LN_CASE(12) SD_LN_CASE(13) SD_LN_CASE(14) SD_LN_CASE(15)
    SD_LN_CASE(16) SD_LN_CASE(17) SD_LN_CASE(18) SD_LN_CASE(19) SD_LN_CASE(20) SD_LN_CASE(21) SD_LN_CASE(22)
    SD_LN_CASE(23) SD_LN_CASE(24) SD_LN_CASE(25) SD_LN_CASE(26) SD_LN_CASE(27) SD_LN_CASE(28) SD_LN_CASE(29)
    SD_LN_CASE(30) SD_LN_CASE(31) SD_LN_CASE(32)
#undef SD_LN_CASE
    default: return hipErrorInvalidValue;
  }
}

__global__ void fill_i32_kernel(int* p, int v, long n) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
hipError_t fill_i32(hipStream_t st, int* p, int v, long n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_i32_kernel, blocks_for(n, 256), dim3(256), 0, st, p, v, n);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- verify rows
// Row i of sequence b: token u_j (i = 0) or draft i (i >= 1) at position j + i; it may look
// at keys [0, j + i + 1) and it scores draft i + 1 (none on the last row).
__global__ void assemble_verify_kernel(SeqState s, RowMap rm, const int* __restrict__ draft, int B, int k, int V) {
  int idx = blockIdx.x * blockDim.x + threadIdx.x;
  int T = k + 1;
  if (idx >= B * T) return;
  int b = idx / T, i = idx - b * T;
  int j = s.len[b];
  int tok = (i == 0) ? s.tokens[(size_t)b * s.tok_pitch + j] : draft[b * k + i - 1];
  rm.row_b[idx] = b;
  rm.row_pos[idx] = j + i;
  rm.row_tok[idx] = min(max(tok, 0), V - 1);   // ids index the embedding table
  rm.row_lim[idx] = j + i + 1;
  rm.row_draft[idx] = (i < k) ? draft[b * k + i] : -1;
  if (i < k) s.last_draft[b * s.k_max + i] = draft[b * k + i];
  if (i == 0) rm.seq_rows[b] = T;
}
hipError_t assemble_verify(hipStream_t st, const SeqState& s, const RowMap& rm, const int* draft, int B, int k, int V) {
  hipLaunchKernelGGL(assemble_verify_kernel, blocks_for((long)B * (k + 1), 128), dim3(128), 0, st, s, rm, draft, B, k, V);
  return hipGetLastError();
}
// The same, one block per row, followed by the row's embedding (embed_rows).
__global__ __launch_bounds__(128) void assemble_embed_verify_kernel(SeqState s, RowMap rm,
                                                                    const int* __restrict__ draft, int B, int k, int V,
                                                                    const bf16* __restrict__ E,
                                                                    const float* __restrict__ pe,
                                                                    float* __restrict__ x, bf16* __restrict__ xb, int d,
                                                                    float scale, uint4* __restrict__ clear, long n16) {
  __shared__ float red[2];
  const int idx = blockIdx.x, T = k + 1;
  if (idx >= B * T) {   // the blocks beyond the rows clear
    for (long i = (long)(idx - B * T) * 128 + threadIdx.x; i < n16; i += (long)(gridDim.x - B * T) * 128)
      clear[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    return;
  }
  const int b = idx / T, i = idx - b * T;
  const int j = s.len[b];
  int tok = (i == 0) ? s.tokens[(size_t)b * s.tok_pitch + j] : draft[b * k + i - 1];
  tok = min(max(tok, 0), V - 1);
  if (threadIdx.x == 0) {
    rm.row_b[idx] = b;
    rm.row_pos[idx] = j + i;
    rm.row_tok[idx] = tok;
    rm.row_lim[idx] = j + i + 1;
    rm.row_draft[idx] = (i < k) ? draft[b * k + i] : -1;
    if (i < k) s.last_draft[b * s.k_max + i] = draft[b * k + i];
    if (i == 0) rm.seq_rows[b] = T;
  }
  embed_row(E + (size_t)tok * d, pe + (size_t)(j + i) * d, x + (size_t)idx * d, xb + (size_t)idx * d, d, scale, threadIdx.x, red);
}
hipError_t assemble_embed_verify(hipStream_t st, const SeqState& s, const RowMap& rm, const int* draft, int B, int k,
                                 int V, const bf16* E, const float* pe, float* x, bf16* xb, int d, void* clear,
                                 size_t clear_bytes) {
  if (B <= 0) return hipSuccess;
  const long n16 = (long)(clear_bytes / 16), more = (n16 + 511) / 512;   // four pieces per thread
  hipLaunchKernelGGL(assemble_embed_verify_kernel, dim3((unsigned)(B * (k + 1) + (more < 1024 ? more : 1024))), dim3(128), 0, st,
                     s, rm, draft, B, k, V, E, pe, x, xb, d, sqrtf((float)d), static_cast<uint4*>(clear), n16);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- prefill / draft rows
// Each sequence owns up to T row slots of the pass.
// Prefill (n_mask = 0): the next up to T uncached stream tokens, causal.
// Draft (Sec. 3.1.3, Eq. 7): the uncached stream tokens (causal) followed by n_mask [MASK]
// slots; slot s sits at the position of the token it predicts and attends to the whole stream
// and to all slots.  The slots' keys/values land beyond the valid cache length and are dead
// after the pass.  new_rows[b] = stream rows of this pass (the amount `cached` advances by).
// One block per row: the row's bookkeeping, then its embedding (embed_rows).  PACKED: the rows
// of the sequences follow each other without padding; a block finds its sequence's first row as
// the sum of the row counts of the sequences before it (each thread derives some of them from the
// state, as the block does for its own), and blocks beyond their sequence's rows do nothing.
struct StreamRows {
  int c0, n, rows;
  bool masks;
};
__device__ __forceinline__ StreamRows stream_rows(const SeqState& s, int role, int b, int T, int n_mask) {
  StreamRows r;
  r.c0 = s.cached[role][b];
  const int target = s.len[b] + (role == 1 ? 1 : 0);       // drafter also ingests the pending token
  r.n = max(0, min(target - r.c0, T - n_mask));
  r.masks = n_mask > 0 && r.c0 + r.n == target;             // slots only once the stream is ingested
  r.rows = r.n + (r.masks ? n_mask : 0);
  return r;
}
template <bool PACKED>
__global__ __launch_bounds__(128) void assemble_embed_stream_kernel(SeqState s, RowMap rm, int role, int B, int T,
                                                                    int n_mask, int mask_id, int pad_id, int V,
                                                                    int* __restrict__ new_rows,
                                                                    const bf16* __restrict__ E,
                                                                    const float* __restrict__ pe,
                                                                    float* __restrict__ x, bf16* __restrict__ xb, int d,
                                                                    float scale, uint4* __restrict__ clear, long n16) {
  __shared__ int wsum[2];
  __shared__ float red[2];
  if ((int)blockIdx.x >= B * T) {   // the blocks beyond the rows clear
    for (long i = (long)((int)blockIdx.x - B * T) * 128 + threadIdx.x; i < n16; i += (long)((int)gridDim.x - B * T) * 128)
      clear[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    return;
  }
  const int b = blockIdx.x / T, i = blockIdx.x - b * T;
  const StreamRows me = stream_rows(s, role, b, T, n_mask);
  int first = b * T;
  if (PACKED) {
    int part = 0;
    for (int o = threadIdx.x; o < b; o += 128) part += stream_rows(s, role, o, T, n_mask).rows;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = part;
    __syncthreads();
    first = wsum[0] + wsum[1];
  }
  if (threadIdx.x == 0 && i == 0) {
    rm.seq_rows[b] = me.rows;
    new_rows[b] = me.n;
    if (PACKED) {
      rm.row_start[b] = first;
      if (b == B - 1) rm.row_start[B] = first + me.rows;
    }
  }
  if (PACKED && i >= me.rows) return;
  const int r = first + i;
  int rb = -1, pos = 0, tok = pad_id, lim = 0;
  if (i < me.n) {
    rb = b; pos = me.c0 + i; tok = min(max(s.tokens[(size_t)b * s.tok_pitch + me.c0 + i], 0), V - 1); lim = me.c0 + i + 1;
  } else if (me.masks && i < me.n + n_mask) {
    rb = b; pos = me.c0 + i; tok = mask_id; lim = me.c0 + me.n + n_mask;
  }
  if (threadIdx.x == 0) {
    rm.row_b[r] = rb; rm.row_pos[r] = pos; rm.row_tok[r] = tok; rm.row_lim[r] = lim; rm.row_draft[r] = -1;
  }
  embed_row(E + (size_t)tok * d, pe + (size_t)pos * d, x + (size_t)r * d, xb + (size_t)r * d, d, scale, threadIdx.x, red);
}
hipError_t assemble_embed_stream(hipStream_t st, const SeqState& s, const RowMap& rm, int role, int B, int T,
                                 int n_mask, int mask_id, int pad_id, int V, int* new_rows, const bf16* E,
                                 const float* pe, float* x, bf16* xb, int d, bool packed, void* clear, size_t clear_bytes) {
  if (B <= 0 || T <= 0) return hipSuccess;
  const long n16 = (long)(clear_bytes / 16), more = (n16 + 511) / 512;   // four pieces per thread
  const dim3 grid((unsigned)(B * T + (more < 1024 ? more : 1024)));
  if (packed)
    hipLaunchKernelGGL(assemble_embed_stream_kernel<true>, grid, dim3(128), 0, st, s, rm, role, B, T, n_mask,
                       mask_id, pad_id, V, new_rows, E, pe, x, xb, d, sqrtf((float)d), static_cast<uint4*>(clear), n16);
  else
    hipLaunchKernelGGL(assemble_embed_stream_kernel<false>, grid, dim3(128), 0, st, s, rm, role, B, T, n_mask,
                       mask_id, pad_id, V, new_rows, E, pe, x, xb, d, sqrtf((float)d), static_cast<uint4*>(clear), n16);
  return hipGetLastError();
}

__global__ void advance_cached_kernel(SeqState s, int role, const int* __restrict__ new_rows, int B, const unsigned* __restrict__ fail) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B && !(fail && *fail != 0u)) s.cached[role][b] += new_rows[b];
}
hipError_t advance_cached(hipStream_t st, const SeqState& s, int role, const int* new_rows, int B, const unsigned* fail) {
  hipLaunchKernelGGL(advance_cached_kernel, blocks_for(B, 64), dim3(64), 0, st, s, role, new_rows, B, fail);
  return hipGetLastError();
}

// dense [B*k][d] copy of the mask-slot rows (row b*T + new_rows[b] + s) for the vocabulary kernel
__global__ void gather_slots_kernel(const bf16* __restrict__ xb, bf16* __restrict__ dst,
                                    const int* __restrict__ new_rows, const int* __restrict__ row_start, int B, int T,
                                    int k, int d) {
  const int o = blockIdx.x;              // b*k + s
  const int b = o / k, sl = o - b * k;
  const int first = row_start ? row_start[b] : b * T;
  const uint4* src = reinterpret_cast<const uint4*>(xb + (size_t)(first + new_rows[b] + sl) * d);
  uint4* out = reinterpret_cast<uint4*>(dst + (size_t)o * d);
  for (int c = threadIdx.x; c < d / 8; c += blockDim.x) out[c] = src[c];
}
hipError_t gather_slots(hipStream_t st, const bf16* xb, bf16* dst, const int* new_rows, const int* row_start, int B,
                        int T, int k, int d) {
  hipLaunchKernelGGL(gather_slots_kernel, dim3(B * k), dim3(64), 0, st, xb, dst, new_rows, row_start, B, T, k, d);
  return hipGetLastError();
}

// Encoder rows without padding: sequence b owns rows row_start[b] .. row_start[b] + src_len[b] - 1 (a running sum, sources
// in batch order), n_rows[0] = their number.  A block embeds kEncRows rows of one sequence; it finds the sequence's first
// row as the sum of the lengths before it (B loads spread over its threads).
constexpr int kEncRows = 8;
__global__ __launch_bounds__(256) void encoder_rows_embed_kernel(const int* __restrict__ src, const int* __restrict__ src_len,
                                                                 int* __restrict__ pos, int* __restrict__ row_b,
                                                                 int* __restrict__ row_start, int* __restrict__ n_rows, int B,
                                                                 int S, int V, const bf16* __restrict__ E,
                                                                 const float* __restrict__ pe, float* __restrict__ x,
                                                                 bf16* __restrict__ xb, int d, float scale) {
  __shared__ int wsum[4];
  __shared__ float red[2][4];   // (rows take turns)
  const int per = (S + kEncRows - 1) / kEncRows, b = blockIdx.x / per, s0 = (blockIdx.x - b * per) * kEncRows;
  const int len = min(max(src_len[b], 0), S);
  if (s0 >= len && s0 > 0) return;
  int part = 0;
  for (int o = threadIdx.x; o < b; o += 256) part += min(max(src_len[o], 0), S);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = part;
  __syncthreads();
  const int first = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  if (s0 == 0 && threadIdx.x == 0) {
    row_start[b] = first;
    if (b == B - 1) { row_start[B] = first + len; n_rows[0] = first + len; }
  }
  // half a wave-quad per row: two rows at a time
  const int lo = threadIdx.x >> 7, t = threadIdx.x & 127;
  for (int i = 0; i < kEncRows && s0 + i < len; i += 2) {
    const bool live = s0 + i + lo < len;
    const int s = min(s0 + i + lo, len - 1), r = first + s, tok = min(max(src[(size_t)b * S + s], 0), V - 1);
    if (t == 0 && live) { pos[r] = s; row_b[r] = b; }
    embed_row(E + (size_t)tok * d, pe + (size_t)s * d, x + (size_t)r * d, xb + (size_t)r * d, d, scale, t, red[(i >> 1) & 1] + 2 * lo, live);
  }
}
hipError_t encoder_rows_embed(hipStream_t st, const int* src, const int* src_len, int* pos, int* row_b, int* row_start,
                              int* n_rows, int B, int S, int V, const bf16* E, const float* pe, float* x, bf16* xb, int d) {
  if (B <= 0 || S <= 0) return hipSuccess;
  hipLaunchKernelGGL(encoder_rows_embed_kernel, dim3(B * ((S + kEncRows - 1) / kEncRows)), dim3(256), 0, st, src, src_len, pos,
                     row_b, row_start, n_rows, B, S, V, E, pe, x, xb, d, sqrtf((float)d));
  return hipGetLastError();
}

// dst [B][S][d] <- the packed rows of every sequence, zeros beyond its length
__global__ void unpack_rows_kernel(const bf16* __restrict__ src, const int* __restrict__ row_start,
                                   const int* __restrict__ src_len, bf16* __restrict__ dst, long n8, int S, int d) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte piece
  if (i >= n8) return;
  const int per = d / 8;
  const long row = i / per;
  const int c = (int)(i - row * per) * 8;
  const int b = (int)(row / S), s = (int)(row - (long)b * S);
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (bf16)0.f;
  if (s < min(max(src_len[b], 0), S)) v = *reinterpret_cast<const bf16x8*>(src + (size_t)(row_start[b] + s) * d + c);
  *reinterpret_cast<bf16x8*>(dst + (size_t)row * d + c) = v;
}
hipError_t unpack_rows(hipStream_t st, const bf16* src, const int* row_start, const int* src_len, bf16* dst, int B,
                       int S, int d) {
  const long n8 = (long)B * S * (d / 8);
  if (n8 <= 0) return hipSuccess;
  hipLaunchKernelGGL(unpack_rows_kernel, blocks_for(n8, 256), dim3(256), 0, st, src, row_start, src_len, dst, n8, S, d);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- acceptance
// Stage 1, one wave per row: merge the per-tile partials of the vocabulary kernel into
//   m = max logit, arg-max = lowest column among maxima, LSE, and the number of logits that
//   are strictly larger than the logit z_d of the draft this row scores.
struct RowMerge {
  float m, lse;
  int arg, cnt;
};
constexpr int kHeldRecords = 8;   // per lane, in registers: one pass over memory up to 512 tiles
struct RowRecords {
  f32x4 rec[kHeldRecords];
  __device__ __forceinline__ void request(const float* __restrict__ pr, int n_tiles, int lane) {
    if (n_tiles > 64 * kHeldRecords) return;
#pragma unroll
    for (int i = 0; i < kHeldRecords; ++i)   // (clamped, so that no load sits behind a lane's own branch)
      rec[i] = *reinterpret_cast<const f32x4*>(pr + (size_t)min(lane + 64 * i, n_tiles - 1) * kPartF);
  }
};
// (held: what was requested of the row)
__device__ __forceinline__ RowMerge merge_row(const RowRecords& held, const float* __restrict__ pr, int n_tiles, int lane) {
  const bool all = n_tiles <= 64 * kHeldRecords;
  float m = kNegInf;
  int am = 0x7fffffff, cnt = 0;
  if (all) {
#pragma unroll
    for (int i = 0; i < kHeldRecords; ++i) {
      if (lane + 64 * i < n_tiles) {
        const float tm = held.rec[i][0];
        const int ti = __float_as_int(held.rec[i][1]);
        if (tm > m || (tm == m && ti < am)) { m = tm; am = ti; }
        cnt += __float_as_int(held.rec[i][3]);
      }
    }
  } else {
    for (int t = lane; t < n_tiles; t += 64) {
      const f32x4 p = *reinterpret_cast<const f32x4*>(pr + (size_t)t * kPartF);
      const float tm = p[0];
      const int ti = __float_as_int(p[1]);
      if (tm > m || (tm == m && ti < am)) { m = tm; am = ti; }
      cnt += __float_as_int(p[3]);
    }
  }
  const float gm = wave_max(m);
  int cand = (m == gm) ? am : 0x7fffffff;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    cand = min(cand, __shfl_xor(cand, o, 64));
    cnt += __shfl_xor(cnt, o, 64);
  }
  float se = 0.f;
  if (all) {
#pragma unroll
    for (int i = 0; i < kHeldRecords; ++i)
      if (lane + 64 * i < n_tiles) se += held.rec[i][2] * __expf(held.rec[i][0] - gm);
  } else {
    for (int t = lane; t < n_tiles; t += 64) {
      const f32x4 p = *reinterpret_cast<const f32x4*>(pr + (size_t)t * kPartF);
      se += p[2] * __expf(p[0] - gm);
    }
  }
  se = wave_sum(se);
  return RowMerge{gm, gm + __logf(se), cand, cnt};
}
__device__ __forceinline__ void store_row_stats(float* rs, const RowMerge& r, float zd) {
  *reinterpret_cast<f32x4*>(rs) = f32x4{r.m, (float)r.arg, r.lse, zd};
  *reinterpret_cast<f32x4*>(rs + 4) = f32x4{(float)r.cnt, 0.f, 0.f, 0.f};
}

// Stage 2, per sequence (paper Sec. 3.2).  With z_d the draft's logit on its row:
// Eq. 8:  log P(draft) >= log P(beta-th ranked)   <=>  #{v : z_v > z_d} < beta
// Eq. 9:  log P(top-1) - log P(draft) <= tau      <=>  m - z_d <= tau
// (log-softmax subtracts the same LSE from every logit of the row; a draft tied with the
// beta-th score passes, as ">=" says).  a = number of leading rows that pass; next = arg-max
// of row a.
//
// Both stages in one launch: a block per sequence, its 16 waves merge the k + 1 <= 32 rows (two a
// wave at most), then lane i of the first one takes row i.  All that comes from memory is requested
// at once, and the block has no wave without a row: bound by round trips (one behind the other and scanned by one thread:
// whole verify passes of 6 rows of d = 512 112.6 us, now 111.6; of 352 182.9 / 181.6; of 352 of d = 1024 517.5 / 514.6).
constexpr int kMergeWaves = 16;
__global__ __launch_bounds__(64 * kMergeWaves) void merge_accept_kernel(const float* __restrict__ part,
                                                           const float* __restrict__ zd_row, int n_tiles,
                                                           float* __restrict__ row_stats, SeqState s, int k,
                                                           int beta, float tau, int pad_id,
                                                           int* __restrict__ accept_len,
                                                           int* __restrict__ next_token,
                                                           const unsigned* __restrict__ fail) {
  __shared__ float sm[32], szd[32];
  __shared__ int sarg[32], scnt[32];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int T = k + 1, rows = (T - wave + kMergeWaves - 1) / kMergeWaves;   // of this wave: wave, wave + 16
  const unsigned failed = fail ? *fail : 0u;
  const int cached = s.cached[0][b], len = s.len[b], finished = s.finished[b];
  RowRecords held[2];
  float zd[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (i < rows) {
      const int r = b * T + wave + i * kMergeWaves;
      held[i].request(part + (size_t)r * n_tiles * kPartF, n_tiles, lane);
      zd[i] = zd_row[r];
    }
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (i < rows) {
      const int t = wave + i * kMergeWaves, r = b * T + t;
      const RowMerge res = merge_row(held[i], part + (size_t)r * n_tiles * kPartF, n_tiles, lane);
      if (lane == 0) {
        store_row_stats(row_stats + (size_t)r * kRowStats, res, zd[i]);
        sm[t] = res.m; szd[t] = zd[i]; sarg[t] = res.arg; scnt[t] = res.cnt;
      }
    }
  lds_barrier();
  if (wave != 0) return;
  // keys/values of u_0..u_{j-1} must be cached: a cache loaded short of the stream (and not
  // completed by a prefill) would have let this pass attend to rows that were never written
  if (failed || (cached < len && !finished)) {
    if (lane == 0) { accept_len[b] = -1; next_token[b] = pad_id; }
    return;
  }
  const int i = min(lane, T - 1);
  const float gap = sm[i] - szd[i];
  const unsigned long long misses = __builtin_amdgcn_ballot_w64(lane >= k || !(scnt[i] < beta && gap <= tau));   // (k <= 31)
  const int a = __builtin_ctzll(misses);
  // rows whose tau test was decided by a margin of at most 1e-2 (up to the bifurcation row)
  const int near = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane <= a && lane < k && fabsf(tau - gap) <= 1e-2f));
  if (lane != 0) return;
  accept_len[b] = finished ? 0 : a;
  next_token[b] = finished ? pad_id : sarg[a];
  if (!finished && near) atomicAdd(&s.scratch[3], near);
}
hipError_t merge_accept(hipStream_t st, const float* part, const float* zd_row, int n_tiles, float* row_stats,
                        const SeqState& s, int B, int k, int beta, float tau, int pad_id, int* accept_len,
                        int* next_token, const unsigned* fail) {
  if (B <= 0) return hipSuccess;
  if (k + 1 > 32) return hipErrorInvalidValue;
  hipLaunchKernelGGL(merge_accept_kernel, dim3(B), dim3(64 * std::min(k + 1, kMergeWaves)), 0, st, part, zd_row, n_tiles, row_stats, s, k, beta,
                     tau, pad_id, accept_len, next_token, fail);
  return hipGetLastError();
}

// Drafter: merge the slot rows, draft[b][s] = arg-max of slot row b*k + s (pad for finished
// sequences); the first B blocks also advance the drafter's cached length by the stream rows
// this pass ingested.
__global__ __launch_bounds__(64) void merge_drafts_kernel(const float* __restrict__ part, int n_tiles,
                                                          float* __restrict__ row_stats, SeqState s, int B, int k,
                                                          int pad_id, const int* __restrict__ new_rows,
                                                          const int* __restrict__ seq_rows,
                                                          int* __restrict__ draft, const unsigned* __restrict__ fail) {
  const int o = blockIdx.x, lane = threadIdx.x;
  // a sequence whose uncached stream did not fit into this pass got no mask slots (its rows of
  // the pass were all stream rows): what sits at its slot rows belongs to another sequence
  const int b = o / k, slots = seq_rows[b] - new_rows[b], finished = s.finished[b], cached = o < B ? s.cached[1][o] + new_rows[o] : 0;
  const bool failed = fail && *fail != 0u;
  RowRecords held;   // (all requests of memory at once, as above)
  held.request(part + (size_t)o * n_tiles * kPartF, n_tiles, lane);
  const RowMerge res = merge_row(held, part + (size_t)o * n_tiles * kPartF, n_tiles, lane);
  if (lane != 0) return;
  store_row_stats(row_stats + (size_t)o * kRowStats, res, kNegInf);
  draft[o] = finished || slots != k || failed ? pad_id : res.arg;
  if (o < B && !failed) s.cached[1][o] = cached;
}
hipError_t merge_drafts(hipStream_t st, const float* part, int n_tiles, float* row_stats, const SeqState& s, int B,
                        int k, int pad_id, const int* new_rows, const int* seq_rows, int* draft, const unsigned* fail) {
  if (B <= 0 || k <= 0) return hipSuccess;
  hipLaunchKernelGGL(merge_drafts_kernel, dim3(B * k), dim3(64), 0, st, part, n_tiles, row_stats, s, B, k, pad_id,
                     new_rows, seq_rows, draft, fail);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- head-based drafting
// Input rows of the drafting heads (Sec. 2 "Draft": FFN heads on the target model's last hidden
// state): for sequence b the verifier's final hidden state at the bifurcation row a_b of the
// latest pass (the row whose arg-max is next_token).  x holds the pass's rows [B*T][d], already
// normalised (g == null) or as the last residual sum still to be normalised with (g, beta).
// Written as bf16 [B][d] (GEMM operand) and, replicated k times, as fp32 [B*k][d] (the residual
// each head adds to).  One wave per sequence.
template <int PER>
__global__ __launch_bounds__(256) void head_rows_kernel(const float* __restrict__ x, const bf16* __restrict__ g,
                                                        const bf16* __restrict__ beta,
                                                        const int* __restrict__ accept_len, int B, int T, int k,
                                                        bf16* __restrict__ rows, float* __restrict__ rep) {
  constexpr int d = 64 * PER;
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= B) return;
  const int a = min(max(accept_len[b], 0), T - 1);
  const float* xr = x + ((size_t)b * T + a) * d;
  float v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = xr[i * 64 + lane];
  if (g) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) s += v[i];
    const float mean = wave_sum(s) / (float)d;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) { float t = v[i] - mean; q += t * t; }
    const float rstd = fast_rsqrt(wave_sum(q) / (float)d + 1e-5f);
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = (v[i] - mean) * rstd * (float)g[i * 64 + lane] + (float)beta[i * 64 + lane];
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int c = i * 64 + lane;
    rows[(size_t)b * d + c] = (bf16)v[i];
    for (int h = 0; h < k; ++h) rep[((size_t)b * k + h) * d + c] = v[i];
  }
}
template <int PER>
static hipError_t head_rows_launch(hipStream_t st, const float* x, const bf16* g, const bf16* beta, const int* accept_len,
                                   int B, int T, int k, bf16* rows, float* rep) {
  hipLaunchKernelGGL(head_rows_kernel<PER>, dim3((B + 3) / 4), dim3(256), 0, st, x, g, beta, accept_len, B, T, k, rows, rep);
  return hipGetLastError();
}
hipError_t head_rows(hipStream_t st, const float* x, const bf16* g, const bf16* beta, const int* accept_len, int B, int T,
                     int k, int d, bf16* rows, float* rep) {
  if (B <= 0 || k <= 0) return hipSuccess;
  switch (d / 64) {
#define SD_LN_CASE(P) case P: return head_rows_launch<P>(st, x, g, beta, accept_len, B, T, k, rows, rep);
    SD_LN_CASE(1) SD_LN_CASE(2) SD_LN_CASE(3) SD_LN_CASE(4) SD_LN_CASE(5) SD_LN_CASE(6) SD_LN_CASE(7) SD_LN_CASE(8)
    SD_LN_CASE(9) SD_LN_CASE(10) SD_LN_CASE(11) SD_LN_CASE(12) SD_LN_CASE(13) SD_LN_CASE(14) SD_LN_CASE(15)
    SD_LN_CASE(16) SD_LN_CASE(17) SD_LN_CASE(18) SD_LN_CASE(19) SD_LN_CASE(20) SD_LN_CASE(21) SD_LN_CASE(22)
    SD_LN_CASE(23) SD_LN_CASE(24) SD_LN_CASE(25) SD_LN_CASE(26) SD_LN_CASE(27) SD_LN_CASE(28) SD_LN_CASE(29)
    SD_LN_CASE(30) SD_LN_CASE(31) SD_LN_CASE(32)
#undef SD_LN_CASE
    default: return hipErrorInvalidValue;
  }
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ src, bf16* __restrict__ dst, long n) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= n) return;   // n % 4 == 0
  const f32x4 v = *reinterpret_cast<const f32x4*>(src + i);
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
  *reinterpret_cast<bf16x4*>(dst + i) = o;
}
hipError_t f32_to_bf16(hipStream_t st, const float* src, bf16* dst, long n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(f32_to_bf16_kernel, blocks_for(n / 4, 256), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

// draft[b][i] = arg-max of head row b*k + i (pad for finished sequences and for sequences whose
// verification reported a failure)
__global__ __launch_bounds__(64) void merge_head_drafts_kernel(const float* __restrict__ part, int n_tiles,
                                                               float* __restrict__ row_stats, SeqState s,
                                                               const int* __restrict__ accept_len, int k, int pad_id,
                                                               int* __restrict__ draft) {
  const int o = blockIdx.x, lane = threadIdx.x, b = o / k;
  const bool none = s.finished[b] || accept_len[b] < 0;
  RowRecords held;
  held.request(part + (size_t)o * n_tiles * kPartF, n_tiles, lane);
  const RowMerge res = merge_row(held, part + (size_t)o * n_tiles * kPartF, n_tiles, lane);
  if (lane != 0) return;
  store_row_stats(row_stats + (size_t)o * kRowStats, res, kNegInf);
  draft[o] = none ? pad_id : res.arg;
}
hipError_t merge_head_drafts(hipStream_t st, const float* part, int n_tiles, float* row_stats, const SeqState& s,
                             const int* accept_len, int B, int k, int pad_id, int* draft) {
  if (B <= 0 || k <= 0) return hipSuccess;
  hipLaunchKernelGGL(merge_head_drafts_kernel, dim3(B * k), dim3(64), 0, st, part, n_tiles, row_stats, s, accept_len, k,
                     pad_id, draft);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- commit
// Eq. 3: the iteration's output is the accepted drafts followed by the verifier's token; a
// sequence stops after its first EOS or when it reaches its cap.  j advances by the number
// of tokens appended: exactly that many of this pass's cache rows become valid.
// 32 lanes a sequence, lane i for token i: one memory round trip for everything that is read, whatever it turns out to be, and the length by a
// ballot.  (With a thread a sequence, which chose and stored its tokens one by one, 8.7 us for 128 sequences; so 5.7.)  Those 32 lanes cost 35 cycles
// a sequence of one CU's instructions, so a block takes kCommitBatch of them at most, and where there are more the last block to end adds up.
// (All by one block: 1024 / 4096 sequences of one draft 20.9 / 71 us, a thread a sequence 13.7 / 33; so 7.7 / 8.2.)
constexpr int kCommitThreads = 1024, kCommitBatch = 128;
__global__ __launch_bounds__(kCommitThreads) void commit_kernel(SeqState s, const int* __restrict__ accept_len, const int* __restrict__ next_token,
                                                                int B, int k, int eos_id, int* n_active) {
  __shared__ int active, tokens;
  if (threadIdx.x == 0) { active = 0; tokens = 0; }
  __syncthreads();
  // the counters are read now and written at the end: their round trip runs under the sequences'
  int c_commits = 0, c_tokens = 0;
  if (threadIdx.x == 0) { c_commits = s.scratch[0]; c_tokens = s.scratch[1]; }
  const int i = threadIdx.x & 31, shift = threadIdx.x & 32;
  int mine = 0, added = 0;
  const int end = min(((int)blockIdx.x + 1) * kCommitBatch, B);
  for (int b0 = blockIdx.x * kCommitBatch; b0 < end; b0 += (int)blockDim.x >> 5) {
    const int b = min(b0 + (int)(threadIdx.x >> 5), end - 1);   // (halves of a wave beyond the last sequence: that one, nothing stored)
    const bool there = b0 + (int)(threadIdx.x >> 5) < end;
    const int fin0 = s.finished[b], a0 = accept_len[b], j0 = s.len[b], cap = s.cap[b], nt = next_token[b];
    const int t = s.last_draft[b * s.k_max + min(i, s.k_max - 1)];
    const bool live = there && !fin0 && a0 >= 0;   // a0 < 0: verification reported a failure, nothing to commit
    const int a = min(a0, k);   // k of the pass whose drafts are stored: entries beyond it are stale
    const int tok = i < a ? t : nt;
    // after which token it ends: the first EOS, or where the length cap is reached (before the first one, if it has been)
    const unsigned ends = (unsigned)(__builtin_amdgcn_ballot_w64(i <= a && (tok == eos_id || j0 + i + 1 >= cap)) >> shift);
    const int n = j0 >= cap ? 0 : ends ? __builtin_ctz(ends) + 1 : a + 1;
    const bool fin = j0 >= cap || ends != 0;
    if (live && i < n) s.tokens[(size_t)b * s.tok_pitch + j0 + 1 + i] = tok;
    if (i != 0) continue;
    if (live) {
      s.len[b] = j0 + n;
      s.cached[0][b] = j0 + n;   // the verifier's rows of the kept tokens are now valid cache
      s.finished[b] = fin;
      added += n;
    }
    if (there && !fin0 && (a0 < 0 || !fin)) ++mine;
  }
  if (mine) atomicAdd(&active, mine);
  if (added) atomicAdd(&tokens, added);
  __syncthreads();
  if (threadIdx.x == 0) {
    int n = active, m = tokens;
    if (gridDim.x > 1) {   // (the three words are zero between commits: specdec_begin clears them, and the last block does)
      atomicAdd(&s.scratch[4], n);
      atomicAdd(&s.scratch[5], m);
      __threadfence();
      if (atomicAdd(&s.scratch[6], 1) + 1 != (int)gridDim.x) return;
      __threadfence();
      n = atomicExch(&s.scratch[4], 0);
      m = atomicExch(&s.scratch[5], 0);
      s.scratch[6] = 0;
    }
    if (n_active) *n_active = n;
    s.scratch[0] = c_commits + 1;   // commits
    s.scratch[1] = c_tokens + m;    // tokens appended
    s.scratch[2] = B - n;           // finished sequences
  }
}
hipError_t commit_rows(hipStream_t st, const SeqState& s, const int* accept_len, const int* next_token, int B,
                       int k, int eos_id, int* n_active) {
  hipLaunchKernelGGL(commit_kernel, dim3((B + kCommitBatch - 1) / kCommitBatch), dim3(std::min((B + 1) / 2 * 64, kCommitThreads)), 0, st, s, accept_len, next_token, B, min(k, s.k_max), eos_id,
                     n_active);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- state
__global__ void begin_kernel(SeqState s, int B, int max_new, int max_tgt, int bos_id, int* flags0, int* flags1, int n_flags) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < n_flags && flags0) flags0[b] = 0;
  if (b < n_flags && flags1) flags1[b] = 0;
  if (b < 8) s.scratch[b] = 0;   // counters: commits, tokens appended, finished, near-threshold rows
  if (b >= B) return;
  s.tokens[(size_t)b * s.tok_pitch] = bos_id;
  s.len[b] = 0;
  s.start[b] = 0;
  s.cap[b] = min(max_new, max_tgt);
  s.finished[b] = (max_new <= 0);
  s.cached[0][b] = 0;
  s.cached[1][b] = 0;
}
hipError_t begin_state(hipStream_t st, const SeqState& s, int B, int max_new, int max_tgt, int bos_id, int* flags0, int* flags1, int n_flags) {
  if (n_flags > 128) return hipErrorInvalidValue;   // (the first block's threads)
  hipLaunchKernelGGL(begin_kernel, blocks_for(B, 128), dim3(128), 0, st, s, B, max_new, max_tgt, bos_id, flags0, flags1, n_flags);
  return hipGetLastError();
}

// Sequence b's stream from the caller's: threads tid, tid + n, ..
__device__ __forceinline__ void set_stream_row(const SeqState& s, const int* tokens, const int* len, int b, int L_max, int max_new, int max_tgt,
                                               int tid, int n) {
  const int j = min(max(len[b], 0), L_max);
  for (int i = tid; i <= j; i += n) s.tokens[(size_t)b * s.tok_pitch + i] = tokens[(size_t)b * (L_max + 1) + i];
  if (tid == 0) {
    s.len[b] = j;
    s.start[b] = j;
    const int cap = j + min(max_new, max(max_tgt - j, 0));   // (max_new may be huge: no j + max_new)
    s.cap[b] = cap;
    s.finished[b] = (j >= cap);
    s.cached[0][b] = 0;
    s.cached[1][b] = 0;
  }
}
__global__ void set_stream_kernel(SeqState s, const int* __restrict__ tokens, const int* __restrict__ len, int B,
                                  int L_max, int max_new, int max_tgt) {
  set_stream_row(s, tokens, len, blockIdx.x, L_max, max_new, max_tgt, threadIdx.x, blockDim.x);
}
hipError_t set_stream(hipStream_t st, const SeqState& s, const int* tokens, const int* len, int B, int L_max,
                      int max_new, int max_tgt) {
  hipLaunchKernelGGL(set_stream_kernel, dim3(B), dim3(64), 0, st, s, tokens, len, B, L_max, max_new, max_tgt);
  return hipGetLastError();
}

// Rollback to given lengths: nothing moves, rows beyond the new j are dead.
__global__ void rewind_kernel(SeqState s, const int* __restrict__ len, int B) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int j = s.len[b];
  int jn = min(j, max(len[b], 0));
  if (jn < j) {
    s.len[b] = jn;
    s.start[b] = min(s.start[b], jn);
    s.cached[0][b] = min(s.cached[0][b], jn);
    s.cached[1][b] = min(s.cached[1][b], jn + 1);
    s.finished[b] = (jn >= s.cap[b]);
  }
}
hipError_t rewind_state(hipStream_t st, const SeqState& s, const int* len, int B) {
  hipLaunchKernelGGL(rewind_kernel, blocks_for(B, 128), dim3(128), 0, st, s, len, B);
  return hipGetLastError();
}

__global__ void copy_i32_kernel(int* dst, const int* src, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}
__global__ void clamp_copy_i32_kernel(int* dst, const int* src, int n, int lo, int hi) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = min(max(src[i], lo), hi);
}
hipError_t set_src_len(hipStream_t st, const SeqState& s, const int* src_len, int B, int S_max) {
  hipLaunchKernelGGL(clamp_copy_i32_kernel, blocks_for(B, 128), dim3(128), 0, st, s.src_len, src_len, B, 1, S_max);
  return hipGetLastError();
}
__global__ void get_output_kernel(SeqState s, int* __restrict__ tokens, int out_cap, int* __restrict__ out_len,
                                  int* __restrict__ finished, int B, int pad_id) {
  int b = blockIdx.x;
  if (b >= B) return;
  int st0 = s.start[b], n = s.len[b] - st0;
  for (int i = threadIdx.x; i < out_cap; i += blockDim.x)
    tokens[(size_t)b * out_cap + i] = (i < n) ? s.tokens[(size_t)b * s.tok_pitch + st0 + 1 + i] : pad_id;
  if (threadIdx.x == 0) {
    out_len[b] = n;
    if (finished) finished[b] = s.finished[b];
  }
}
hipError_t get_output(hipStream_t st, const SeqState& s, int* tokens, int out_cap, int* out_len, int* finished,
                      int B, int pad_id) {
  hipLaunchKernelGGL(get_output_kernel, dim3(B), dim3(64), 0, st, s, tokens, out_cap, out_len, finished, B, pad_id);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- cache layout
// Keys and values of all layers [layer][B][H][Lcap][64] <-> flat [layer][B][L][d], 16 bytes a thread, in one launch (z < 2 layers: a part of one
// sequence's rows).  LOAD, z = 2 layers: sequence b's number of cached rows, and its stream where there is one.  In launches of their own, 2.9
// us for each layer's keys or values (of 64 sequences, 32 rows of 512) and 3.3 and 1.4 us for streams and lengths, each behind the one before,
// the drafter's pass from a stored prefix took 159.5 us, so 150.1.
template <bool LOAD>
__global__ __launch_bounds__(256) void cache_flat_kernel(SeqState s, CacheFlat a) {
  const int b = blockIdx.y, z = blockIdx.z;
  if (LOAD && z == 2 * a.layers) {
    if (blockIdx.x) return;
    if (a.tokens) set_stream_row(s, a.tokens, a.n, b, a.L, a.max_new, a.max_tgt, threadIdx.x, 256);
    if (threadIdx.x == 0) s.cached[a.role][b] = min(max(a.n[b], 0), a.L);   // (after the stream's, by the same thread)
    return;
  }
  const int at = blockIdx.x * 256 + threadIdx.x, ch = at & 7, l = (at >> 3) / a.H, h = (at >> 3) - l * a.H, layer = z >> 1;
  if (l >= a.L) return;
  bf16* cache = (z & 1 ? a.vc : a.kc) + a.kv_layer * layer;
  bf16* flat = (z & 1 ? a.v : a.k) + ((size_t)layer * gridDim.y + b) * a.L * a.H * kHeadDim;
  uint4* c = reinterpret_cast<uint4*>(cache + (((size_t)b * a.H + h) * a.Lcap + l) * kHeadDim + ch * 8);
  uint4* f = reinterpret_cast<uint4*>(flat + ((size_t)l * a.H + h) * kHeadDim + ch * 8);
  if (LOAD) *c = *f; else *f = *c;
}
hipError_t cache_load(hipStream_t st, const SeqState& s, const CacheFlat& a, int B) {
  hipLaunchKernelGGL(cache_flat_kernel<true>, dim3(std::max((a.L * a.H * 8 + 255) / 256, 1), B, 2 * a.layers + 1), dim3(256), 0, st, s, a);
  return hipGetLastError();
}
hipError_t cache_read(hipStream_t st, const CacheFlat& a, int B) {
  hipLaunchKernelGGL(cache_flat_kernel<false>, dim3((a.L * a.H * 8 + 255) / 256, B, 2 * a.layers), dim3(256), 0, st, SeqState{}, a);
  return hipGetLastError();
}

// ---- FP8 E4M3 weight storage (1-4-3, bias 7, largest value 448, no infinities) ----------------
// Nearest code of |x|, ties to the even mantissa, saturating at 448 (0x7e).
__device__ __forceinline__ unsigned e4m3_code(float x) {
  const unsigned sign = (__float_as_uint(x) >> 24) & 0x80u;
  const float a = fabsf(x);
  unsigned code;
  if (a >= 448.f) {
    code = 0x7eu;
  } else if (a < 0x1p-6f) {
    const unsigned q = (unsigned)rintf(a * 512.f);   // subnormal grid: multiples of 2^-9
    code = q >= 8u ? 0x08u : q;
  } else {
    const unsigned bits = __float_as_uint(a);
    int E = (int)(bits >> 23) - 127;
    unsigned m = (bits >> 20) & 7u;
    const unsigned rem = bits & 0xfffffu;
    if (rem > 0x80000u || (rem == 0x80000u && (m & 1u))) ++m;
    if (m == 8u) { m = 0u; ++E; }
    code = min(((unsigned)(E + 7) << 3) | m, 0x7eu);
  }
  return code | sign;
}
__global__ __launch_bounds__(256) void quantize_rows_kernel(const bf16* __restrict__ w, int K,
                                                            unsigned char* __restrict__ codes,
                                                            float* __restrict__ scale) {
  __shared__ float red[4];
  const bf16* row = w + (size_t)blockIdx.x * K;
  float amax = 0.f;
  for (int k = threadIdx.x * 8; k < K; k += 256 * 8) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(row + k);
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf((float)v[i]));
  }
  amax = wave_max(amax);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const float s = amax > 0.f ? __fdiv_rn(amax, 448.f) : 1.f;
  if (threadIdx.x == 0) scale[blockIdx.x] = s;
  for (int k = threadIdx.x * 8; k < K; k += 256 * 8) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(row + k);
    unsigned lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo |= e4m3_code(__fdiv_rn((float)v[i], s)) << (8 * i);
      hi |= e4m3_code(__fdiv_rn((float)v[4 + i], s)) << (8 * i);
    }
    *reinterpret_cast<uint2*>(codes + (size_t)blockIdx.x * K + k) = make_uint2(lo, hi);
  }
}
// One wave per block of 8 keys.  Keys: lane = (row lane/8, dims 8*(lane%8) .. +7).  Values (key-blocked:
// element (key r, dim e) of the block at e*8 + r): lane = dim e, its 8 elements are the 8 keys.
__global__ __launch_bounds__(256) void quantize_cross_kv_kernel(const bf16* __restrict__ xk, const bf16* __restrict__ xv,
                                                                long n_blocks, unsigned char* __restrict__ k8,
                                                                unsigned char* __restrict__ v8, float* __restrict__ ksc,
                                                                float* __restrict__ vsc) {
  const long blk = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (blk >= n_blocks) return;
  const int lane = threadIdx.x & 63;
  const long off = blk * 512 + lane * 8;
  {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(xk + off);
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf((float)v[i]));
    amax = fmaxf(amax, __shfl_xor(amax, 1, 64));
    amax = fmaxf(amax, __shfl_xor(amax, 2, 64));
    amax = fmaxf(amax, __shfl_xor(amax, 4, 64));
    const float s = amax > 0.f ? __fdiv_rn(amax, 448.f) : 1.f;
    unsigned lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lo |= e4m3_code(__fdiv_rn((float)v[i], s)) << (8 * i);
      hi |= e4m3_code(__fdiv_rn((float)v[4 + i], s)) << (8 * i);
    }
    *reinterpret_cast<uint2*>(k8 + off) = make_uint2(lo, hi);
    if ((lane & 7) == 0) ksc[blk * 8 + (lane >> 3)] = s;
  }
  {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(xv + off);
    unsigned lo = 0, hi = 0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float amax = wave_max(fabsf((float)v[r]));
      const float s = amax > 0.f ? __fdiv_rn(amax, 448.f) : 1.f;
      const unsigned code = e4m3_code(__fdiv_rn((float)v[r], s));
      if (r < 4) lo |= code << (8 * r); else hi |= code << (8 * (r - 4));
      if (lane == r) vsc[blk * 8 + r] = s;
    }
    *reinterpret_cast<uint2*>(v8 + off) = make_uint2(lo, hi);
  }
}
hipError_t quantize_cross_kv(hipStream_t st, const bf16* xk, const bf16* xv, long rows, unsigned char* k8,
                             unsigned char* v8, float* ksc, float* vsc) {
  if (rows <= 0) return hipSuccess;
  if (rows % 8 != 0 || rows / 8 > 0x7fffffffL * 4) return hipErrorInvalidValue;
  const long n_blocks = rows / 8;
  hipLaunchKernelGGL(quantize_cross_kv_kernel, dim3((unsigned)((n_blocks + 3) / 4)), dim3(256), 0, st, xk, xv, n_blocks, k8,
                     v8, ksc, vsc);
  return hipGetLastError();
}

hipError_t quantize_rows_e4m3(hipStream_t st, const bf16* w, int N, int K, unsigned char* codes, float* scale) {
  if (N <= 0) return hipSuccess;
  if (K <= 0 || K % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(quantize_rows_kernel, dim3(N), dim3(256), 0, st, w, K, codes, scale);
  return hipGetLastError();
}

}  // namespace sd
