// The decoder layers of a pass as one kernel, each XCD on sequences of its own (xcd_core.h): layout of the weights, plans, the call.
#include "xcd_core.h"

namespace sd {
namespace xcd {
// ---- layout of the weights -----------------------------------------------------------------
// A wave's stream: layers, chunks of a layer in the order of the stages (FFN2: chunks of K, column tiles inside).  One block a chunk.
template <int D>
__global__ __launch_bounds__(64) void pl_pack_kernel(const PlLayer* __restrict__ layers, int n_layers, char* __restrict__ stream) {
  typedef PlDim<D> Dim;
  const int chunk = blockIdx.x, c = chunk % Dim::kPerLayer, l = chunk / Dim::kPerLayer % n_layers, ww = chunk / (Dim::kPerLayer * n_layers);
  const int wave = ww % kPlWaves, w = ww / kPlWaves, lane = threadIdx.x;
  int s = 0, i = c;
  while (i >= pl_chunks<Dim>(s)) i -= pl_chunks<Dim>(s++);
  const PlLayer& Y = layers[l];
  const void* W = s == 0 ? Y.wqkv.p : s == 2 ? Y.wo.p : s == 3 ? Y.cwq.p : s == 5 ? Y.cwo.p : s == 6 ? Y.w1.p : Y.w2.p;
  const int K = s == 7 ? 4 * D : D, tile = s == 7 ? w * Dim::kTD + i % Dim::kTD : w * pl_chunks<Dim>(s) + i, k0 = s == 7 ? i / Dim::kTD * D : 0;
  const bf16* src = static_cast<const bf16*>(W) + (size_t)(tile * 16 + (lane & 15)) * K + k0 + wave * Dim::KW + 8 * (lane >> 4);
#pragma unroll
  for (int u = 0; u < Dim::KS; ++u)
    *reinterpret_cast<bf16x8*>(stream + (size_t)chunk * Dim::kChunk + u * 1024 + lane * 16) = *reinterpret_cast<const bf16x8*>(src + u * 32);
}
// Column vectors of one layer and workgroup (PlDim::kVec*).
template <int D>
__global__ __launch_bounds__(256) void pl_pack_vectors_kernel(const PlLayer* __restrict__ layers, float* __restrict__ vecs) {
  typedef PlDim<D> Dim;
  const int l = blockIdx.x / kPlMembers, w = blockIdx.x % kPlMembers;
  const PlLayer& Y = layers[l];
  float* out = vecs + (size_t)blockIdx.x * Dim::kVecPitch;
  auto put = [&](const float* v, int n) {
    for (int i = threadIdx.x; i < n; i += 256) out[i] = v[w * n + i];
    out += n;
  };
  put(Y.qkv_cs, Dim::kNQ); put(Y.qkv_bf, Dim::kNQ);
  put(Y.cq_cs, Dim::kND); put(Y.cq_bf, Dim::kND);
  put(Y.w1_cs, Dim::kNF); put(Y.w1_bf, Dim::kNF);
  const float* sums[3] = {Y.vo, Y.vco, Y.v2};
  for (int k = 0; k < 3; ++k)
    for (int i = 0; i < 3; ++i) put(sums[k] + i * D, Dim::kND);
}
// The cross-attention's query matrix as operands of its 16-column tiles (PlOwnQueries): [layer][tile][wave], a chunk each.  One block a chunk.
template <int D>
__global__ __launch_bounds__(64) void pl_pack_queries_kernel(const PlLayer* __restrict__ layers, char* __restrict__ out) {
  typedef PlDim<D> Dim;
  const int chunk = blockIdx.x, wave = chunk % kPlWaves, tile = chunk / kPlWaves % (D / 16), l = chunk / (kPlWaves * (D / 16)), lane = threadIdx.x;
  const bf16* src = static_cast<const bf16*>(layers[l].cwq.p) + (size_t)(tile * 16 + (lane & 15)) * D + wave * Dim::KW + 8 * (lane >> 4);
#pragma unroll
  for (int u = 0; u < Dim::KS; ++u)
    *reinterpret_cast<bf16x8*>(out + (size_t)chunk * Dim::kChunk + u * 1024 + lane * 16) = *reinterpret_cast<const bf16x8*>(src + u * 32);
}
}  // namespace xcd
size_t xcd_stream_bytes(int layers, int d, int F) { return (size_t)layers * (6 * (size_t)d * d + 2 * (size_t)d * F) * sizeof(bf16); }
size_t xcd_vec_bytes(int layers, int d) {
  return (size_t)layers * xcd::kPlMembers * (d == 512 ? xcd::PlDim<512>::kVecPitch : xcd::PlDim<1024>::kVecPitch) * sizeof(float) +
         (d == 512 ? (size_t)layers * d * d * sizeof(bf16) : 0);   // (the query matrix, see PlOwnQueries)
}
template <int D>
static hipError_t pack(hipStream_t st, const PlLayer* layers, int n, char* stream, float* vecs) {
  if (stream) hipLaunchKernelGGL(xcd::pl_pack_kernel<D>, dim3(xcd::kPlMembers * xcd::kPlWaves * n * xcd::PlDim<D>::kPerLayer), dim3(64), 0, st, layers, n, stream);
  hipLaunchKernelGGL(xcd::pl_pack_vectors_kernel<D>, dim3(n * xcd::kPlMembers), dim3(256), 0, st, layers, vecs);
  if constexpr (D == 512)
    hipLaunchKernelGGL(xcd::pl_pack_queries_kernel<D>, dim3(n * (D / 16) * xcd::kPlWaves), dim3(64), 0, st, layers,
                       reinterpret_cast<char*>(vecs + (size_t)n * xcd::kPlMembers * xcd::PlDim<D>::kVecPitch));
  return hipGetLastError();
}
// (stream null: column vectors alone)
hipError_t xcd_pack(hipStream_t st, const PlLayer* layers, int n, int d, char* stream, float* vecs) {
  return d == 512 ? pack<512>(st, layers, n, stream, vecs) : pack<1024>(st, layers, n, stream, vecs);
}

namespace xcd {
// ---- launcher ------------------------------------------------------------------------------
// (each in a file of its own: they take a minute to compile)
extern template hipError_t pl_launch_both<false, 512>(hipStream_t, XcdArgs, int);
extern template hipError_t pl_launch_both<true, 512>(hipStream_t, XcdArgs, int);
extern template hipError_t pl_launch_both<false, 1024>(hipStream_t, XcdArgs, int);
extern template hipError_t pl_launch_both<true, 1024>(hipStream_t, XcdArgs, int);
}  // namespace xcd

int xcd_copy_rows_most(int max_batch, int max_T, int d) {
  const int of_group = xcd::pl_copy_rows_most(d);
  int most = 0;
  for (int T = 1; T <= max_T && T <= of_group; ++T) {
    const int B = std::min(max_batch, xcd::kPlGroups * (of_group / T));
    most = std::max(most, B * T);
  }
  return most;
}
size_t xcd_plan(XcdArgs& a, int d, int F) {
  a.RP = xcd::pl_group_rows(a.B, a.T);
  a.d = d;
  a.G = a.B < xcd::kPlGroups ? a.B : xcd::kPlGroups;
  if (a.RP > xcd::pl_rows_most(d)) return 0;
  a.copy = a.RP <= xcd::pl_copy_rows_most(d);
  // waves to a unit of attention: as many as leave every unit its own
  const int units = (a.B + a.G - 1) / a.G * a.H * ((a.T + 15) >> 4);
  a.wpu = xcd::kPlWaves;
  while (a.wpu > 1 && units > xcd::kPlMembers * (xcd::kPlWaves / a.wpu)) a.wpu >>= 1;
  a.form = 2 * units <= xcd::kPlMembers;
  return xcd::pl_exch_bytes(a.B, a.RP, d, F, a.RP > xcd::kPlRows ? 1 : 2);
}
hipError_t xcd_decoder(hipStream_t st, XcdArgs a, const XcdRoom& room, int d, int F, bool give_up) {
  if (a.R < 1 || a.T < 1 || a.T > xcd::pl_rows_most(d) || a.R != a.B * a.T || !persist_supported(a.n_layers, d, F)) return hipErrorInvalidValue;
  const XcdRoom need = xcd_needs(a.B, a.T, d, F);
  if (xcd_plan(a, d, F) == 0 || (a.stream && !a.copy) || need.rows > room.rows || need.exch > room.exch) return hipErrorInvalidValue;
  a.tickets = reinterpret_cast<PlTickets*>(a.exch);
  a.exch += kPlTicketBytes;
  a.raised = a.err;
  // give_up: a place of every group stays empty, as where other kernels hold compute units: the waits for it end at their bound.  (A bound
  // passed as an argument, or where a wait's count starts, cost 0.1 - 0.6 % of every pass.)  Weights in place: at their first look at the flag,
  // which is raised beforehand; whether it is, the workgroups then ask of the second run's.
  const int blocks = give_up ? kPlBlocks - xcd::kPlGroups : kPlBlocks;
  if (give_up && !a.stream) {
    const hipError_t e = fill_i32(st, reinterpret_cast<int*>(a.err), kPlTicketPasses, 1);
    if (e != hipSuccess) return e;
    a.raised = a.err + 1;
  }
  if (d == 512) return a.xk_scale ? xcd::pl_launch_both<true, 512>(st, a, blocks) : xcd::pl_launch_both<false, 512>(st, a, blocks);
  return a.xk_scale ? xcd::pl_launch_both<true, 1024>(st, a, blocks) : xcd::pl_launch_both<false, 1024>(st, a, blocks);
}

}  // namespace sd
