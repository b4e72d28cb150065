// Scaled dot-product attention for few queries against a streamed key/value set, on MFMA.
//
// A wave owns one (sequence, head) pair and a group of up to 16*NQT queries; it walks the keys
// in chunks of 32 with an online softmax.  Query, key and blocked-value operands are 16-byte
// global loads in exactly the register layout the instruction wants.
//
//   S^T[key][q]  = sum_e K[key][e] Q[q][e]        mfma 16x16x32: A = key rows, B = query rows
//   O^T[e][q]   += sum_key V^T[e][key] P^T[key][q] mfma 16x16x32: A = V^T rows, B = P (registers)
//
// Row i of key tile t stands for key c0 + 8*(i/4) + 4*t + i%4, so that the eight scores a lane
// holds after the two S^T tiles (q = lane%16, keys c0 + 8*(lane/16) .. +7) are already the B
// operand of the second product, and its V^T operand is one contiguous 16-byte load.  This is
// what the key-blocked value layout (vt_off) of the cross-attention values is for; values in
// row layout (the self-attention cache, appended row by row) are turned around through a
// wave-private LDS tile instead.  Both results keep q = lane%16, so the running max / sum of
// a query live in the lanes that hold its accumulators.
//
// A query sees keys [0, limit): causal verify rows (limit grows by one per row), the
// drafter's mask slots (limit = whole block), padded cross / encoder attention (limit = source
// length).  With key_split the 4 waves of a block share one pair and take every 4th chunk;
// their partial (max, sum, O) are merged through LDS.
#include "attn_core.h"
#include "gemm_core.h"

namespace sd {

constexpr int kAttnThreads = 256;

template <int NQT, bool VBLK, bool KV8>
__global__ __launch_bounds__(kAttnThreads) void attn_kernel(AttnArgs a) {
  __shared__ float Om[4][NQT * 16][kHeadDim + 1];
  __shared__ float Ms[4][NQT * 16], Ls[4][NQT * 16];
  __shared__ __attribute__((aligned(16))) bf16 Vs[VBLK ? 1 : 4][VBLK ? 1 : 32][kVtPitch];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 15, g = lane >> 4;
  const int qgroups = (a.T + NQT * 16 - 1) / (NQT * 16);
  int pair, q0, kw, kstep;
  if (a.key_split) {
    pair = blockIdx.x / qgroups; q0 = (blockIdx.x % qgroups) * NQT * 16; kw = wave; kstep = 4;
  } else {
    const int u = blockIdx.x * 4 + wave;
    pair = u / qgroups; q0 = (u % qgroups) * NQT * 16; kw = 0; kstep = 1;
  }
  const bool active_pair = pair < a.B * a.H;
  const int b = active_pair ? pair / a.H : 0, h = active_pair ? pair % a.H : 0;
  float mrun[NQT], lrun[NQT];
  f32x4 oacc[NQT][4];
  int nq = active_pair ? -1 : 0;   // -1: the pair's query count is read inside, after the first requests
  attn_wave<NQT, VBLK, false, false, KV8>(a, b, h, q0, nq, kw, kstep, Vs[VBLK ? 0 : wave], mrun, lrun, oacc);
  bf16* obase = a.q_off ? a.o + (long)(active_pair ? a.q_off[b] : 0) * a.o_row : a.o + b * a.o_b;

  // oacc[qt][et][r] = O^T[e = et*16 + 4g + r][q = qt*16 + lq]
  if (!a.key_split) {
    if (!active_pair) return;
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
      const int qi = qt * 16 + lq;
      if (qi < nq) {
        const float inv = lrun[qt] > 0.f ? 1.f / lrun[qt] : 0.f;
        bf16* op = obase + (long)(q0 + qi) * a.o_row + h * kHeadDim;
#pragma unroll
        for (int et = 0; et < 4; ++et) {
          bf16x4 w;
#pragma unroll
          for (int r = 0; r < 4; ++r) w[r] = (bf16)(oacc[qt][et][r] * inv);
          *reinterpret_cast<bf16x4*>(op + et * 16 + 4 * g) = w;
        }
      }
    }
    return;
  }
  // merge the four key splits
#pragma unroll
  for (int qt = 0; qt < NQT; ++qt) {
    const int qi = qt * 16 + lq;
    if (g == 0) { Ms[wave][qi] = mrun[qt]; Ls[wave][qi] = lrun[qt]; }
#pragma unroll
    for (int et = 0; et < 4; ++et)
#pragma unroll
      for (int r = 0; r < 4; ++r) Om[wave][qi][et * 16 + 4 * g + r] = oacc[qt][et][r];
  }
  __syncthreads();
  for (int idx = tid; idx < NQT * 16 * kHeadDim; idx += kAttnThreads) {
    const int qi = idx >> 6, e = idx & 63;
    if (qi < nq) {
      float M = kNegInf;
#pragma unroll
      for (int w = 0; w < 4; ++w) M = fmaxf(M, Ms[w][qi]);
      float L = 0.f, O = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float mw = Ms[w][qi];
        const float f = (mw > kNegInf) ? __expf(mw - M) : 0.f;
        L += Ls[w][qi] * f;
        O += Om[w][qi][e] * f;
      }
      obase[(long)(q0 + qi) * a.o_row + h * kHeadDim + e] = (bf16)(L > 0.f ? O / L : 0.f);
    }
  }
}

// ----------------------------------------------------------------------------- many queries (encoder, prefill)
// A block owns 128 queries of one (sequence, head) pair, 32 per wave, and walks the keys in tiles of 64 that its four
// waves share through LDS (global -> LDS requests, two buffers, one barrier per tile):
//   S^T[key][q]  = K Q^T     mfma 32x32x16: A = key rows (LDS), B = query rows (registers)
//   O^T[e][q]   += V^T P^T   mfma 32x32x16: A = V^T (LDS), B = P (registers)
// Row i of a 32-key half stands for key 16 (i/16) + 8 ((i/4)%2) + 4 ((i/8)%2) + i%4, so that a lane's scores are runs of
// eight consecutive keys of its query: already the B operand of the second product.  Values in row layout become V^T
// operands through the transposing LDS read (a 16-lane group turns 4 keys x 16 dims); key-blocked ones are the operand.
// Per 64 keys and wave: 16 MFMAs (512 cycles) against about 1100 cycles of softmax (a quarter-rate exponential per
// score), so the vector pipe bounds it (busy 79 % of the time, the matrix pipe 43) and what matters is instructions per score: row maxima
// are exchanged once per tile, row sums once per pass, masking happens only on tiles a limit cuts, accumulators are rescaled only when some
// maximum has moved by more than kSlack (at every move, which with 32 rows is nearly every tile, it took 6 % longer).  120 registers,
// four waves a SIMD; with 140, three of them, 16 % longer.
// 32 x 16 heads, 1024 queries on 1024 keys: 163 us in an encoder (843 TFLOP/s), 775 with the kernel above, whose waves fetch keys and values
// one by one.
constexpr int kTileQ = 128, kTileK = 64;

template <bool VBLK>
__global__ __launch_bounds__(256, 3) void attn_tile_kernel(AttnArgs a, int qgroups, int units) {
  __shared__ __attribute__((aligned(1024))) bf16 smem[2][2][kTileK * 64];   // [buffer][keys, values]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, half = lane >> 5;
  // an XCD takes consecutive pairs, all query groups of a pair one after the other: keys / values stay in its L2
  const int per = (units + 7) >> 3, u = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || u >= units) return;
  const int pair = u / qgroups, q0 = (u - pair * qgroups) * kTileQ;
  const int b = pair / a.H, h = pair - b * a.H;
  const int nq = a.q_count ? a.q_count[b] : a.T;
  if (q0 >= nq) return;
  const int qo = a.q_off ? a.q_off[b] : 0;
  const int qi = q0 + wave * 32 + lq, row = min(qi, nq - 1);   // (a lane without a query repeats the last one)
  const bf16* qp = a.q + (a.q_off ? (long)qo * a.q_row : b * a.q_b) + (long)row * a.q_row + h * kHeadDim + half * 8;
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
  const int lim = a.lim_row ? a.lim_row[(a.q_off ? qo : b * a.T) + row] : a.lim_seq[b];
  const int kmax = wave_max_i(lim), kmin = -wave_max_i(-lim);   // of this wave's queries
  // the block's last key: limits grow with the row or are the same for all (lim_row of the last query otherwise short)
  __shared__ int kmaxs[4];
  if (lane == 0) kmaxs[wave] = kmax;
  lds_barrier();
  const int kend = max(max(kmaxs[0], kmaxs[1]), max(kmaxs[2], kmaxs[3]));

  const bf16* kbase = a.k + (a.kv_off ? (long)a.kv_off[b] * a.k_row : b * a.k_b) + h * a.k_h;
  const bf16* vbase = a.v + (a.kv_off ? (long)a.kv_off[b] * a.v_row : b * a.v_b) + h * a.v_h;
  // Request i of a wave moves rows 16 wave + 8 i .. + 7 of a tile's keys or values.  A lane's offsets from a tile's first row are the same for
  // every tile but one that the last key cuts, and the tile's own place is scalar (row strides are whole lines): with an address a lane
  // and request, 25 instructions more a tile, 168 us in place of 163 below.
  const int row0 = wave * 16 + (lane >> 3), kpitch = a.k_row * 2, vpitch = a.v_row * 2;
  const unsigned kpiece = ((lane & 7) ^ (lane >> 4)) << 4, vpiece = ((lane & 7) ^ ((lane >> 2) & 4)) << 4;   // row 8 i on: keys ^ 64, values the same
  const unsigned koff = row0 * kpitch + kpiece, voff = row0 * vpitch + vpiece;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(&smem[0][0][0])) + wave * 2048;
  auto stage = [&](int c0, int buf) {
    const bf16* kt = kbase + (long)c0 * a.k_row;
    const unsigned l = lds0 + buf * (2 * kTileK * 128);
    const bool whole = c0 + kTileK <= kend;
    if (whole) {
      dma16(kt, koff, l);
      dma16(kt + 8 * a.k_row, koff ^ 64, l + 1024);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) dma16(kt, min(row0 + 8 * i, kend - 1 - c0) * kpitch + (kpiece ^ (i * 64)), l + i * 1024);
    }
    if constexpr (VBLK) {   // 1 KB = one block of 8 keys
#pragma unroll
      for (int i = 0; i < 2; ++i)
        dma16(vbase + (long)min((c0 >> 3) + wave * 2 + i, (a.cap >> 3) - 1) * (8 * kHeadDim), lane * 16, l + kTileK * 128 + i * 1024);
    } else {
      const bf16* vt = vbase + (long)c0 * a.v_row;
      if (whole) {
        dma16(vt, voff, l + kTileK * 128);
        dma16(vt + 8 * a.v_row, voff, l + kTileK * 128 + 1024);
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) dma16(vt, min(row0 + 8 * i, kend - 1 - c0) * vpitch + vpiece, l + kTileK * 128 + i * 1024);
      }
    }
  };
  if (kend > 0) stage(0, 0);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[ks][e] = (bf16)((float)qf[ks][e] * 0.125f);   // exact: power of two

  constexpr float kLog2e = 1.44269504088896341f;
  // What the exponentials are relative to (mrun) follows the row's maximum only when some row's has grown by more than this
  // (then for all): probabilities up to 256 instead of 1 cost no precision, and sums of them no range.
  constexpr float kSlack = 8.f / kLog2e;
  float mrun = kNegInf, lrun = 0.f;
  f32x16 oacc[2];
#pragma unroll
  for (int et = 0; et < 2; ++et)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[et][r] = 0.f;
  // LDS offsets: K row of this lane (permuted), V^T sources
  const int krow = 16 * (lq >> 4) + 8 * ((lq >> 2) & 1) + 4 * ((lq >> 3) & 1) + (lq & 3);
  const int t16 = lane & 15, vr = t16 >> 2, vc = ((lane >> 4) & 1) * 16 + 4 * (t16 & 3);

  int buf = 0;
  for (int c0 = 0; c0 < kend; c0 += kTileK, buf ^= 1) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    block_barrier();   // tile c0 has landed for every wave, and everyone is done with the other buffer
    if (c0 + kTileK < kend) stage(c0 + kTileK, buf ^ 1);
    if (c0 >= kmax) continue;   // (same for the whole wave)
    const bf16 *ks_ = smem[buf][0], *vs_ = smem[buf][1];
    f32x16 s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(ks_ + lds_off<64>(t * 32 + krow, ks * 2 + half));
        s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[t], 0, 0, 0);
      }
    }
    mfma_settle(s[0], s[1]);
    if (c0 + kTileK > kmin) {   // some query of the wave does not see the whole tile
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = c0 + t * 32 + 16 * (r >> 3) + 8 * half + (r & 7);
          s[t][r] = key < lim ? s[t][r] : kNegInf;
        }
    }
    float cm = s[0][0];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) cm = fmaxf(cm, s[t][r]);
    cm = half_max(cm);
    const float mnew = fmaxf(mrun, cm);
    const bool move = __builtin_amdgcn_ballot_w64(mnew > mrun + kSlack) != 0;
    const float mref = move ? mnew : mrun, nb = mref > kNegInf ? -mref * kLog2e : 0.f;
    if (move) {
      const float alpha = __builtin_amdgcn_exp2f(__builtin_fmaf(mrun, kLog2e, nb));   // 0 on first use
      lrun *= alpha;
#pragma unroll
      for (int et = 0; et < 2; ++et)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[et][r] *= alpha;
      mrun = mnew;
    }
    bf16x8 pf[4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], kLog2e, nb));
        lrun += p;
        pf[2 * t + (r >> 3)][r & 7] = (bf16)p;
      }
    const bool cut = VBLK && c0 + kTileK > kend;   // blocks hold keys beyond the last one, which may be anything
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int et = 0; et < 2; ++et) {
        bf16x8 vf;
        if constexpr (VBLK) {
          vf = *reinterpret_cast<const bf16x8*>(vs_ + ((2 * kb + half) * 64 + et * 32 + lq) * 8);
          if (cut) vf = zero_tail(vf, kend - (c0 + 16 * kb + 8 * half));
        } else {
          s16x4 p[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int r = 16 * kb + 8 * half + 4 * i + vr, c = et * 32 + vc;
            p[i] = lds_tr16(vs_ + r * 64 + (((c >> 3) ^ ((r & 2) << 1)) << 3) + (c & 7));
          }
          __builtin_memcpy(&vf, p, 16);
        }
        oacc[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kb], oacc[et], 0, 0, 0);
      }
  }
  mfma_settle(oacc[0]);
  mfma_settle(oacc[1]);
  lrun = half_add(lrun);
  const float inv = lrun > 0.f ? 1.f / lrun : 0.f;
  // a lane holds dims et*32 + 8 q + 4 half .. + 3; the halves swap so that each stores eight consecutive dims
  bf16* op = a.o + (a.q_off ? (long)qo * a.o_row : b * a.o_b) + (long)qi * a.o_row + h * kHeadDim;
#pragma unroll
  for (int et = 0; et < 2; ++et)
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
      bf16x4 w[2];
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) w[g][i] = (bf16)(oacc[et][(q + g) * 4 + i] * inv);
      const bf16x8 v = join_halves(w[0], w[1]);
      if (qi < nq) *reinterpret_cast<bf16x8*>(op + et * 32 + 8 * (q + half)) = v;
    }
}

template <bool VBLK>
static hipError_t attention_tile_launch(hipStream_t st, const AttnArgs& a) {
  const int qgroups = (a.T + kTileQ - 1) / kTileQ, units = a.B * a.H * qgroups;
  SD_LAUNCH_TIMED((attn_tile_kernel<VBLK>), dim3(8 * ((units + 7) / 8)), dim3(256), 0, st, a, qgroups, units);
  return hipGetLastError();
}

template <bool VBLK, bool KV8>
static hipError_t attention_launch(hipStream_t st, const AttnArgs& a) {
  const int nqt = a.T <= 16 ? 1 : (a.T <= 32 || !KV8 ? 2 : 4);   // (4: 8-bit keys / values only, see attention())
  const int qgroups = (a.T + nqt * 16 - 1) / (nqt * 16);
  const long units = (long)a.B * a.H * qgroups;
  const unsigned blocks = (unsigned)(a.key_split ? units : (units + 3) / 4);
  if (nqt == 1) SD_LAUNCH_TIMED((attn_kernel<1, VBLK, KV8>), dim3(blocks), dim3(kAttnThreads), 0, st, a);
  else if (nqt == 2) SD_LAUNCH_TIMED((attn_kernel<2, VBLK, KV8>), dim3(blocks), dim3(kAttnThreads), 0, st, a);
  else if constexpr (KV8) SD_LAUNCH_TIMED((attn_kernel<4, VBLK, KV8>), dim3(blocks), dim3(kAttnThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t attention(hipStream_t st, const AttnArgs& a) {
  if (a.B <= 0 || a.T <= 0) return hipSuccess;
  if (a.cap < 32 || a.cap % 32 != 0) return hipErrorInvalidValue;   // whole chunks are read
  if (a.k_scale || a.v_scale) {   // FP8 keys and values
    if (!a.k_scale || !a.v_scale || !a.v_blocked) return hipErrorInvalidValue;
    return attention_launch<true, true>(st, a);
  }
  // Beyond 32 queries a sequence the tile kernel, whose 128 queries a block may mostly not be there: a drafter pass of k = 16, 25, 31
  // (T = 2 k + 1 bounds its 17 .. 63 rows a sequence), 1 - 55 sequences of 16 - 230 cached tokens on 32 - 1024 source keys, mean of
  // its self- and cross-attention launches: 6.1 - 18.5 us against 8.6 - 21.5 with attn_kernel<4> and its split keys, better at
  // every one of 99 points.
  if (a.T > 32 || a.kv_off) return a.v_blocked ? attention_tile_launch<true>(st, a) : attention_tile_launch<false>(st, a);
  return a.v_blocked ? attention_launch<true, false>(st, a) : attention_launch<false, false>(st, a);
}

}  // namespace sd
