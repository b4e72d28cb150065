// The decoder layers of a pass of few rows as ONE kernel whose workgroups hand over through memory.
//
// With few rows a decoder layer is eight dependent products and attentions of a microsecond each, and as separate kernels
// every hand-over costs a launch (about 4 us from one kernel's operands to the next one's).  Here up to kPlBlocks workgroups
// of four (d = 512) or eight (1024) waves stay resident for all layers, with seven hand-overs in each: queries / keys / values,
// self-attention, its output product, cross-attention (whose units form their queries themselves), its output product, and
// the two FFN matrices.  What one workgroup produces for another goes to an exchange buffer that holds kPoison in
// every 32-bit word beforehand (the pass's first kernel writes it); the consumers load the words they need, coherently and
// straight into MFMA operand registers, until none of them is kPoison any more.  The value is its own flag: a hand-over is
// one store and one load through memory, 1.0 - 1.4 us, plus 0.6 - 1.1 us of work, with no barrier, no counter and no fence.
// No word of a result is ever stored as kPoison (not_poison).
//
// Work items of a stage are dealt to the workgroups round robin; the three residual-sum products of a layer give a workgroup
// the same tile each time, so that the fp32 residual stays in its LDS.  An item is 16 MR rows x 16 FB columns: the
// waves split K, each lane requests its weight fragments before it waits for the rows (they arrive meanwhile), the partial
// tiles are summed through LDS in wave order, and the waves divide the 16 x 16 results.  LayerNorm is folded into the products as
// in the general kernels (gemm.hip), with statistics per 16 columns.
//
// What bounds it: the chain of 7 hand-overs a layer.  A whole verify pass of 6 layers, separate launches -> this kernel: d = 512, 6 rows
// 200 -> 112 us, 48 228 -> 131; d = 1024, 6 rows 252 -> 159, 26 293 -> 193, with E4M3 weights 285 -> 200.  Beyond 64 rows
// of d = 1024, items of 32 rows: 121 rows 323 -> 283.  More rows (from 129 of d = 1024 on), and at d = 512 all passes with bf16 weights on a
// stream that has every compute unit, are the per-XCD decoder's (xcd_core.h).  Larger items were tried (48 x 64, 352 rows) and are level with separate launches: every item fetches its rows and weights at the 60 - 75 GB/s one CU takes in,
// whether the rows come through the L2 (counters instead of kPoison) or not, and whether or not the next weights are requested ahead.
//
// The workgroups wait for each other, so all of them have to be running.  There are no more of them than the stream has CUs and
// the host lets one such pass at a time onto a GPU, but a kernel of another stream or process may hold some of the CUs.  Waits
// are therefore bounded: after kPlSpinMax polls, or once another workgroup has raised the error flag, a wave raises it and ends,
// and the same stages are run again by the kernel launched behind this one (TICKETS), which returns at once where the flag is
// not raised.  Its workgroups draw (stage, virtual workgroup) tickets in the order of the stages and wait only for
// stages whose tickets have all been drawn, that is for workgroups that are running: it needs no more than one CU.  It computes
// the same bits.  The flag counts the passes that go to it directly (kPlTicketPasses, this one included) before one waits again.
// A whole verify pass with the second launch returning at once and without it: 125.3 / 124.8 us (d = 512, 6 rows),
// 380.2 / 378.0 (d = 1024, 128 rows); by tickets 0.51 and 2.7 ms.
#include "resident_core.h"

namespace sd {

constexpr unsigned kPlSpinMax = 1u << 17;   // (0.1 - 0.2 s)
constexpr int kPlTicketBlocks = 64;
__device__ __forceinline__ bool pl_missing(const u32x4& v) {
  return v[0] == kPoison || v[1] == kPoison || v[2] == kPoison || v[3] == kPoison;
}
__device__ __forceinline__ void pl_store8(void* p, unsigned a, unsigned b) {
  u32x2 v = {not_poison(a), not_poison(b)};
  asm volatile("global_store_dwordx2 %0, %1, off sc0 sc1" ::"v"(p), "v"(v) : "memory");
}

// One more round of a wait: false once the pass is to be abandoned.
__device__ __forceinline__ bool pl_again(unsigned& spins, const PlArgs& a) {
  ++spins;
  if ((spins & a.poll_mask) == 0) {
    const bool raised = __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    if (raised || spins > a.spin_max) {
      __hip_atomic_store(a.err, kPlTicketPasses, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
  }
  __builtin_amdgcn_s_sleep(1);
  return true;
}

struct PlStat { float rstd, nmr; };
// mean and rstd of row lq from its chunk pairs of 16 columns; this lane holds NS of them
template <int NS>
__device__ __forceinline__ PlStat pl_stat(const u32x2 (&pairs)[NS], int d) {
  f32x2 p[NS];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    p[i] = __builtin_bit_cast(f32x2, pairs[i]);
    s += p[i][0];
  }
  const float inv_d = __builtin_amdgcn_rcpf((float)d), mean = pl_row_sum(s) * inv_d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const float dv = p[i][0] * (1.f / 16) - mean;
    q += p[i][1] + 16.f * dv * dv;
  }
  const float rstd = fast_rsqrt(pl_row_sum(q) * inv_d + 1e-5f);
  return PlStat{rstd, -mean * rstd};
}

__device__ __forceinline__ int pl_opaque(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

constexpr int kPlQPitch = 72;   // (16 rows of 144 bytes: a 16-byte read of every row meets all banks once)

// NP: pairs (row tile, column tile) of the largest item; more than four: one set of partial tiles instead of two in turn
template <int NW, int NP>
struct PlLds {
  static constexpr int kFlips = NP > 4 ? 1 : 2, kRows = NP > 4 ? 32 : 16;
  f32x4 red[kFlips][NW * NP * 64];                // partial tiles
  float resid[kRows * 16];                        // of the workgroup's residual-sum tile
  float stat[kFlips][2 * kRows];                  // {rstd, -mean rstd} of the rows, beside red
  bf16 q[16 * kPlQPitch];                         // queries of the workgroup's unit (cross-attention)
  unsigned long long layers[kPlLayers * sizeof(PlLayer) / 8];   // every stage's pointers
  unsigned raised;                                // (of the first wave's look at the flag)
  // attention: partial results in the first half of red, the value tiles of the waves ([32 keys][64], swizzled like the tile
  // kernel's) in the second
  static_assert(kFlips * NP >= 8, "attention's share of red");
  __device__ __forceinline__ f32x4* om() { return red[0]; }
  __device__ __forceinline__ float* ml() { return reinterpret_cast<float*>(red[0] + NW * 4 * 64); }
  __device__ __forceinline__ bf16* vs(int wave) { return reinterpret_cast<bf16*>(red[0] + NW * 4 * 64) + wave * (32 * 64); }
};

// Product of one item: rows row0 .. row0 + 16 MR - 1 below rlim of A (exchange buffer, or plain rows), columns n0 .. n0 +
// 16 FB - 1 of W [N][32 * NW * KS].  done(mr, f, v, s) receives the finished sums of row row0 + 16 mr + lane % 16, columns
// n0 + 16 f + 4 (lane / 16) .. + 3 (on the waves these pairs fall to, f = wave % FB), and the statistics of that row (stats
// null: {1, 0}); wave NW - 1 - mr reduces those of row tile mr.  late: the statistics are as new as the rows and are waited for
// with them; otherwise they were there long ago and are taken first.
// WT: bf16 values, or E4M3 codes that become bf16 operands as they arrive (the caller applies the columns' scales).
template <class WT> struct PlFrag { typedef bf16x8 type; };
template <> struct PlFrag<fp8> { typedef fp8x8 type; };
__device__ __forceinline__ bf16x8 pl_operand(const bf16x8& f) { return f; }
__device__ __forceinline__ bf16x8 pl_operand(const fp8x8& f) { return e4m3x8_to_bf16(f); }
template <class WT, int NW, int KS, int MR, int FB, int NS, bool LATE, class Lds, class Done>
__device__ __forceinline__ bool pl_product(const PlArgs& a, Lds& L, int flip, const void* Wv, const char* A, bool plain, int row0,
                                           int rlim, int n0, const char* stats, Done&& done) {
  constexpr int K = 32 * NW * KS;
  static_assert(MR <= NW && NW % FB == 0, "a wave per row tile's statistics; a wave's column tile");
  const int lane = pl_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lq = lane & 15, g = lane >> 4;
  f32x4* red = L.red[flip];
  float* rstat = L.stat[flip];
  const WT* W = static_cast<const WT*>(Wv);
  typename PlFrag<WT>::type wf[FB][KS];
#pragma unroll
  for (int f = 0; f < FB; ++f)
#pragma unroll
    for (int u = 0; u < KS; ++u)
      wf[f][u] = *reinterpret_cast<const typename PlFrag<WT>::type*>(W + (size_t)(n0 + 16 * f + lq) * K + (wave * KS + u) * 32 + 8 * g);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  const int smr = NW - 1 - wave;   // whose statistics this wave reduces
  const bool has_stat = stats && smr < MR;
  const int srow = min(row0 + 16 * smr + lq, rlim - 1);
  const bool s_on = row0 + 16 * smr + lq < rlim;
  u32x2 st[NS];
  auto stat_request = [&]() {   // chunks g * NS .. of the row
    const PlBuf sb = pl_buf(stats);
#pragma unroll
    for (int i = 0; i < NS; ++i) st[i] = __builtin_amdgcn_raw_buffer_load_b64(sb, (g * NS * a.RP + srow) * 8, i * a.RP * 8, kPlSc1);
  };
  auto stat_missing = [&]() {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < NS; ++i) bad |= st[i][0] == kPoison || st[i][1] == kPoison;
    return bad && s_on;
  };
  unsigned spins = 0;
  auto stat_reduce = [&]() {
    const PlStat s = pl_stat<NS>(st, a.d);
    if (g == 0) { rstat[32 * smr + 2 * lq] = s.rstd; rstat[32 * smr + 2 * lq + 1] = s.nmr; }
  };
  if (Lds::kFlips == 1) lds_barrier();   // the partial tiles and statistics of the item before have been read
  if (!LATE && has_stat) {
    stat_request();
    while (__builtin_amdgcn_ballot_w64(stat_missing())) {
      if (!pl_again(spins, a)) return false;
      asm volatile("" ::: "memory");
      stat_request();
    }
    stat_reduce();
  }
  // row fragments in chunks of CH, DEPTH chunks requested ahead; chunk c: k fragments (c / MR) * CH .. of row tile c % MR
  constexpr int CH = 4, NC = MR * KS / CH, DEPTH = NC < 4 ? NC : 4;
  static_assert(KS % CH == 0, "whole chunks");
  const PlBuf buf = pl_buf(A);
  u32x4 af[DEPTH][CH];
  auto request = [&](int c) {
    const int row = min(row0 + 16 * (c % MR) + lq, rlim - 1), k = (wave * KS + c / MR * CH) * 32 + 8 * g;
    if (plain) {   // rows another kernel wrote, [R][K]
#pragma unroll
      for (int u = 0; u < CH; ++u) af[c % DEPTH][u] = *reinterpret_cast<const u32x4*>(A + ((size_t)row * K + k + u * 32) * 2);
    } else {
      const int off = pl_at(a.RP, row, k);
#pragma unroll
      for (int u = 0; u < CH; ++u) af[c % DEPTH][u] = pl_request(buf, off, u * a.RP * 64);
    }
  };
#pragma unroll
  for (int c = 0; c < DEPTH; ++c) request(c);
  if (LATE && has_stat) stat_request();
  f32x4 acc[MR][FB];
#pragma unroll
  for (int mr = 0; mr < MR; ++mr)
#pragma unroll
    for (int f = 0; f < FB; ++f) acc[mr][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Waits for chunks c .. c + n - 1; what is missing, of those in flight behind them as well, once more, and nothing else: with all of them again
  // at every look, those that were there held up the others' next look (128 rows of d = 1024 370.9 us, so 363.1; 6 rows 173.7 / 168.0; load by
  // load instead of chunk by chunk 365.5).
  auto arrive = [&](int c, int n) {
    while (true) {
      bool miss[DEPTH], any = false;
#pragma unroll
      for (int i = 0; i < DEPTH; ++i) {
        miss[i] = false;
        if (c + i >= NC) continue;
        unsigned m = 0u;   // (rows beyond the last: that one again)
#pragma unroll
        for (int u = 0; u < CH; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) m = max(m, af[(c + i) % DEPTH][u][e]);
        miss[i] = __builtin_amdgcn_ballot_w64(m == kPoison) != 0;
        if (i < n) any |= miss[i];
      }
      bool late = false;
      if (LATE && has_stat && c == 0) late = __builtin_amdgcn_ballot_w64(stat_missing()) != 0;
      if (!any && !late) return true;
      if (!pl_again(spins, a)) return false;
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i < DEPTH; ++i)
        if (miss[i]) request(c + i);
      if (late) stat_request();
    }
  };
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (!plain && (c == 0 || c >= DEPTH) && !arrive(c, c == 0 ? DEPTH : 1)) return false;
    if (LATE && c == 0 && has_stat) stat_reduce();
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
      for (int u = 0; u < CH; ++u)
        acc[c % MR][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pl_operand(wf[f][c / MR * CH + u]), __builtin_bit_cast(bf16x8, af[c % DEPTH][u]),
                                                                 acc[c % MR][f], 0, 0, 0);
    if (c + DEPTH < NC) request(c + DEPTH);
  }
#pragma unroll
  for (int mr = 0; mr < MR; ++mr)
#pragma unroll
    for (int f = 0; f < FB; ++f) {
      mfma_settle(acc[mr][f]);
      red[((wave * MR + mr) * FB + f) * 64 + lane] = acc[mr][f];
    }
  lds_barrier();
#pragma unroll
  for (int p0 = 0; p0 < MR * FB; p0 += NW) {
    const int p = p0 + wave;
    if (p >= MR * FB) break;
    f32x4 t[NW], v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) t[w] = red[(w * MR * FB + p) * 64 + lane];
    PlStat s{1.f, 0.f};
    const int mr = p / FB;
    if (stats) s = PlStat{rstat[32 * mr + 2 * lq], rstat[32 * mr + 2 * lq + 1]};
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += t[w][e];
    done(mr, p % FB, v, s);
  }
  return true;
}

// hidden(LayerNorm folded) W^T + b of one item; epi(row, n, float[4]) on live rows
template <class WT, int NW, int KS, int MR, int FB, int NS, class Lds, class Epi>
__device__ __forceinline__ bool pl_project(const PlArgs& a, Lds& L, int flip, const PlWeight& W, const float* cs, const float* bf,
                                           const char* A, bool plain, const char* stats, int row0, int rlim, int n0, Epi&& epi) {
  const int lane = pl_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lq = lane & 15, g = lane >> 4;
  const int n = n0 + 16 * (wave % FB) + 4 * g;
  const f32x4 c4 = *reinterpret_cast<const f32x4*>(cs + n), b4 = *reinterpret_cast<const f32x4*>(bf + n);
  f32x4 w4 = {1.f, 1.f, 1.f, 1.f};
  if constexpr (sizeof(WT) == 1) w4 = *reinterpret_cast<const f32x4*>(W.scale + n);
  return pl_product<WT, NW, KS, MR, FB, NS, true>(a, L, flip, W.p, A, plain, row0, rlim, n0, stats, [&](int mr, int, const f32x4& v, const PlStat& s) {
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(sizeof(WT) == 1 ? v[e] * w4[e] : v[e], s.rstd, __builtin_fmaf(s.nmr, c4[e], b4[e]));
    const int row = row0 + 16 * mr + lq;
    if (row < rlim) epi(row, n, o);
  });
}

// residual sum of one item: y = LN_prev(x) + A W^T + b; xg, statistics and the workgroup's copy of y
template <class WT, int NW, int KS, int MR, int NS, class Lds>
__device__ __forceinline__ bool pl_sum(const PlArgs& a, Lds& L, int flip, float* resid, const PlWeight& W, const float* vecs,
                                       const char* A, const char* stats_prev, bool first, bool last, char* xg, char* st_out,
                                       int row0, int n0) {
  const int lane = pl_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lq = lane & 15, g = lane >> 4;
  const int n = n0 + 4 * g;
  f32x4 cv[3], w4 = {1.f, 1.f, 1.f, 1.f};
  if constexpr (sizeof(WT) == 1) w4 = *reinterpret_cast<const f32x4*>(W.scale + n);
#pragma unroll
  for (int i = 0; i < 3; ++i) cv[i] = *reinterpret_cast<const f32x4*>(vecs + i * a.d + n);
  static_assert(MR <= NW, "a pair per wave");
  const int mine = min(wave, MR - 1);
  float* own = resid + (mine * 16 + lq) * 16 + 4 * g;
  f32x4 x;
  if (first) x = *reinterpret_cast<const f32x4*>(a.x + (size_t)min(row0 + 16 * mine + lq, a.R - 1) * a.d + n);
  else x = *reinterpret_cast<const f32x4*>(own);
  return pl_product<WT, NW, KS, MR, 1, NS, false>(a, L, flip, W.p, A, false, row0, a.R, n0, stats_prev, [&](int mr, int, const f32x4& v, const PlStat& s) {
    const int row = row0 + 16 * mr + lq;
    float y[4], gx[4], sum = 0.f, ss = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y[e] = (sizeof(WT) == 1 ? v[e] * w4[e] : v[e]) + __builtin_fmaf(__builtin_fmaf(x[e], s.rstd, s.nmr), cv[0][e], cv[1][e]);
      gx[e] = y[e] * cv[2][e];
    }
    const bool live = row < a.R;
    if (last) {
      if (live) *reinterpret_cast<f32x4*>(a.y + (size_t)row * a.d + n) = f32x4{y[0], y[1], y[2], y[3]};
      return;
    }
    const u32x2 w = pl_pack4(gx);
    if (live) pl_store8(xg + pl_at(a.RP, row, n), w[0], w[1]);
#pragma unroll
    for (int e = 0; e < 4; ++e) { sum += y[e]; ss = __builtin_fmaf(y[e], y[e], ss); }
    sum = pl_row_sum(sum);
    ss = pl_row_sum(ss);
    if (live && g == 0)
      pl_store8(st_out + ((n0 >> 4) * a.RP + row) * 8, __builtin_bit_cast(unsigned, sum),
                __builtin_bit_cast(unsigned, fmaxf(ss - sum * sum * (1.0f / 16), 0.f)));
    *reinterpret_cast<f32x4*>(own) = f32x4{y[0], y[1], y[2], y[3]};
  });
}

template <bool SELF>
__device__ __forceinline__ PlUnit pl_unit(const PlArgs& a, int u) {
  const int tiles = (a.T + 15) >> 4, pair = u / tiles;
  PlUnit t;
  t.b = pair / a.H; t.h = pair - t.b * a.H; t.q0 = (u - pair * tiles) * 16;
  t.j = SELF ? a.row_pos[t.b * a.T] : 0;
  t.nkey = SELF ? t.j + min(a.T, t.q0 + 16) : a.src_len[t.b];
  return t;
}

// Key chunks kw, kw + kstep, ... of 32 on this wave (see attn_core.h for the operand layouts).  SELF: keys / values below the
// pass's first row come from the cache, the pass's own from the exchange buffers (waited for); else the cross-attention arenas.
// QLDS: the queries are in LDS (q_lds) once form_q() has returned; it runs behind the first keys' and values' requests.
// KV8 (cross): codes with one fp32 scale per key and per value, as in attn_core.h.
template <bool SELF, bool QLDS, bool KV8, class FormQ>
__device__ __forceinline__ bool pl_attn_wave(const PlArgs& a, const PlExch& ex, int l, const PlUnit& t, int kw, int kstep,
                                             const bf16* q_lds, FormQ&& form_q, bf16* Vs, float& mrun, float& lrun,
                                             f32x4 (&oacc)[4]) {
  const int lane = pl_lane(), lq = lane & 15, g = lane >> 4;
  const int r0 = t.b * a.T;                                // first row of the sequence
  const int j = t.j, nkey = t.nkey;
  const int cap = SELF ? a.Lcap : a.Scap;
  const size_t arena = ((size_t)t.b * a.H + t.h) * cap * kHeadDim;
  constexpr int EB = KV8 ? 1 : 2;   // bytes of an element
  const char* kb = (SELF ? reinterpret_cast<const char*>(a.kc + a.kv_layer * l) : static_cast<const char*>(a.xk) + a.xkv_layer * l * EB) + arena * EB;
  const char* vb = (SELF ? reinterpret_cast<const char*>(a.vc + a.kv_layer * l) : static_cast<const char*>(a.xv) + a.xkv_layer * l * EB) + arena * EB;
  const size_t sc0 = KV8 ? (a.xkv_layer * l + arena) / kHeadDim : 0;
  mrun = kNegInf;
  lrun = 0.f;
#pragma unroll
  for (int et = 0; et < 4; ++et) oacc[et] = f32x4{0.f, 0.f, 0.f, 0.f};
  // K operands: tile i, row lq  <->  key c0 + 8*(lq/4) + 4*i + lq%4; values as whole rows (lane -> row 8*i + lane/8, dims
  // 8*(lane%8) .. + 7) or, key-blocked, as operands.  What the cache holds is requested once, the pass's own rows until they
  // are there.
  PlChunk now, next;
  u32x4 f[2];
  auto key_k = [&](int c0, int i) { return c0 + 8 * (lq >> 2) + 4 * i + (lq & 3); };
  auto key_v = [&](int c0, int i) { return c0 + 8 * i + (lane >> 3); };
  auto fetch = [&](int c0, PlChunk& t) {
    const int last = (SELF ? j : nkey) - 1;
    if (SELF && c0 > last) return;
    if constexpr (KV8) {
      const int k8 = min(c0 + 8 * g, cap - 8);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const char* p = kb + max(min(key_k(c0, i), last), 0) * 64 + g * 8;
        t.kf8[2 * i] = *reinterpret_cast<const fp8x8*>(p);
        t.kf8[2 * i + 1] = *reinterpret_cast<const fp8x8*>(p + 32);
        t.sck[i] = *reinterpret_cast<const f32x4*>(a.xk_scale + sc0 + k8 + 4 * i);
        t.scv[i] = *reinterpret_cast<const f32x4*>(a.xv_scale + sc0 + k8 + 4 * i);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) t.vf8[i] = *reinterpret_cast<const fp8x8*>(vb + vt_off(k8, i * 16 + lq));
      return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const char* p = kb + max(min(key_k(c0, i), last), 0) * 128 + g * 16;
      t.kf[2 * i] = *reinterpret_cast<const u32x4*>(p);
      t.kf[2 * i + 1] = *reinterpret_cast<const u32x4*>(p + 64);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      t.vf[i] = *reinterpret_cast<const u32x4*>(SELF ? vb + min(key_v(c0, i), last) * 128 + (lane & 7) * 16
                                                   : vb + vt_off(min(c0 + 8 * g, cap - 8), i * 16 + lq) * 2);
  };
  // the chunk's own rows (SELF) and, with_q, the queries
  auto await = [&](int c0, bool with_q) {
    const bool own = SELF && c0 + 32 > j;
    if (!own && !with_q) return true;
    const PlBuf kxb = pl_buf(ex.kx()), vxb = pl_buf(ex.vx()), qb = pl_buf(ex.q(SELF ? 0 : 1));
    const int off = pl_at(a.RP, r0, t.h * kHeadDim), xtile = a.RP * 32;
    const int offk = off + pl_at(a.RP, 0, 8 * g), offv = off + pl_at(a.RP, 0, 8 * (lane & 7));
    unsigned spins = 0;
    while (true) {
      u32x4 kn[4], vn[4];
      bool bad = false;
      if (own) {
#pragma unroll
        for (int i = 0; i < 4; ++i) kn[i] = pl_request(kxb, offk + min(max(key_k(c0, i >> 1) - j, 0), a.T - 1) * 32, (i & 1) * 2 * xtile);
#pragma unroll
        for (int i = 0; i < 4; ++i) vn[i] = pl_request(vxb, offv + min(max(key_v(c0, i) - j, 0), a.T - 1) * 32, 0);
      }
      if (with_q) {
#pragma unroll
        for (int i = 0; i < 2; ++i) f[i] = pl_request(qb, offk + min(t.q0 + lq, a.T - 1) * 32, i * 2 * xtile);
      }
      if (own) {   // (keys at and beyond nkey are masked later: not waited for)
#pragma unroll
        for (int i = 0; i < 4; ++i) bad |= key_k(c0, i >> 1) >= j && key_k(c0, i >> 1) < nkey && pl_missing(kn[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) bad |= key_v(c0, i) >= j && key_v(c0, i) < nkey && pl_missing(vn[i]);
      }
      if (with_q) bad |= pl_missing(f[0]) || pl_missing(f[1]);
      if (!__builtin_amdgcn_ballot_w64(bad)) {
        if (own) {
          // (values beyond nkey meet a probability of zero: they must be finite)
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              now.kf[i][e] = key_k(c0, i >> 1) >= j ? kn[i][e] : now.kf[i][e];
              now.vf[i][e] = key_v(c0, i) >= nkey ? 0u : key_v(c0, i) >= j ? vn[i][e] : now.vf[i][e];
            }
        }
        return true;
      }
      if (!pl_again(spins, a)) return false;
      asm volatile("" ::: "memory");
    }
  };
  const int cfirst = kw * 32;
  fetch(cfirst, now);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (QLDS) {   // formed by this workgroup
    if (!await(cfirst, false)) return false;
    if (!form_q()) return false;
#pragma unroll
    for (int i = 0; i < 2; ++i) f[i] = *reinterpret_cast<const u32x4*>(q_lds + lq * kPlQPitch + i * 32 + 8 * g);
  } else {
    if (!await(cfirst, true)) return false;
  }
  const bf16x8 q0 = __builtin_bit_cast(bf16x8, f[0]), q1 = __builtin_bit_cast(bf16x8, f[1]);
  const int lim = t.q0 + lq < a.T ? (SELF ? j + t.q0 + lq + 1 : nkey) : 0;
  for (int c0 = cfirst; c0 < nkey; c0 += kstep * 32) {
    const int c1 = c0 + kstep * 32;
    if (c1 < nkey) fetch(c1, next);
    bf16x8 vo[4];
    if constexpr (KV8) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        now.kf[i] = __builtin_bit_cast(u32x4, e4m3x8_to_bf16(now.kf8[i]));
        now.vf[i] = __builtin_bit_cast(u32x4, e4m3x8_to_bf16(now.vf8[i]));
      }
    }
    if constexpr (SELF) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + (lane >> 3);
        *reinterpret_cast<u32x4*>(Vs + r * 64 + (((lane & 7) ^ ((r & 2) << 1)) << 3)) = now.vf[i];
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int et = 0; et < 4; ++et) {
        const int r = 8 * g + ((lane >> 2) & 3), c = et * 16 + 4 * (lane & 3);
        const bf16* src = Vs + r * 64 + (((c >> 3) ^ ((r & 2) << 1)) << 3) + (c & 7);   // (row r + 4 has the same swizzle)
        s16x4 p[2] = {lds_tr16(src), lds_tr16(src + 4 * 64)};
        __builtin_memcpy(&vo[et], p, 16);
      }
    } else {
#pragma unroll
      for (int et = 0; et < 4; ++et) vo[et] = __builtin_bit_cast(bf16x8, now.vf[et]);
      if (c0 + 32 > nkey) {
#pragma unroll
        for (int et = 0; et < 4; ++et) vo[et] = zero_tail(vo[et], nkey - (c0 + 8 * g));
      }
    }
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, now.kf[0]), q0, s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, now.kf[2]), q0, s1, 0, 0, 0);
    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, now.kf[1]), q1, s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, now.kf[3]), q1, s1, 0, 0, 0);
    mfma_settle(s0, s1);
    if constexpr (KV8) {
#pragma unroll
      for (int r = 0; r < 4; ++r) { s0[r] *= now.sck[0][r]; s1[r] *= now.sck[1][r]; }
    }
    const int left = lim - (c0 + 8 * g);   // this lane: query lq, keys c0 + 8 g .. + 7, of which it sees the first `left`
    float s[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = r < left ? s0[r] : kNegInf;
      s[4 + r] = 4 + r < left ? s1[r] : kNegInf;
    }
    float cm = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
    {
      const unsigned u = __builtin_bit_cast(unsigned, cm);
      const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
      cm = half_max(fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])));
    }
    const float mnew = fmaxf(mrun, cm);
    const float nb = mnew > kNegInf ? -mnew * kCexp : 0.f;   // nothing seen yet: every exponential below is of -inf
    bf16x8 pf;
    float p[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], kCexp, nb));
      // (a masked key's scale may be anything, NaN included)
      if constexpr (KV8) pf[r] = (bf16)(r < left ? p[r] * now.scv[r >> 2][r & 3] : 0.f);
      else pf[r] = (bf16)p[r];
    }
    const float ps = pl_row_sum(((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])));
    if (c0 == cfirst) {
      lrun = ps;
    } else {
      const float alpha = __builtin_amdgcn_exp2f(__builtin_fmaf(mrun, kCexp, nb));
      lrun = lrun * alpha + ps;
#pragma unroll
      for (int et = 0; et < 4; ++et)
#pragma unroll
        for (int r = 0; r < 4; ++r) oacc[et][r] *= alpha;
    }
    mrun = mnew;
#pragma unroll
    for (int et = 0; et < 4; ++et) oacc[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vo[et], pf, oacc[et], 0, 0, 0);
    if (c1 < nkey) {
      now = next;
      if (!await(c1, false)) return false;
    }
  }
  mfma_settle(oacc);
  return true;
}

// All units of one attention stage.  No more units than workgroups: a workgroup each (mine); else as many waves each as there
// are, a power of two, several units to a workgroup.  The waves of a unit take chunks of 32 keys in turn and merge through LDS.
template <int NW, bool SELF, bool QLDS, bool KV8, class Lds, class FormQ>
__device__ __forceinline__ bool pl_attention(const PlArgs& a, const PlExch& ex, int l, int w, int NB, int units, const PlUnit& mine, Lds& L,
                                             FormQ&& form_q) {
  const int lane = pl_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lq = lane & 15, g = lane >> 4;
  if (units <= NB && (unsigned)w >= (unsigned)units) return true;   // (w: number among the workgroups that take units)
  char* out = ex.att(SELF ? 0 : 1);
  const int wpu = QLDS ? NW : a.wpu, per = NW / wpu, kw = wave & (wpu - 1);   // waves of a unit, units at a time
  for (int u0 = w * per; u0 < units; u0 += NB * per) {
    const int u = u0 + wave / wpu;
    const bool any = u < units;
    PlUnit t = mine;
    if (!QLDS && units > NB) t = pl_unit<SELF>(a, any ? u : units - 1);
    const int chunks = (t.nkey + 31) >> 5, used = any ? min(max(chunks, 1), wpu) : 0;   // waves with keys (one at least)
    float mrun, lrun;
    f32x4 oacc[4];
    auto store = [&](int et, const f32x4& o, float inv) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = o[r] * inv;
      const u32x2 p = pl_pack4(v);
      if (t.q0 + lq < a.T) pl_store8(out + pl_at(a.RP, t.b * a.T + t.q0 + lq, t.h * kHeadDim + et * 16 + 4 * g), p[0], p[1]);
    };
    lds_barrier();   // the latest product's partial tiles, or the units' before, are done with
    // (every wave takes part in forming the queries; one beyond the keys then finds none)
    if ((QLDS || kw < used) &&
        !pl_attn_wave<SELF, QLDS, KV8>(a, ex, l, t, kw, wpu, L.q, form_q, L.vs(wave), mrun, lrun, oacc))
      return false;
    if (wpu == 1 || (per == 1 && used <= 1)) {   // nothing to merge
      const float inv = lrun > 0.f ? __builtin_amdgcn_rcpf(lrun) : 0.f;
      if (any && kw == 0)
#pragma unroll
        for (int et = 0; et < 4; ++et) store(et, oacc[et], inv);
      continue;
    }
    // O of every wave to LDS; wave et of the unit (two or more et's where it has few waves) merges dims 16 et .. + 15
    f32x4* om = L.om();   // [wave][et][lane]
    float* ml = L.ml();   // [wave][max, sum][16]  (the value tiles are done with)
    lds_barrier();
    if (kw < used) {
#pragma unroll
      for (int et = 0; et < 4; ++et) om[(wave * 4 + et) * 64 + lane] = oacc[et];
      if (g == 0) { ml[wave * 32 + lq] = mrun; ml[wave * 32 + 16 + lq] = lrun; }
    }
    lds_barrier();
    if (any) {
      const int first = wave - kw;
      float M = kNegInf, Ls = 0.f;
      for (int s = first; s < first + used; ++s) M = fmaxf(M, ml[s * 32 + lq]);
      for (int s = first; s < first + used; ++s) {
        const float ms = ml[s * 32 + lq];
        Ls += ml[s * 32 + 16 + lq] * (ms > kNegInf ? __builtin_amdgcn_exp2f((ms - M) * kCexp) : 0.f);
      }
      const float inv = Ls > 0.f ? __builtin_amdgcn_rcpf(Ls) : 0.f;
      for (int et = kw; et < 4; et += wpu) {
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        for (int s = first; s < first + used; ++s) {
          const float ms = ml[s * 32 + lq], e = ms > kNegInf ? __builtin_amdgcn_exp2f((ms - M) * kCexp) : 0.f;
          const f32x4 v = om[(s * 4 + et) * 64 + lane];
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] += v[r] * e;
        }
        store(et, o, inv);
      }
    }
  }
  lds_barrier();
  return true;
}

// WT: weights (bf16 or E4M3 codes).  KV8: cross-attention keys / values as E4M3 codes.
// MR: row tiles of an item.  FBW: column tiles of an item of the wide projections (QKV, first FFN matrix).
// TICKETS: see the head of this file; a.NB virtual workgroups, the residual in memory instead of LDS (MR = 1).
template <class WT, bool KV8, int NW, int KSD, int KSF, int MR, int FBW, bool TICKETS>
__global__ __launch_bounds__((64 * NW), 2) void pl_decoder_kernel(PlArgs a) {
  extern __shared__ __attribute__((aligned(16))) char pl_smem[];
  typedef PlLds<NW, (MR > 1 ? MR * FBW : 4)> Lds;
  static_assert(Lds::kRows == 16 * MR, "residual tile");
  Lds& L = *reinterpret_cast<Lds*>(pl_smem);
  constexpr int d = 32 * NW * KSD, F = 32 * NW * KSF, NS = d / 64;   // statistics: d / 16 pairs over four lanes
  // wide projections from the top, sums from the bottom, attention units from att0 on: where there is room a workgroup has one
  // kind of item and its weights are on their way long before the rows are
  const int NB = TICKETS ? a.NB : gridDim.x;
  int w = blockIdx.x;
  // Without tickets one look for all waves: others may raise the flag meanwhile, and a wave that goes on needs what every other one
  // has put into L.layers.  (With them nothing else writes it until every workgroup has drawn a ticket.)
  unsigned raised = 0;
  if (TICKETS || threadIdx.x == 0) raised = __hip_atomic_load(a.raised, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (TICKETS && raised == 0u) return;
  {
    const int words = a.n_layers * (int)(sizeof(PlLayer) / 8);
    for (int i = threadIdx.x; i < words; i += (64 * NW)) L.layers[i] = reinterpret_cast<const unsigned long long*>(a.layers)[i];
  }
  const int units = a.B * a.H * ((a.T + 15) >> 4);
  PlUnit self{}, cross{};
  auto take_units = [&]() {
    const int wa = w - a.att0;
    if ((unsigned)wa < (unsigned)units && units <= NB) {
      self = pl_unit<true>(a, wa);
      cross = pl_unit<false>(a, wa);
    }
  };
  if (!TICKETS) take_units();
  if (!TICKETS && threadIdx.x == 0) L.raised = raised;
  __syncthreads();
  if (!TICKETS && __builtin_amdgcn_readfirstlane(L.raised) != 0u) return;
  int flip = 0;
  auto turn = [&]() { return Lds::kFlips == 1 ? 0 : flip ^= 1; };
  const int RT = (a.R + 16 * MR - 1) / (16 * MR);
  // items of a projection with N columns: 16 MR rows x 16 FB columns each, column tile fastest (tiles of one column range then share an XCD)
  auto project = [&](auto fbt, int N, const PlWeight& W, const float* cs, const float* bf, const char* A, bool plain,
                     const char* stats, auto&& epi) -> bool {
    constexpr int FB = decltype(fbt)::value;
    const int nt = pl_opaque(N / (16 * FB)), items = nt * RT;
    for (int it = NB - 1 - w; it < items; it += NB) {
      const int mt = it / nt;
      if (!pl_project<WT, NW, KSD, MR, FB, NS>(a, L, turn(), W, cs, bf, A, plain, stats, mt * 16 * MR, a.R, (it - mt * nt) * 16 * FB, epi)) return false;
    }
    return true;
  };
  auto sum = [&](auto kst, const PlWeight& W, const float* vecs, const char* A, const char* stats_prev, bool first, bool last,
                 char* xg, char* st) -> bool {
    constexpr int KS = decltype(kst)::value, nt = d / 16;
    for (int it = w; it < nt * RT; it += NB) {
      const int mt = it / nt;
      if (!pl_sum<WT, NW, KS, MR, NS>(a, L, turn(), TICKETS ? a.resid + it * (256 * MR) : L.resid, W, vecs, A, stats_prev, first, last,
                                      xg, st, mt * 16 * MR, (it - mt * nt) * 16)) return false;
      if (!TICKETS) break;   // (the plan gives a workgroup at most one)
    }
    return true;
  };
  typedef std::integral_constant<int, KSD> CD;
  typedef std::integral_constant<int, KSF> CF;
  typedef std::integral_constant<int, FBW> CW;
  typedef std::integral_constant<int, 1> C1;
  // stage s of layer l, of workgroup w
  auto stage = [&](int s, int l) __attribute__((always_inline)) -> bool {
    // (what follows from the layer is worked out where it is used: ahead of its stages, where the compiler would have it, it does not fit the
    // scalar registers; 26 rows of d = 1024, 8-bit weights 206.5 us, so 204.1)
    asm volatile("" : "+s"(l));
    const int wa = units <= NB ? w - a.att0 : w;
    const PlLayer& Y = reinterpret_cast<const PlLayer*>(L.layers)[l];
    const PlExch ex(a.exch + (size_t)l * pl_layer_bytes(a.RP, d, F), a.RP, d), before(a.exch + (size_t)(l - 1) * pl_layer_bytes(a.RP, d, F), a.RP, d);
    const bool top = l == 0;
    const char* st0 = top ? nullptr : before.st(2);
    switch (s) {
      case 0:   // queries, keys, values (appended to the cache as well)
        return project(CW{}, 3 * d, Y.wqkv, Y.qkv_cs, Y.qkv_bf, top ? reinterpret_cast<const char*>(a.xb) : before.xg(2), top, st0,
                       [&](int row, int n, const float (&v)[4]) {
          const int part = n / d, c = n - part * d;
          const u32x2 p = pl_pack4(v);
          char* dst = (part == 0 ? ex.q(0) : part == 1 ? ex.kx() : ex.vx()) + pl_at(a.RP, row, c);
          pl_store8(dst, p[0], p[1]);
          const int b = a.row_b[row];
          if (part == 0 || b < 0) return;
          bf16* cache = (part == 1 ? a.kc : a.vc) + a.kv_layer * l +
                        (((size_t)b * a.H + (c >> 6)) * a.Lcap + a.row_pos[row]) * kHeadDim + (c & 63);
          *reinterpret_cast<u32x2*>(cache) = p;
        });
      case 1: return pl_attention<NW, true, false, false>(a, ex, l, wa, NB, units, self, L, [] { return true; });
      case 2: return sum(CD{}, Y.wo, Y.vo, ex.att(0), st0, top, false, ex.xg(0), ex.st(0));
      case 3:
        return units <= NB || project(C1{}, d, Y.cwq, Y.cq_cs, Y.cq_bf, ex.xg(0), false, ex.st(0), [&](int row, int n, const float (&v)[4]) {
          const u32x2 p = pl_pack4(v);
          pl_store8(ex.q(1) + pl_at(a.RP, row, n), p[0], p[1]);
        });
      case 4:
        if (units > NB) return pl_attention<NW, false, false, KV8>(a, ex, l, wa, NB, units, cross, L, [] { return true; });
        // a unit's workgroup forms its queries itself: a product of 64 columns instead of a hand-over
        return pl_attention<NW, false, true, KV8>(a, ex, l, wa, NB, units, cross, L, [&] {
          const int row0 = cross.b * a.T + cross.q0, n0 = cross.h * kHeadDim;
          if (!pl_project<WT, NW, KSD, 1, 4, NS>(a, L, turn(), Y.cwq, Y.cq_cs, Y.cq_bf, ex.xg(0), false, ex.st(0), row0, (cross.b + 1) * a.T,
                                          n0, [&](int row, int n, const float (&v)[4]) {
                *reinterpret_cast<u32x2*>(&L.q[(row - row0) * kPlQPitch + n - n0]) = pl_pack4(v);
              })) return false;
          lds_barrier();
          return true;
        });
      case 5: return sum(CD{}, Y.cwo, Y.vco, ex.att(1), ex.st(0), false, false, ex.xg(1), ex.st(1));
      case 6:
        return project(CW{}, F, Y.w1, Y.w1_cs, Y.w1_bf, ex.xg(1), false, ex.st(1), [&](int row, int n, const float (&v)[4]) {
          const float r[4] = {fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
          const u32x2 p = pl_pack4(r);
          pl_store8(ex.hid() + pl_at(a.RP, row, n), p[0], p[1]);
        });
      default: return sum(CF{}, Y.w2, Y.v2, ex.hid(), ex.st(1), false, l + 1 == a.n_layers, ex.xg(2), ex.st(2));
    }
  };
  if constexpr (!TICKETS) {
    for (int l = 0; l < a.n_layers; ++l) {
      if (!stage(0, l) || !stage(1, l) || !stage(2, l) || !stage(3, l) || !stage(4, l) || !stage(5, l) || !stage(6, l) || !stage(7, l)) return;
    }
  } else {
    __shared__ int drawn;
    const int total = a.n_layers * kPlStages * NB;   // (ids of a pass: below 2^24)
    int st = -1;
    while (true) {
      // (In one block: of one at the loop's end and one at its top the compiler can make one with two ways back, and lanes 1 - 63 then go
      // round, barriers and all, without lane 0.)
      if (threadIdx.x == 0) {
        if (st >= 0) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the caches' write-back, which the fence only starts)
          __hip_atomic_fetch_add(&a.tickets->done[st], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        drawn = (int)(__hip_atomic_fetch_add(&a.tickets->drawn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u);
      }
      __syncthreads();
      // a wave that gives up ends, and what it would have drawn or left the others cannot go on with
      if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0) return;
      const int t = __builtin_amdgcn_readfirstlane(drawn);
      st = t / NB;
      const int l = st / kPlStages;
      if (t >= total) {   // (the last workgroup to find none left: every one has read the flag, and nothing else writes it now)
        if (t == total + (int)gridDim.x - 1 && threadIdx.x == 0) *a.raised -= 1;
        return;
      }
      w = t - st * NB;
      // everything before this stage: its tickets are out, so whoever holds them is running
      unsigned spins = 0;
      while (st > 0 && __hip_atomic_load(&a.tickets->done[st - 1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) + 1u != (unsigned)NB)
        if (!pl_again(spins, a)) return;
      take_units();
      if (!stage(st - l * kPlStages, l)) return;
      __syncthreads();   // all stores of the workgroup are out (and the ticket has been read)
    }
  }
}

// ---- launcher ------------------------------------------------------------------------------
bool persist_supported(int layers, int d, int F) {
  return layers <= kPlLayers && ((d == 512 && F == 2048) || (d == 1024 && F == 4096));
}
size_t persist_exch_bytes(int rows, int layers, int d, int F) {
  return kPlTicketBytes + (size_t)layers * pl_layer_bytes((rows + 15) & ~15, d, F);
}

int persist_plan(PlArgs& a, int d, int F) {
  a.RP = (a.R + 15) & ~15;
  a.d = d;
  // Rows of an item: 16 as long as every workgroup has at most one residual sum of 16 x 16, else 32 (weights are read once per
  // item).
  const int most = 3 * d > F ? 3 * d : F, units = a.B * a.H * ((a.T + 15) >> 4);
  a.mr = d / 16 * (a.RP / 16) <= kPlBlocks ? 1 : 2;
  const int rt = (a.R + 16 * a.mr - 1) / (16 * a.mr), sums = d / 16 * rt;
  // The narrowest items of the wide projections that leave every workgroup one kind of item; failing that, that give every
  // workgroup at most one of them.
  auto wide = [&](int fb) { const int n = most / (16 * fb) * rt; return n > sums ? n : sums; };
  int fb = a.mr > 1 ? 4 : 2;
  while (fb < 4 && sums + units + wide(fb) > kPlBlocks) fb *= 2;
  if (a.mr == 1 && sums + units + wide(fb) > kPlBlocks) {
    fb = 2;
    while (fb < 4 && wide(fb) > kPlBlocks) fb *= 2;
  }
  a.fbw = fb;
  int NB = sums + units + wide(fb);
  if (NB > kPlBlocks) NB = kPlBlocks;
  a.att0 = sums + units <= NB ? sums : 0;
  const int nw = d == 512 ? 4 : 8;
  a.wpu = nw;
  while (a.wpu > 1 && units > NB * (nw / a.wpu)) a.wpu >>= 1;
  return sums <= NB ? NB : 0;
}

template <class WT, bool KV8, int NW, int KSD, int KSF, int MR, int FBW, bool TICKETS>
static hipError_t pl_launch(hipStream_t st, const PlArgs& a, int blocks) {
  constexpr int kBytes = (int)sizeof(PlLds<NW, (MR > 1 ? MR * FBW : 4)>);
  static_assert(kBytes <= 160 * 1024, "LDS of a CU");
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(pl_decoder_kernel<WT, KV8, NW, KSD, KSF, MR, FBW, TICKETS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  SD_LAUNCH_TIMED((pl_decoder_kernel<WT, KV8, NW, KSD, KSF, MR, FBW, TICKETS>), dim3(blocks), dim3((64 * NW)), kBytes, st, a);
  return hipGetLastError();
}
template <class WT, bool KV8, int NW>
static hipError_t pl_launch_items(hipStream_t st, const PlArgs& a) {
  if (a.mr == 1) return a.fbw == 2 ? pl_launch<WT, KV8, NW, 4, 16, 1, 2, false>(st, a, a.NB) : pl_launch<WT, KV8, NW, 4, 16, 1, 4, false>(st, a, a.NB);
  if constexpr (sizeof(WT) == 1 || NW == 4) return hipErrorInvalidValue;   // codes, d = 512: passes of fewer rows only
  else return pl_launch<WT, KV8, NW, 4, 16, 2, 4, false>(st, a, a.NB);
}
// the pass, and its second run by tickets (kPlTicketBlocks workgroups: a fraction of the chip, so that it costs little to start)
template <class WT, bool KV8, int NW>
static hipError_t pl_launch_both(hipStream_t st, PlArgs a) {
  const hipError_t e = pl_launch_items<WT, KV8, NW>(st, a);
  if (e != hipSuccess) return e;
  a.err += 1;
  a.poll_mask = 63;
  a.spin_max = kPlTicketSpinMax;
  return pl_launch<WT, KV8, NW, 4, 16, 1, 2, true>(st, a, kPlTicketBlocks);
}
template <class WT, bool KV8>
static hipError_t pl_launch_dims(hipStream_t st, const PlArgs& a, int d) {
  return d == 512 ? pl_launch_both<WT, KV8, 4>(st, a) : pl_launch_both<WT, KV8, 8>(st, a);
}

hipError_t persist_decoder(hipStream_t st, PlArgs a, int d, int F, bool give_up) {
  if (a.R < 1 || a.T < 1 || a.T > 32 || a.R != a.B * a.T || !persist_supported(a.n_layers, d, F)) return hipErrorInvalidValue;
  a.NB = persist_plan(a, d, F);
  if (a.NB < 1) return hipErrorInvalidValue;
  a.tickets = reinterpret_cast<PlTickets*>(a.exch);
  a.exch += kPlTicketBytes;
  a.raised = a.err;
  a.poll_mask = give_up ? 0 : 63;
  a.spin_max = give_up ? 0 : kPlSpinMax;
  if (a.fp8) return a.xk_scale ? pl_launch_dims<fp8, true>(st, a, d) : pl_launch_dims<fp8, false>(st, a, d);
  return a.xk_scale ? pl_launch_dims<bf16, true>(st, a, d) : pl_launch_dims<bf16, false>(st, a, d);
}

}  // namespace sd
