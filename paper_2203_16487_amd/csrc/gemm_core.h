// bf16 "NT" GEMM main loop on MFMA 32x32x16 (gfx950), fp32 accumulation.
//   C[m][n] = sum_k A[m][k] * W[n][k]      A [M,K] row-major (lda), W [N,K] row-major (ldw)
// Both operands are K-contiguous (activations and nn-style weights), so every global access
// is a 16-byte row segment and every MFMA operand is one 16-byte LDS read.
//
// Tiles of BM x BN x 64 move from global memory straight into LDS (global_load_lds, 16 bytes
// per lane, no register staging) through a ring of STAGES buffers, so that STAGES-1 tiles of
// loads are in flight while one is being multiplied: HBM/L2 latency (~1-2 us) is covered by
// depth, not by occupancy.  Waves form a WAVES_M x WAVES_N arrangement (4 or 8 waves).
#pragma once
#include "common.h"
#include <stdint.h>
#include <type_traits>

namespace sd {

constexpr int kGemmThreads = 256;


template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Workgroup barrier without the release/acquire fences of __syncthreads(): those would wait
// for every outstanding global_load_lds (vmcnt(0)) and flatten the pipeline.  The memory
// clobber keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// LDS tile rows hold GK bf16 (the k extent of one pipeline stage) = GK/8 chunks of 16 B.
// GK = 64: chunk c of row r lives at chunk c ^ ((r >> 1) & 7); GK = 32: at c ^ ((r >> 2) & 3).
// Either way 16 consecutive rows reading the same logical chunk touch all 64 banks once.
template <int GK>
__device__ __forceinline__ int lds_off(int row, int chunk) {
  static_assert(GK == 64 || GK == 32, "stage depth");
  return GK == 64 ? row * 64 + ((chunk ^ ((row >> 1) & 7)) << 3) : row * 32 + ((chunk ^ ((row >> 2) & 3)) << 3);
}

template <int BM, int BN, int STAGES, int WAVES_M = 2, int WAVES_N = 2, int GK_ = 64>
struct GemmCfg {
  static constexpr int GK = GK_;
  static constexpr int kRowsPerLoad = 512 / GK;        // tile rows moved by one global_load_lds
  static constexpr int kBM = BM, kBN = BN, kStages = STAGES;
  static constexpr int kWavesM = WAVES_M, kWavesN = WAVES_N, kWaves = WAVES_M * WAVES_N;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kRows = BM + BN;                 // LDS rows per stage (A rows then W rows)
  static constexpr int kIPW = kRows / kRowsPerLoad / kWaves;   // global_load_lds per wave per stage
  static constexpr int kStageElems = kRows * GK;
  static constexpr int kSmemBytes = STAGES * kStageElems * 2;
  // LDS beyond the ring that a bf16 copy of the tile (rows padded by 16 bytes) needs
  static constexpr int kTailBytes = BM * (BN + 8) * 2 > kSmemBytes ? BM * (BN + 8) * 2 - kSmemBytes : 0;
  static constexpr int kWM = BM / WAVES_M, kWN = BN / WAVES_N;   // wave tile
  static constexpr int kTM = kWM / 32, kTN = kWN / 32;           // MFMA tiles per wave
  static_assert(kRows % (kRowsPerLoad * kWaves) == 0 && BM % kRowsPerLoad == 0 && kWM % 32 == 0 && kWN % 32 == 0,
                "tile shape");
};

template <class Cfg>
struct GemmAcc {
  f32x16 c[Cfg::kTM][Cfg::kTN];
};

// Global -> LDS request of 64 lanes x 16 bytes, landing at lds_dst + lane * 16 (lds_dst is the same
// for the whole wave).  An asm statement, so that the compiler does not order it against the LDS
// reads in flight (it would wait for all of them before every request); the ring protocol of the
// main loop guarantees that the slot being filled is not read between the two barriers around the
// request.  The compiler's own vmcnt bookkeeping stays safe: loads complete in order, and a count it
// computes without these requests can only make it wait longer.
__device__ __forceinline__ void dma16(const bf16* g, bf16* lds_dst) {
  const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(lds_dst));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(l), "v"(g));
}

// The same with the address split into a wave-uniform base (scalar registers) and a byte offset per lane: moving on to
// the next stage is then scalar arithmetic, and a request's offset costs one multiply-add.
__device__ __forceinline__ void dma16(const bf16* base, unsigned voff, unsigned lds_dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_dst), "v"(voff), "s"(base));
}

// wait until at most allow * IPW of this wave's requests are outstanding (allow in [0, MAXA])
template <int IPW, int MAXA>
__device__ __forceinline__ void wait_vm_stages(int allow) {
  if constexpr (MAXA <= 0) {
    wait_vmcnt<0>();
  } else {
    if (allow >= MAXA) wait_vmcnt<IPW * MAXA>();
    else wait_vm_stages<IPW, MAXA - 1>(allow);
  }
}

// Whole K range [k_begin, k_begin + GK*KT) of the block tile at (m0, n0).  Rows beyond M / N
// are clamped to the last valid row (their products land in outputs that are never stored).
// Requirements: K % GK == 0, lda/ldw % 8 == 0, A and W 16-byte aligned, smem 1024-aligned.
//
// Stage j (GK columns of k) lives in ring slot j % S and is multiplied in GK/16 sub-steps of one
// MFMA per 32x32 tile each.  What keeps the matrix pipe busy:
//  * the fragments of sub-step s+1 are read from LDS into a second register set while the MFMAs
//    of sub-step s issue, in a fixed order written out in the source (MFMA, LDS read, MFMA, ...);
//  * the block's one barrier per stage sits before the LAST sub-step of stage kt and certifies
//    that stage kt+1 has landed for every wave, so the fragments of (kt+1, 0) are read while the
//    last MFMAs of stage kt run: no wave ever waits for LDS latency right after a barrier;
//  * with S >= 3 the requests of stage kt+S-1 (slot of stage kt-1, free since the barrier inside
//    stage kt-1) go out a few per sub-step during stage kt instead of in one burst; with S = 2
//    the requests of stage kt+2 follow the barrier inside stage kt (the slot just vacated).
// SWAP: W rows take the MFMA's row operand and A rows its column operand: register r of lane l of
// tile (i, j) then holds row m = 32 i + l%32, column n = 32 j + 8*(r/4) + 4*(l/32) + r%4 (relative to
// the wave tile), i.e. a lane owns 16 columns of ONE row per tile instead of 16 rows of one column.
// hook() runs once the first stages are requested (its own loads then travel behind them).
struct NoHook {
  __device__ __forceinline__ void operator()() const {}
};
// The lane, as a value that is not carried over from before: a loop over tiles would hold all addresses that follow from it.
__device__ __forceinline__ int fresh_lane() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}
// The loop of the 256 x 256 tiles (2 x 4 waves of 128 x 64, two ring slots, SWAP): same products in the same order, but a stage is
// walked by A row tile (phase i = row tile i, four steps of k) and not by k.  W's fragments of the whole stage are held (32
// registers, replaced step by step in the last phase), so that a slot is given back a piece at a time: W and row tile 0 before the
// stage's first product, then row tile after row tile, and the next occupant's requests go out two a phase instead of sixteen behind
// one barrier, four to six phases before they are needed.  Barriers stand before phases 0 and 2; what each certifies is what the two
// phases behind it read:
//   before phase 0 of stage kt: row tiles 1, 2 of kt      requested in phase 3 of stage kt - 2
//   before phase 2:             row tile 3 of kt          phase 0 of kt - 1
//                               row tile 0 of kt + 1      phase 0 of kt - 1
//                               W of kt + 1               phases 1, 2 of kt - 1
// Written plainly, 8192^3: 832 us, now 775 (1.42 PFLOP/s; on zeros 710 and 584: the rate of real data is what the card's power
// allows); 32768 x 1024 x 4096: 217, now 207; at K = 1024 1 - 2 % (a tile's fixed costs are a fifth there).
//
// One tile after the other (Tiles): next(m, n) says which follows (false: none; m, n are then the tile's own), done() finishes one and
// says whether every wave sent off exactly STORES vector stores.  The requests of the next tile's first two stages go out in the last two of the
// tile before as if they were its own (behind the last tile, once more its own, which nobody reads), so its first products need not wait,
// and what done() stores is on its way under them: only the waits of the next tile's first stage count the stores among what may
// still be in flight.  KT even and at least 4 (a slot's number does not depend on the tile); done() keeps out of the ring.
struct OneTile {
  static constexpr bool kStream = false;
  static constexpr int kStores = 0;
  __device__ __forceinline__ bool next(int&, int&) const { return false; }
  __device__ __forceinline__ bool done() const { return false; }
};
template <class Cfg, class Hook = NoHook, class Tiles = OneTile>
__device__ __forceinline__ void gemm_mainloop_square(const bf16* __restrict__ A, int lda, const bf16* __restrict__ W, int ldw, int M, int N,
                                                     int k_begin, int KT, int m0, int n0, bf16* smem, GemmAcc<Cfg>& acc, Hook hook = Hook(),
                                                     Tiles tiles = Tiles()) {
  static_assert(Cfg::kBM == 256 && Cfg::kBN == 256 && Cfg::kWavesM == 2 && Cfg::kWavesN == 4 && Cfg::GK == 64 && Cfg::kStages == 2, "shape");
  constexpr int TM = 4, TN = 2, NS = 4, E = Cfg::kStageElems;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
  // request q of a stage: 0 .. 3 row tile q of A (32 rows of either half), 4 .. 7 quarter q - 4 of W; a wave moves 8 rows of each
  unsigned voff[8], voff3;   // (3: of the stage after this one, which is the tile's where the others may be the next tile's)
  const bf16 *abase, *wbase, *abase3;
  auto place = [&](int tm, int tn) {
    const int l = Tiles::kStream ? fresh_lane() : lane;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int row = q < 4 ? wm + q * 32 + (wave & 3) * 8 + (l >> 3) : (q - 4) * 64 + wave * 8 + (l >> 3);
      const int chunk = (l & 7) ^ ((row >> 1) & 7);
      voff[q] = (q < 4 ? (unsigned)min(row, M - 1 - tm) * (unsigned)lda : (unsigned)min(row, N - 1 - tn) * (unsigned)ldw) * 2u + chunk * 16;
    }
    abase = A + (size_t)tm * lda + k_begin;
    wbase = W + (size_t)tn * ldw + k_begin;
  };
  place(m0, n0);
  abase3 = abase;
  voff3 = voff[3];
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(smem));
  const unsigned ldsA = lds0 + (wm + (wave & 3) * 8) * 128, ldsW = lds0 + (256 + wave * 8) * 128;
  auto request = [&](int q, int kt) {
    const unsigned s = (kt & 1) * (E * 2);
    if (q < 4) dma16((q == 3 ? abase3 : abase) + kt * 64, q == 3 ? voff3 : voff[q], ldsA + s + q * 32 * 128);
    else dma16(wbase + kt * 64, voff[q], ldsW + s + (q - 4) * 64 * 128);
  };
#pragma unroll
  for (int q = 4; q < 8; ++q) request(q, 0);
#pragma unroll
  for (int q = 0; q < 4; ++q) request(q, 0);
  if (KT > 1) {
    request(0, 1);
#pragma unroll
    for (int q = 4; q < 8; ++q) request(q, 1);
    request(1, 1);
    request(2, 1);
  }
  hook();
  const int lrow = lane & 31, lhalf = lane >> 5;
  int offA[NS], offB[NS];
#pragma unroll
  for (int ss = 0; ss < NS; ++ss) {
    offA[ss] = lds_off<64>(wm + lrow, ss * 2 + lhalf);
    offB[ss] = 256 * 64 + lds_off<64>(wn + lrow, ss * 2 + lhalf);
  }
  bf16x8 fa[2][NS], fb[NS][TN];
  auto read_a = [&](int kt, int i, int ss) { fa[i & 1][ss] = *reinterpret_cast<const bf16x8*>(smem + (kt & 1) * E + offA[ss] + i * 2048); };
  auto read_b = [&](int kt, int ss, int j) { fb[ss][j] = *reinterpret_cast<const bf16x8*>(smem + (kt & 1) * E + offB[ss] + j * 2048); };
  // MODE 0: a stage with two more behind it, 1: one more, 2: the last
  auto phase = [&](auto I, auto MODE, int kt) {
    constexpr int i = decltype(I)::value, mode = decltype(MODE)::value;
    constexpr bool two = mode == 0;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int ss = s >> 1, j = s & 1;
      acc.c[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[ss][j], fa[i & 1][ss], acc.c[i][j], 0, 0, 0);
      if (i < 3) {
        if (s < 4) read_a(kt, i + 1, s);
      } else if (mode < 2) {
        if (!(s & 1)) read_a(kt + 1, 0, s >> 1);
        else { read_b(kt + 1, ss, 0); read_b(kt + 1, ss, 1); }
      }
      if (s == 3 || s == 5) {
        const int w = s == 5;
        if (i == 0) { if (w == 0 && mode != 2) request(3, kt + 1); if (w == 1 && two) request(0, kt + 2); }
        if (i == 1 && two) request(4 + w, kt + 2);
        if (i == 2 && two) request(6 + w, kt + 2);
        if (i == 3 && two) request(1 + w, kt + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // stored: STORES vector stores went out between the requests of this stage's last pieces and those of the next ones'
  auto stage = [&](auto MODE, int kt, bool stored = false) {
    constexpr int mode = decltype(MODE)::value, ST = Tiles::kStores;
    phase(std::integral_constant<int, 0>{}, MODE, kt);
    phase(std::integral_constant<int, 1>{}, MODE, kt);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (mode == 0 && ST > 0 && stored) wait_vmcnt<6 + ST>();
    else wait_vmcnt<mode == 0 ? 6 : mode == 1 ? 3 : 0>();
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
    phase(std::integral_constant<int, 2>{}, MODE, kt);
    phase(std::integral_constant<int, 3>{}, MODE, kt);
    if (mode != 2) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (mode == 0 && ST > 0 && stored) wait_vmcnt<8 + ST>();
      else wait_vmcnt<mode == 0 ? 8 : 1>();
      block_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto start = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc.c[i][j][r] = 0.f;
#pragma unroll
    for (int ss = 0; ss < NS; ++ss) {
      read_a(0, 0, ss);
      read_b(0, ss, 0);
      read_b(0, ss, 1);
    }
    // (the first requests of the stage go to where these lay)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto settle = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) mfma_settle(acc.c[i][j]);
  };
  constexpr std::integral_constant<int, 0> kGoing{};
  if (KT > 1) wait_vmcnt<8>(); else wait_vmcnt<1>();
  block_barrier();
  start();
  if constexpr (Tiles::kStream) {
    static_assert(8 + Tiles::kStores <= 63, "what a wave counts");
    bool stored = false, more;
    do {
      int m1 = 0, n1 = 0;
      more = tiles.next(m1, n1);
      for (int kt = 0; kt < KT; ++kt) {
        if (kt == KT - 2) {
          place(m1, n1);
          abase -= KT * 64;
          wbase -= KT * 64;
        }
        stage(kGoing, kt, stored);
        abase3 = abase;
        voff3 = voff[3];
        stored = false;
      }
      settle();
      stored = tiles.done();
      abase += KT * 64;
      wbase += KT * 64;
      abase3 = abase;
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (more) start();
    } while (more);
    wait_vmcnt<0>();
  } else {
    int kt = 0;
    for (; kt + 2 < KT; ++kt) stage(kGoing, kt);
    if (kt + 1 < KT) { stage(std::integral_constant<int, 1>{}, kt); ++kt; }
    stage(std::integral_constant<int, 2>{}, kt);
    settle();
    block_barrier();
  }
}
template <class Cfg, bool SWAP = false, class Hook = NoHook>
__device__ __forceinline__ void gemm_mainloop(const bf16* __restrict__ A, int lda,
                                              const bf16* __restrict__ W, int ldw, int M, int N,
                                              int k_begin, int KT, int m0, int n0, bf16* smem,
                                              GemmAcc<Cfg>& acc, Hook hook = Hook()) {
  if constexpr (SWAP && Cfg::kBM == 256 && Cfg::kBN == 256 && Cfg::kStages == 2 && Cfg::kWavesM == 2 && Cfg::kWavesN == 4 && Cfg::GK == 64) {
    gemm_mainloop_square<Cfg>(A, lda, W, ldw, M, N, k_begin, KT, m0, n0, smem, acc, hook);
    return;
  }
  constexpr int IPW = Cfg::kIPW, S = Cfg::kStages, GK = Cfg::GK, RPL = Cfg::kRowsPerLoad, CPR = GK / 8;
  constexpr int TM = Cfg::kTM, TN = Cfg::kTN, NS = GK / 16, TMIN = TM < TN ? TM : TN;
  static_assert(S >= 2 && NS % 2 == 0, "ring depth / fragment buffer parity");
  constexpr bool SPREAD = S >= 3;
  constexpr int PRO = SPREAD ? S - 1 : S;      // stages requested before the loop
  constexpr int AHEAD = PRO;                   // during stage kt the requests of stage kt + AHEAD go out
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / Cfg::kWavesN) * Cfg::kWM, wn = (wave % Cfg::kWavesN) * Cfg::kWN;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc.c[i][j][r] = 0.f;

  // One request moves 64 lanes x 16 B = RPL tile rows; lane l lands at row l/CPR, physical chunk
  // l%CPR, so it fetches the logical chunk that the swizzle maps there.  A lane keeps its byte offsets from the tile's first
  // row; what moves on with the stages is wave-uniform (scalar registers), and so is the place in LDS: per request one scalar
  // move and the load itself.  With full addresses per lane and LDS pointers made uniform at every request, ten instructions
  // more, launches of the encoder and the batch-128 loop took, us: 32768 x 4096 x 1024 on 256 x 256 tiles 276.9, now 266.8; 9216 x
  // 3072 x 1024 on 128 x 128 77.2, now 73.0; 1408 x 4096 x 1024 on 256 x 128 21.0, now 20.2; 64 x 64 tiles 0 - 3 % more.
  unsigned voff[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int r0 = (wave * IPW + i) * RPL, row = r0 + lane / CPR;
    const int chunk = GK == 64 ? ((lane & 7) ^ ((row >> 1) & 7)) : ((lane & 3) ^ ((row >> 2) & 3));
    voff[i] = (r0 < Cfg::kBM ? (unsigned)min(row, M - 1 - m0) * (unsigned)lda : (unsigned)min(row - Cfg::kBM, N - 1 - n0) * (unsigned)ldw) * 2u + chunk * 16;
  }
  const bf16 *abase = A + (size_t)m0 * lda + k_begin, *wbase = W + (size_t)n0 * ldw + k_begin;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(smem)) + wave * (IPW * 1024);
  auto request = [&](int i, int kt, int slot) {
    // (where a wave's requests are all of one operand the choice is made once)
    const int r0 = (wave * IPW + (Cfg::kBM % (IPW * RPL) == 0 ? 0 : i)) * RPL;
    dma16((r0 < Cfg::kBM ? abase : wbase) + kt * GK, voff[i], lds0 + (slot * Cfg::kStageElems + i * 512) * 2);
  };
#pragma unroll
  for (int s = 0; s < PRO; ++s)
    if (s < KT) {
#pragma unroll
      for (int i = 0; i < IPW; ++i) request(i, s, s);
    }
  hook();
  const int lrow = lane & 31, lhalf = lane >> 5;
  int offA[TM][NS], offB[TN][NS];   // fragment offsets inside a stage
#pragma unroll
  for (int ss = 0; ss < NS; ++ss) {
#pragma unroll
    for (int i = 0; i < TM; ++i) offA[i][ss] = lds_off<GK>(wm + i * 32 + lrow, ss * 2 + lhalf);
#pragma unroll
    for (int j = 0; j < TN; ++j) offB[j][ss] = Cfg::kBM * GK + lds_off<GK>(wn + j * 32 + lrow, ss * 2 + lhalf);
  }
  bf16x8 fa[2][TM], fb[2][TN];
  // fragment q of a sub-step in read order a0 b0 a1 b1 ..: the first product of the next sub-step
  // gets its operands first
  auto read_frag = [&](int buf, const bf16* st, int ss, int q) {
    const bool isA = q < 2 * TMIN ? (q & 1) == 0 : TM > TN;
    const int idx = q < 2 * TMIN ? q >> 1 : q - TMIN;
    if (isA) fa[buf][idx] = *reinterpret_cast<const bf16x8*>(st + offA[idx][ss]);
    else fb[buf][idx] = *reinterpret_cast<const bf16x8*>(st + offB[idx][ss]);
  };
  // One sub-step in issue order.  cur: fragment set multiplied now; READ: the fragments of
  // (nst, nss) go to the other set; requests [d0, d1) of stage dkt go to slot dslot.
  auto substep = [&](int cur, bool READ, const bf16* nst, int nss, int dkt, int dslot, int d0, int d1) {
    int nread = 0, nd = d0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc.c[i][j] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][j], fa[cur][i], acc.c[i][j], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc.c[i][j], 0, 0, 0);
        if (READ && nread < TM + TN) read_frag(cur ^ 1, nst, nss, nread++);
        if (((i * TN + j) & 1) && nd < d1) {
          request(nd, dkt, dslot);
          ++nd;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    if (READ) {   // fewer products than fragments
#pragma unroll
      for (; nread < TM + TN; ++nread) read_frag(cur ^ 1, nst, nss, nread);
    }
#pragma unroll
    for (; nd < d1; ++nd) request(nd, dkt, dslot);
  };
  // stage 0 has landed for everyone
  wait_vm_stages<IPW, PRO - 1>(min(PRO, KT) - 1);
  block_barrier();
#pragma unroll
  for (int q = 0; q < TM + TN; ++q) read_frag(0, smem, 0, q);
  constexpr int LASTBUF = (NS - 1) & 1;
  int kt = 0;
  // stages during which another stage is still to be requested
  for (; kt + AHEAD < KT; ++kt) {
    const bf16* st = smem + (kt % S) * Cfg::kStageElems;
    const int nslot = (kt + AHEAD) % S;
#pragma unroll
    for (int ss = 0; ss + 1 < NS; ++ss)
      substep(ss & 1, true, st, ss + 1, kt + AHEAD, nslot, SPREAD ? ss * IPW / NS : 0, SPREAD ? (ss + 1) * IPW / NS : 0);
    // my reads of this stage are done (its slot may be refilled after the barrier), my part of
    // stage kt+1 has landed (younger requests may still be in flight)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait_vmcnt<SPREAD ? IPW * (S - 3) + (NS - 1) * IPW / NS : IPW * (S - 2)>();
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
    substep(LASTBUF, true, smem + ((kt + 1) % S) * Cfg::kStageElems, 0, kt + AHEAD, nslot,
            SPREAD ? (NS - 1) * IPW / NS : 0, IPW);
  }
  // the last stages: nothing left to request
  for (; kt + 1 < KT; ++kt) {
    const bf16* st = smem + (kt % S) * Cfg::kStageElems;
#pragma unroll
    for (int ss = 0; ss + 1 < NS; ++ss) substep(ss & 1, true, st, ss + 1, 0, 0, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait_vm_stages<IPW, AHEAD - 2>(KT - kt - 2);
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
    substep(LASTBUF, true, smem + ((kt + 1) % S) * Cfg::kStageElems, 0, 0, 0, 0, 0);
  }
  {
    const bf16* st = smem + (kt % S) * Cfg::kStageElems;
#pragma unroll
    for (int ss = 0; ss + 1 < NS; ++ss) substep(ss & 1, true, st, ss + 1, 0, 0, 0, 0);
    substep(LASTBUF, false, st, 0, 0, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) mfma_settle(acc.c[i][j]);
  block_barrier();   // LDS may be reused by the caller's epilogue
}

// Visits every output element the calling lane holds: f(m, n, value).
// MFMA 32x32 result layout: register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, col l%32.
template <class Cfg, class F>
__device__ __forceinline__ void gemm_foreach(const GemmAcc<Cfg>& acc, int m0, int n0, F&& f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave / Cfg::kWavesN) * Cfg::kWM, wn = (wave % Cfg::kWavesN) * Cfg::kWN;
#pragma unroll
  for (int i = 0; i < Cfg::kTM; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::kTN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int m = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        int n = n0 + wn + j * 32 + (lane & 31);
        f(m, n, acc.c[i][j][r]);
      }
}

}  // namespace sd
