// The decoder layers of a pass of few rows as ONE kernel, each XCD on sequences of its own.
//
// With few rows a decoder layer is eight dependent products and attentions of a microsecond each, and as separate kernels
// every hand-over costs a launch (about 4 us from one kernel's operands to the next one's).  Here 32 workgroups on the 32 CUs
// of an XCD stay resident for all layers and carry up to 96 rows (d = 512: 160; whole sequences, dealt over the XCDs; sequences do not meet)
// through them.  A product's columns are dealt over the 32 workgroups, whose eight computing waves split K.  What one workgroup
// produces for another goes to an exchange buffer that holds kPoison in every 32-bit word beforehand; the consumers load the
// words they need past their L1, straight into MFMA operand registers, until none of them is kPoison any more.  The value is
// its own flag: a hand-over is one store to and one load from the XCD's own L2, with no barrier, no counter and no fence.
// Measured with nothing else in between: 0.38 us among the 32 workgroups of an XCD; through memory, among workgroups spread
// over the chip, 0.97 (32 of them), 1.27 (128) and 1.85 us (256).  No word of a result is ever stored as kPoison
// (not_poison).
//
// Weights: every XCD reads all of them.  Every wave has its share in one piece, in the order it is used (laid out when the model is bound,
// xcd_pack), and requests it ahead through a ring in LDS of its own.  A CU's loads return in the order they were requested,
// whichever wave did, so a poll behind weights waits for them (1.1 - 1.5 us while an XCD takes in all it can, 0.9 TB/s where all
// eight do so and 1.3 TB/s where one does): what a product has used is therefore requested anew when its rows are there, not
// while they are waited for.  (In waves of their own, the requests held up the barriers instead: a verify pass of 352 rows of d = 512
// took 244 us so, 227 without them.)
//
// A pass of at most 63 rows of d = 512 needs no such copy: it reads the matrices as bound, a chunk of 16 rows x 128 bytes at a time (DIRECT;
// 113.6 us for 6 rows, from a copy 112.7).
//
// A drafter's pass of at least 200 drafts (d = 512; stream rows and slots of as many places a sequence as it can need) is one of these, its matrices read in place whatever
// its rows (fewer drafts are launches, see draft_way).  Passes behind a loaded cache, statistics read back, launches / this kernel, us: 32 x 11
// 124 / 83, on 500 source tokens and 200 cached ones 133 / 100, 64 x 8 123 / 96.  An iteration of the loop with a base verifier, 24 x 11 (504 places
// for the drafter, some 340 in use) 291 / 261.
//
// More than four row tiles (65 rows and more of an XCD; one column tile is summed at a time and, where LDS has no room for its row tiles, these in two
// parts; of d = 512 the matrices are read in place): a tile more costs 0.4 us a stage where the launches of a pass beyond 512 rows cost 6 each.
// Whole passes, launches / this kernel, us: verification, d = 512: 48 x 11 rows 337 / 241, 64 x 11 350 / 267, 80 x 11 368 / 309, 96 x 11 421 / 360, 112 x
// 11 441 / 436 (eleven tiles, 128 x 11: 471 / 496), on 250 source tokens 128 x 9 565 / 483; d = 1024: 48 x 11 560 / 506, 64 x 11 589 / 555, on 512
// source tokens 753 / 724; drafting 48 x 11 133 / 105, 64 x 11 150 / 126, 80 x 11 157 / 141.
//
// A prefill pass is one of these as well (all of its rows see the keys up to their own); it ends where the last layer's keys and values are stored.
//
// What bounds it: a hand-over and instructions in a row at every stage (of 11 rows 0.8 - 3.5 us, of 44 1.8 - 3.9), and with the weights of d =
// 1024 what an XCD takes in.  Whole verify passes, launches / this kernel, us: d = 512: 6 rows 200 / 109, 77 239 / 121, 176 255 / 140, 352
// 287 / 168; d = 1024: 6 rows 252 / 217, 128 366 / 335, 176 358 / 317, 352 462 / 363.  (Which passes it takes, and what the kernel over the whole GPU
// (persist.hip) takes for them, is in api.hip.)
//
// LayerNorm is folded into the products as in the general kernels (gemm.hip), with statistics per 16 columns; the fp32 residual
// of a workgroup's columns stays in its LDS.  The exchange buffers of two layers are used in turn.  Those of layer l - 1 are
// filled with kPoison again once the output product of layer l's self-attention has all its rows: every workgroup has then
// stored its queries, keys and values of layer l, after the last it read of layer l - 1 (the units of a sequence's eight heads wait for all
// columns of one key and value of the pass at least: of a sequence without rows, which a prefill pass may have, those of its first place, which
// nothing else needs; before, a group of such sequences alone left the workgroups behind that make keys and values alone, and one of them
// could find what it was still to read filled again); and whoever waits for a word of
// layer l + 1 has had rows of layer l from every workgroup, stored after the refill was acknowledged.  The pass's first kernel fills both layers'; of
// more than 64 rows of a group the first layer's alone, the other half in the first layer as in later ones (d = 1024, launches / both / one: 48 x 11
// rows 560 / 506 / 490, 64 x 11 589 / 555 / 541; 6 rows of d = 512 both 110.4, one 111.3).
//
// The workgroups of an XCD wait for each other, so all of them have to be running.  There is one for every CU of the GPU and
// the host lets one such pass at a time onto a GPU, but a kernel of another stream or process may hold some of the CUs.  Waits
// are therefore bounded: after kPlSpinMax polls, or once another workgroup has raised the error flag, a wave raises it and ends,
// and the pass is computed again by the kernel launched behind this one (TICKETS), which returns at once where the flag is
// not raised.  Its workgroups draw (stage, group, member) tickets in the order of the stages, as in persist.hip, and wait only for stages whose
// tickets have all been drawn, that is for workgroups that are running: it needs no more than one CU.  It computes the same bits.
// Whole passes so: one sentence of d = 512 0.44 ms, 8 x 7 rows 2.1, 352 rows 2.1, of d = 1024 2.8.  (By one workgroup a group, its 32 members one after
// the other, 6.6, 6.6, 6.9 and 12.6.)  The flag counts the passes that go to it directly (kPlTicketPasses, this one included) before one waits
// again.  A whole verify pass with the second launch returning at once and without it: 105.8 / 104.5 us (d = 512, 6 rows), 123.3 / 121.8 (77), 171.9 /
// 170.9 (352), 373.2 / 372.2 (d = 1024, 352 rows).
// (A workgroup takes the XCD it finds itself on for its group and the eighth of its number for its place there, as ids are dealt to
// the XCDs in turn.  Were they dealt otherwise, a place would be missing or taken twice: the same words written twice, or waits
// given up.)
#pragma once
#include <algorithm>

#include "gemm_core.h"
#include "resident_core.h"

namespace sd {
namespace xcd {

constexpr unsigned kPlSpinMax = 3u << 18;   // (0.13 - 0.3 s: 2^17 polls of the L2 take 21 - 49 ms)
constexpr int kPlMembers = 32;          // workgroups of each XCD
constexpr int kPlWaves = 8, kPlThreads = 64 * kPlWaves;
static_assert(kPlGroups * kPlMembers == kPlBlocks && kPlWaves == 8, "a workgroup per CU; pairs of a row's four lanes");
// (a word of each 8 bytes: results are stored 8 bytes at a time)
__device__ __forceinline__ bool pl_missing(const u32x4& v) { return v[1] == kPoison || v[3] == kPoison; }
__device__ __forceinline__ void pl_store8(void* p, unsigned a, unsigned b) {
  u32x2 v = {not_poison(a), not_poison(b)};
  asm volatile("global_store_dwordx2 %0, %1, off sc0" ::"v"(p), "v"(v) : "memory");
}
// One more round of a wait; ends the wave once the pass is to be abandoned.  (The end of the wave, not a result that every caller
// hands on: with one, the rows a wave holds were copied at every join of the ways, and spilled.  And as an instruction like any other: the
// builtin is an end of the program's ways, and the others then came with a dozen flags at every wait.)
__device__ __forceinline__ void pl_again(unsigned& spins, const XcdArgs& a) {
  ++spins;
  if ((spins & 63u) == 0) {
    // (the same for the whole wave, and said so: no wait is a loop of single lanes)
    const unsigned raised = __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (raised != 0u || spins > kPlSpinMax) {
      __hip_atomic_store(a.err, kPlTicketPasses, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // (weights on their way to LDS: it may be another workgroup's next)
      asm volatile("s_waitcnt vmcnt(0)\n\ts_endpgm" ::: "memory");
    }
  }
  __builtin_amdgcn_s_sleep(1);
  asm volatile("" ::: "memory");
}

// What depends on the dimensions and the type of the weights alone.  A chunk of weights: 16 rows (output columns) x an eighth of D of K,
// as MFMA fragments: [K / 32][lane][8 values], lane = row + 16 (K / 8 % 4).
template <int D>
struct PlDim {
  static constexpr int KW = D / kPlWaves, KS = KW / 32, kChunk = 32 * KW, kReq = kChunk / 1024;
  static constexpr int kRing = D == 512 ? 5 : 3;   // (what LDS has room for)
  static_assert(kReq >= 1 && kRing * kReq <= 56, "whole requests, as many as a wave can have in flight");
  // columns and column tiles of a workgroup: QKV, the square ones, first FFN matrix; chunks of K of the second; all chunks of a layer
  static constexpr int kNQ = 3 * D / kPlMembers, kND = D / kPlMembers, kNF = 4 * D / kPlMembers;
  static constexpr int kTQ = kNQ / 16, kTD = kND / 16, kTF = kNF / 16, kKC = 4, kPerLayer = kTQ + 3 * kTD + kTF + kKC * kTD;
  // Chunks requested in stage s.  Rows are waited for behind what a CU has requested before (0.6 us a chunk of d = 512), so where the ring holds
  // more than a stage's chunks they are spread over the stages, attention among them, as far as the ring goes: with as many requested as a
  // stage had used, three or four at a time, a verify pass of 77 rows took 130.0 us, so 125.2; 352 rows 175.0 / 173.5.
  static constexpr int kAsk[8] = {D == 512 ? 2 : kTQ, D == 512 ? 2 : 0, kTD, kTD, D == 512 ? 1 : 0, kTD, D == 512 ? 3 : kTF, D == 512 ? 3 : kTD * kKC};
  static constexpr int kAskFirst = D == 512 ? kTQ : kRing;   // ahead of the first
  // column vectors of a layer, floats: cs and bf of the three projections, three of each sum
  static constexpr int kVecQ = 0, kVecC = 2 * kNQ, kVecF = kVecC + 2 * kND, kVecS = kVecF + 2 * kNF;
  static constexpr int kVecs = kVecS + 9 * kND, kVecReq = (kVecs / 4 + 63) / 64, kVecPitch = kVecReq * 256;   // requests of 64 x 16 bytes
};

// A sequence of the group: the position of its first row, rows that see the keys up to their own, rows of the pass (see pl_attn_wave), source.
struct alignas(16) PlSeq { int j, causal, live, src_len; };

template <int D, int MR>
struct PlLds {
  typedef PlDim<D> Dim;
  // column tiles summed together: as many as their partial tiles have room for, and as leave some of the ring
  static constexpr int kBatch = D == 1024 || MR > 4 ? 1 : MR <= 2 ? 4 : 2;
  // row tiles summed together, and tiles there is room for
  static constexpr int kSub = D == 1024 ? (MR <= 4 ? MR : 3) : MR <= 7 ? MR : MR == 8 ? 4 : 5;
  static constexpr int kRedTiles = D == 1024 || kSub < MR ? (kSub > 4 ? kSub : 4) : MR > 4 ? MR : 8;
  static constexpr int kFlips = 2 * kBatch * kSub <= kRedTiles ? 2 : 1;
  char ring[kPlWaves][Dim::kRing * Dim::kChunk];
  f32x4 red[kPlWaves * kRedTiles * 64];           // partial tiles, kFlips sets; attention: value tiles of the waves ([32 keys][64],
                                                  // swizzled like the tile kernel's), then partial results, 4 KB a wave either way
  float vec[2][Dim::kVecPitch];                   // column vectors, layers in turn
  float ml[kPlWaves * 32];
  float resid[Dim::kTD * 16 * MR * 16];           // of the workgroup's columns
  float stat[2][2 * 16 * MR];                     // {rstd, -mean rstd} of the rows, LayerNorms in turn
  float part[kPlWaves][2 * 16 * MR];              // {sum, squared deviations from its mean} of a row's columns, an eighth of them a wave
  PlSeq seq[16 * MR];
  int row_at[16 * MR];                            // of the row in the self-attention cache of head 0 (< 0: none)
  int drawn;                                      // (TICKETS)
  __device__ __forceinline__ bf16* vs(int wave) { return reinterpret_cast<bf16*>(red + wave * 256); }
  // Where units of attention can form their queries (see PlOwnQueries): these, behind the first 32 KB of red.
  static constexpr bool kForm = D == 512 && MR <= 2;
  __device__ __forceinline__ bf16* queries() { static_assert(!kForm || kRedTiles == 8, "64 KB"); return reinterpret_cast<bf16*>(red + 2048); }
};

// A workgroup's place: group g carries sequences b0 .. b0 + nb - 1, rows row0 .. row0 + rows - 1 of the pass.
struct PlPlace { int g, w, b0, nb, row0, rows; };
__device__ __forceinline__ PlPlace pl_place(const XcdArgs& a, int g, int w) {
  const int n = a.B / a.G, more = a.B - n * a.G;
  PlPlace p{g, w, g * n + min(g, more), n + (g < more ? 1 : 0), 0, 0};
  p.row0 = p.b0 * a.T;
  p.rows = p.nb * a.T;
  return p;
}

// Stages of a layer: 0 queries, keys, values; 1 self-attention; 2 its output sum; 3 cross-attention queries; 4 cross-attention;
// 5 its output sum; 6 first FFN matrix; 7 second, sum.
template <class Dim>
__device__ __forceinline__ int pl_chunks(int s) {
  return s == 0 ? Dim::kTQ : s == 6 ? Dim::kTF : s == 7 ? Dim::kTD * Dim::kKC : s == 1 || s == 4 ? 0 : Dim::kTD;
}
// Attention of a group: waves of a unit (XcdArgs::wpu), units of a workgroup at a time, rounds.
__device__ __forceinline__ int pl_units(const XcdArgs& a, const PlPlace& p) { return p.nb * a.H * ((a.T + 15) >> 4); }
__device__ __forceinline__ int pl_rounds(const XcdArgs& a, const PlPlace& p) {
  const int per = kPlMembers * (kPlWaves / a.wpu);
  return (pl_units(a, p) + per - 1) / per;
}

// What a wave carries along: its stream of weights (the next chunk to request, how many are left, where it goes in the ring, where the
// next one to use lies) and the sums so far.  Where the weights are read in place (XcdArgs::stream null), at[]: the matrices of which this
// stage requests chunks.
struct PlTurn { const char* next; int left, slot, use, sums, w; const char* at[2]; };
__device__ __forceinline__ unsigned pl_lds_addr(const void* p) {
  return __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)SD_LDS_PTR(const_cast<void*>(p)));
}
// 1 KB from base + OFF + voff (16 bytes a lane) to LDS at lds + OFF: the instruction's offset counts on both sides
template <int OFF>
__device__ __forceinline__ void pl_dma(const char* base, unsigned voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"s"(lds), "v"(voff), "s"(base), "n"(OFF) : "memory");
}
// a wave's stream from chunk c of layer l on, n chunks
template <int D>
__device__ __forceinline__ PlTurn pl_turn(const XcdArgs& a, int w, int wave, int l, int c, int n) {
  typedef PlDim<D> Dim;
  return PlTurn{a.stream + ((size_t)((w * kPlWaves + wave) * a.n_layers + l) * Dim::kPerLayer + c) * Dim::kChunk, n, 0, 0, 0, w, {nullptr, nullptr}};
}
// One chunk of a matrix [columns][K] as it is bound: 16 rows of 128 bytes from `from` on (a workgroup's waves read whole rows), two requests of 8 whole
// lines.  In the ring 16-byte piece c of row r lies at r * 128 + 16 (c ^ (r / 2 % 8)): 16 rows' same piece meets all banks once.  (As fragments,
// like a chunk of the copy, a request touches half of each of 16 lines: a pass of 6 rows 122.0 us, so 113.6; from a copy in order of use 112.7.)
template <int D, int MR>
__device__ __forceinline__ void pl_request_rows(PlLds<D, MR>& L, PlTurn& t, int wave, const char* from, int pitch) {
  typedef PlDim<D> Dim;
  static_assert(D != 512 || (Dim::KW == 64 && Dim::kReq == 2), "rows of a line");
  const int lane = pl_lane();
  const unsigned to = pl_lds_addr(L.ring) + wave * (Dim::kRing * Dim::kChunk) + t.slot, voff = (lane >> 3) * pitch + (((lane & 7) ^ (lane >> 4)) << 4);
  pl_dma<0>(from, voff, to);
  pl_dma<0>(from + 8 * pitch, voff ^ 64, to + 1024);
  t.slot = t.slot + Dim::kChunk == Dim::kRing * Dim::kChunk ? 0 : t.slot + Dim::kChunk;
  --t.left;
}
// where workgroup w's first chunk of a matrix lies: of one with N column tiles a workgroup, K = KC * D
template <int D>
__device__ __forceinline__ const char* pl_rows_at(const void* W, int w, int wave, int N, int KC) {
  return static_cast<const char*>(W) + (size_t)w * N * (16 * KC * D * 2) + wave * (PlDim<D>::KW * 2);
}
// A layer's pointers, for scalar loads (nothing writes them while the kernel runs).
typedef const __attribute__((address_space(4))) PlLayer* PlLayerPtr;
__device__ __forceinline__ PlLayerPtr pl_layer(const XcdArgs& a, int l) { return (PlLayerPtr)(uintptr_t)(a.layers + l); }
// Requests chunks c .. c + n - 1 of layer l (as many as are left).
template <int D, int MR>
__device__ __forceinline__ void pl_ask_rows(const XcdArgs& a, PlLds<D, MR>& L, PlTurn& t, int wave, int l, int c, int n) {
  typedef PlDim<D> Dim;
  constexpr int kPitch = D * 2;
  static_assert(Dim::kTD == 1 || D != 512, "one chunk a square matrix");
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the fragments read from the places that are filled again)
  const PlLayerPtr Y = pl_layer(a, l);
  for (int e = c + min(n, t.left); c < e; ++c) {
    const int f = c - (Dim::kTQ + 3), k = f - Dim::kTF;
    if (c < Dim::kTQ) pl_request_rows(L, t, wave, pl_rows_at<D>(Y->wqkv.p, t.w, wave, Dim::kTQ, 1) + c * 16 * kPitch, kPitch);
    else if (f < 0) pl_request_rows(L, t, wave, pl_rows_at<D>(f == -3 ? Y->wo.p : f == -2 ? Y->cwq.p : Y->cwo.p, t.w, wave, 1, 1), kPitch);
    else if (k < 0) pl_request_rows(L, t, wave, pl_rows_at<D>(Y->w1.p, t.w, wave, Dim::kTF, 1) + f * 16 * kPitch, kPitch);
    else pl_request_rows(L, t, wave, pl_rows_at<D>(Y->w2.p, t.w, wave, 1, Dim::kKC) + k * kPitch, Dim::kKC * kPitch);
  }
}
// The matrices of which stage S of layer l requests chunks (PlDim::kAsk; the last requests the next layer's): as they are bound, so that nothing
// waits for them before they are used.
template <int D, int S>
__device__ __forceinline__ void pl_ask_at(const XcdArgs& a, PlTurn& t, int l) {
  const PlLayerPtr Y = pl_layer(a, S == 7 ? min(l + 1, a.n_layers - 1) : l);
  auto set = [&](int i, const void* W) { t.at[i] = static_cast<const char*>(W); };
  if (S == 0) { set(0, Y->wo.p); set(1, Y->cwq.p); }
  if (S == 1) { set(0, Y->cwo.p); set(1, Y->w1.p); }
  if (S >= 2 && S <= 4) set(0, Y->w1.p);
  if (S == 5 || S == 6) set(0, Y->w2.p);
  if (S == 7) set(0, Y->wqkv.p);
}
// Requests the next n chunks there are.
template <int D, int MR>
__device__ __forceinline__ void pl_ask_next(PlLds<D, MR>& L, PlTurn& t, int wave, int n) {
  typedef PlDim<D> Dim;
  const unsigned ring = pl_lds_addr(L.ring) + wave * (Dim::kRing * Dim::kChunk), voff = pl_lane() * 16;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (as above)
  for (int i = min(n, t.left); i > 0; --i) {
    pl_dma<0>(t.next, voff, ring + t.slot);
    if constexpr (Dim::kReq > 1) pl_dma<1024>(t.next, voff, ring + t.slot);
    if constexpr (Dim::kReq > 2) {
      pl_dma<2048>(t.next, voff, ring + t.slot);
      pl_dma<3072>(t.next, voff, ring + t.slot);
    }
    static_assert(Dim::kReq <= 2 || Dim::kReq == 4, "requests of a chunk");
    t.next += Dim::kChunk;
    t.slot = t.slot + Dim::kChunk == Dim::kRing * Dim::kChunk ? 0 : t.slot + Dim::kChunk;
    --t.left;
  }
}
// Requests number FIRST .. FIRST + N - 1 of stage S.
template <int D, int MR, int S, int FIRST, int N>
__device__ __forceinline__ void pl_ask(const XcdArgs& a, PlLds<D, MR>& L, PlTurn& t, int wave) {
  if (D != 512 || a.stream) return pl_ask_next(L, t, wave, N);
  if (N == 0 || t.left == 0) return;
  constexpr int kRows = 16 * D * 2;   // to a matrix's next column tile
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = FIRST; i < FIRST + N; ++i) {
    typedef PlDim<D> Dim;
    const char* W = t.at[S <= 1 ? i : 0];
    if (S == 0 || (S == 1 && i == 0)) pl_request_rows(L, t, wave, pl_rows_at<D>(W, t.w, wave, 1, 1), D * 2);
    else if (S <= 4) pl_request_rows(L, t, wave, pl_rows_at<D>(W, t.w, wave, Dim::kTF, 1) + (S - 1) * kRows, D * 2);
    else if (S <= 6) pl_request_rows(L, t, wave, pl_rows_at<D>(W, t.w, wave, 1, Dim::kKC) + (S == 5 ? 0 : 1 + i) * (D * 2), Dim::kKC * D * 2);
    else pl_request_rows(L, t, wave, pl_rows_at<D>(W, t.w, wave, Dim::kTQ, 1) + i * kRows, D * 2);
  }
}
// Requests the column vectors of layer l (a request each of the first waves).
template <int D, int MR>
__device__ __forceinline__ void pl_ask_vectors(const XcdArgs& a, PlLds<D, MR>& L, int l, int w, int wave) {
  typedef PlDim<D> Dim;
  static_assert(Dim::kVecReq <= kPlWaves, "a request a wave");
  if (wave < Dim::kVecReq)
    pl_dma<0>(reinterpret_cast<const char*>(a.vecs + (size_t)(l * kPlMembers + w) * Dim::kVecPitch + wave * 256), pl_lane() * 16,
              pl_lds_addr(L.vec) + (l & 1) * (Dim::kVecPitch * 4) + wave * 1024);
}

// The fragments of the next chunk, once it is there.  AHEAD: chunks that may have been requested after it
// (< 0: it was requested before rows that have arrived).
template <int D, int MR, int AHEAD>
__device__ __forceinline__ void pl_weights(const XcdArgs& a, PlLds<D, MR>& L, PlTurn& t, int wave, int lane, bf16x8 (&wf)[PlDim<D>::KS]) {
  typedef PlDim<D> Dim;
  if constexpr (AHEAD >= 0) {   // (what else is in flight only makes this stricter)
    if (t.left > 0) wait_vmcnt<AHEAD * Dim::kReq>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
  }
  const char* c = L.ring[wave] + t.use;
  if (D != 512 || a.stream) {
#pragma unroll
    for (int u = 0; u < Dim::KS; ++u) wf[u] = *reinterpret_cast<const bf16x8*>(c + lane * 16 + u * 1024);
  } else {   // (see pl_request_rows)
    const int lq = lane & 15, o = lq * 128 + (((lane >> 4) ^ (lq >> 1)) << 4);
#pragma unroll
    for (int u = 0; u < Dim::KS; ++u) wf[u] = *reinterpret_cast<const bf16x8*>(c + (o ^ (u * 64)));
  }
  t.use = t.use + Dim::kChunk == Dim::kRing * Dim::kChunk ? 0 : t.use + Dim::kChunk;
}

// Rows of a group as MFMA operands: af[mr][u] = row 16 mr + lq, columns kc * D + this wave's share of D.
template <int D, int MR>
struct PlRows {
  static constexpr int KW = D / kPlWaves, KS = KW / 32, NS = D / 512;
  const XcdArgs& a;
  const char* A;
  bool plain;     // rows another kernel wrote, [R][D]
  int rows, lane, wave;
  PlBuf buf;
  __device__ __forceinline__ PlRows(const XcdArgs& a_, const char* A_, bool plain_, int rows_, int lane_, int wave_)
      : a(a_), A(A_), plain(plain_), rows(rows_), lane(lane_), wave(wave_), buf(pl_buf(A_)) {}
  __device__ __forceinline__ void request(int mr, int kc, u32x4 (&af)[MR][KS]) const {
    const int lq = lane & 15, g = lane >> 4, row = min(16 * mr + lq, rows - 1), k = kc * D + wave * KW + 8 * g;
    if (plain) {
#pragma unroll
      for (int u = 0; u < KS; ++u) af[mr][u] = *reinterpret_cast<const u32x4*>(A + ((size_t)row * D + k + u * 32) * 2);
    } else {
      const int off = pl_at(a.RP, row, k);
#pragma unroll
      for (int u = 0; u < KS; ++u) af[mr][u] = pl_request(buf, off, u * a.RP * 64);
    }
  }
  // (rows beyond the group's are its last one again)
  __device__ __forceinline__ bool missing(int mr, const u32x4 (&af)[MR][KS]) const {
    unsigned m = 0u;
#pragma unroll
    for (int u = 0; u < KS; ++u) m = max(m, max(af[mr][u][1], af[mr][u][3]));
    return __builtin_amdgcn_ballot_w64(m == kPoison) != 0;
  }
  struct NoStats {
    __device__ __forceinline__ void request() const {}
    __device__ __forceinline__ bool missing() const { return false; }
  };
  struct LateStats {   // chunks NS (4 wave + g) .. of the row, as new as the rows
    const PlRows& R;
    PlBuf sb;
    u32x2 (&st)[MR][NS];
    __device__ __forceinline__ void request() const {
#pragma unroll
      for (int mr = 0; mr < MR; ++mr)
#pragma unroll
        for (int i = 0; i < NS; ++i)
          st[mr][i] = __builtin_amdgcn_raw_buffer_load_b64(sb, (NS * (4 * R.wave + (R.lane >> 4)) * R.a.RP + min(16 * mr + (R.lane & 15), R.rows - 1)) * 8,
                                                           i * R.a.RP * 8, kPlSc1);
    }
    __device__ __forceinline__ bool missing() const {
      unsigned m = 0u;
#pragma unroll
      for (int mr = 0; mr < MR; ++mr)
#pragma unroll
        for (int i = 0; i < NS; ++i) m = max(m, st[mr][i][1]);
      return __builtin_amdgcn_ballot_w64(m == kPoison) != 0;
    }
  };
  // Requested before: what is not there yet, again, all of it at once.  (A tile after the other, and the statistics behind them, one more round
  // trip of 0.4 us each: verify pass of 352 rows of d = 512 186.7 us, so 175.0; 209 rows of d = 1024 403 / 393.)
  template <class Stats = NoStats>
  __device__ __forceinline__ void arrive(u32x4 (&af)[MR][KS], Stats stats = Stats()) const {
    if constexpr (MR * KS > 12) {   // (held twice over at the loop's end, such rows do not fit the registers)
      arrive_later(0, af);
      for (unsigned spins = 0; stats.missing(); stats.request()) pl_again(spins, a);
      return;
    }
    unsigned spins = 0;
    while (true) {
      bool miss[MR], late = stats.missing(), any = late;
#pragma unroll
      for (int mr = 0; mr < MR; ++mr) {
        miss[mr] = missing(mr, af);
        any |= miss[mr];
      }
      if (!any) break;
      pl_again(spins, a);
#pragma unroll
      for (int mr = 0; mr < MR; ++mr)
        if (miss[mr]) request(mr, 0, af);
      if (late) stats.request();
    }
  }
  // the same of later columns, a tile after the other (two sets of rows are held)
  __device__ __forceinline__ void arrive_later(int kc, u32x4 (&af)[MR][KS]) const {
    unsigned spins = 0;
#pragma unroll
    for (int mr = 0; mr < MR; ++mr)
      while (missing(mr, af)) {
        pl_again(spins, a);
        request(mr, kc, af);
      }
  }
  // All columns of a few rows, KC sets of them.
  template <int KC>
  __device__ __forceinline__ void all(u32x4 (&af)[KC][MR][KS]) const {
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int mr = 0; mr < MR; ++mr) request(mr, kc, af[kc]);
    unsigned spins = 0;
    while (true) {
      bool miss[KC], any = false;
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        miss[kc] = false;
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) miss[kc] |= missing(mr, af[kc]);
        any |= miss[kc];
      }
      if (!any) break;
      pl_again(spins, a);
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)
        if (miss[kc]) {
#pragma unroll
          for (int mr = 0; mr < MR; ++mr) request(mr, kc, af[kc]);
        }
    }
  }
  // All row tiles of the first D columns; with them (stats not null) the statistics of the same columns, merged into one pair a row
  // (part).  What has been requested of the weights is there, too.
  __device__ __forceinline__ void first(u32x4 (&af)[MR][KS], const char* stats, float* part) const {
#pragma unroll
    for (int mr = 0; mr < MR; ++mr) request(mr, 0, af);
    if (plain) {
      wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      return;
    }
    if (stats) {
      const int lq = lane & 15, g = lane >> 4;
      u32x2 st[MR][NS];
      const LateStats late{*this, pl_buf(stats), st};
      late.request();
      arrive(af, late);
      merge(st, lq, g, part);
    } else {
      arrive(af);
    }
  }
  static __device__ __forceinline__ void merge(const u32x2 (&st)[MR][NS], int lq, int g, float* part) {
#pragma unroll
    for (int mr = 0; mr < MR; ++mr) {
      f32x2 p[NS];
      float s = 0.f, q = 0.f;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        p[i] = __builtin_bit_cast(f32x2, st[mr][i]);
        s += p[i][0];
      }
      s = pl_row_sum(s);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const float dv = (p[i][0] - s * (16.f / KW)) * (1.f / 16);
        q += __builtin_fmaf(16.f * dv, dv, p[i][1]);
      }
      q = pl_row_sum(q);
      if (g == 0) *reinterpret_cast<f32x2*>(part + 2 * (16 * mr + lq)) = f32x2{s, q};
    }
  }
  // The statistics alone.
  __device__ __forceinline__ void statistics(const char* stats, float* part) const {
    u32x2 st[MR][NS];
    const LateStats late{*this, pl_buf(stats), st};
    late.request();
    for (unsigned spins = 0; late.missing(); late.request()) pl_again(spins, a);
    merge(st, lane & 15, lane >> 4, part);
  }
};
// {rstd, -mean rstd} of row 16 mr + lq from the waves' pairs, two of them a lane of the row's four
template <int D>
__device__ __forceinline__ f32x2 pl_row_stat(const float* part, int pitch, int row, int g) {
  f32x2 p[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) p[i] = *reinterpret_cast<const f32x2*>(part + (2 * g + i) * pitch + 2 * row);
  const float mean = pl_row_sum(p[0][0] + p[1][0]) * (1.f / D);
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float dv = p[i][0] * ((float)kPlWaves / D) - mean;
    q += __builtin_fmaf((float)(D / kPlWaves) * dv, dv, p[i][1]);
  }
  const float rstd = fast_rsqrt(pl_row_sum(q) * (1.f / D) + 1e-5f);
  return f32x2{rstd, -mean * rstd};
}

// The partial tiles of NT column tiles: stored, met at the barrier, summed in wave order, each by one wave (not the ones that
// summed last where there are enough).  There pre(i, mr) reads what the epilogue needs ahead of the barrier and done(i, mr, v, pre's)
// finishes: row 16 mr + lq, columns 4 g .. + 3 of tile i.
template <int D, int MR, int NT, int M0, int MS, class Pre, class Done>
__device__ __forceinline__ void pl_reduce_some(PlLds<D, MR>& L, PlTurn& t, int wave, int lane, f32x4 (&acc)[NT][MR], Pre&& pre, Done&& done) {
  constexpr int P = NT * MS;
  static_assert(PlLds<D, MR>::kFlips * P <= PlLds<D, MR>::kRedTiles && P <= kPlWaves, "room for the partial tiles");
  f32x4* red = L.red;
  if (PlLds<D, MR>::kFlips == 1) lds_barrier();   // the tiles before have been summed
  else red += (t.sums & 1) * (kPlWaves * PlLds<D, MR>::kRedTiles / 2 * 64);
  const int p = P <= 4 ? (wave + 4 * t.sums) & (kPlWaves - 1) : wave, q0 = min(p, P - 1);
  ++t.sums;
  const auto have = pre(q0 / MS, M0 + q0 % MS);
  asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[NT - 1][MR - 1]));   // (the last of the products; see mfma_settle)
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int mr = 0; mr < MS; ++mr) {
      asm volatile("" : "+v"(acc[i][M0 + mr]));   // (not ahead of it)
      red[((i * MS + mr) * kPlWaves + wave) * 64 + lane] = acc[i][M0 + mr];
    }
  lds_barrier();
  if (p >= P) return;
  f32x4 q[kPlWaves], v;
#pragma unroll
  for (int w = 0; w < kPlWaves; ++w) q[w] = red[(p * kPlWaves + w) * 64 + lane];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = q[0][e];
#pragma unroll
    for (int w = 1; w < kPlWaves; ++w) v[e] += q[w][e];
  }
  done(p / MS, M0 + p % MS, v, have);
}
// (row tiles a few at a time, where the partial tiles of all have no room)
template <int D, int MR, int NT, class Pre, class Done>
__device__ __forceinline__ void pl_reduce(PlLds<D, MR>& L, PlTurn& t, int wave, int lane, f32x4 (&acc)[NT][MR], Pre&& pre, Done&& done) {
  constexpr int SUB = PlLds<D, MR>::kSub;
  static_assert(MR <= 2 * SUB, "twice at most");
  pl_reduce_some<D, MR, NT, 0, SUB>(L, t, wave, lane, acc, pre, done);
  if constexpr (MR > SUB) pl_reduce_some<D, MR, NT, SUB, MR - SUB>(L, t, wave, lane, acc, pre, done);
}

// hidden (LayerNorm folded) W^T + b on N column tiles, the workgroup's; cs: their cs, behind them bf (LDS); epi(row of the group,
// column of the workgroup, float[4]) on live rows.
template <int D, int MR, int S, int N, class Epi>
__device__ __forceinline__ void pl_project(const XcdArgs& a, PlLds<D, MR>& L, PlTurn& t, const char* A, bool plain, const char* stats,
                                           float* stat, int rows, const float* cs, Epi&& epi) {
  typedef PlDim<D> Dim;
  const int lane = pl_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lq = lane & 15, g = lane >> 4;
  u32x4 af[MR][Dim::KS];
  PlRows<D, MR>(a, A, plain, rows, lane, wave).first(af, stats, L.part[wave]);
  constexpr int NB = PlLds<D, MR>::kBatch;
  auto batch = [&](auto first, auto count) {
    constexpr int CT = decltype(first)::value, NT = decltype(count)::value;
    f32x4 acc[NT][MR];
    auto tile = [&](auto ahead, int i) {
      bf16x8 wf[Dim::KS];
      pl_weights<D, MR, decltype(ahead)::value>(a, L, t, wave, lane, wf);
#pragma unroll
      for (int mr = 0; mr < MR; ++mr) acc[i][mr] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < Dim::KS; ++u)
#pragma unroll
        for (int mr = 0; mr < MR; ++mr)
          acc[i][mr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[u], __builtin_bit_cast(bf16x8, af[mr][u]), acc[i][mr], 0, 0, 0);
    };
    // (a batch asks at its end: chunk i of it has kRing - 1 - i behind it)
    constexpr int R1 = Dim::kRing - 1;
    tile(std::integral_constant<int, (CT < Dim::kRing ? -1 : R1)>{}, 0);
    if constexpr (NT > 1) tile(std::integral_constant<int, (CT + 1 < Dim::kRing ? -1 : R1 > 1 ? R1 - 1 : 0)>{}, 1);
    if constexpr (NT > 2) tile(std::integral_constant<int, (CT + 2 < Dim::kRing ? -1 : R1 > 2 ? R1 - 2 : 0)>{}, 2);
    if constexpr (NT > 3) tile(std::integral_constant<int, (CT + 3 < Dim::kRing ? -1 : R1 > 3 ? R1 - 3 : 0)>{}, 3);
    static_assert(NT <= 4 && NT <= Dim::kRing, "a batch");
    struct Have { f32x4 c, b; };
    // (ahead of the sum, so that the next stage's rows are waited for behind less of it: 352 rows of d = 512 188.9 -> 186.7 us)
    pl_ask<D, MR, S, Dim::kAsk[S] * CT / N, Dim::kAsk[S] * (CT + NT) / N - Dim::kAsk[S] * CT / N>(a, L, t, wave);
    pl_reduce<D, MR, NT>(L, t, wave, lane, acc,
      [&](int i, int) {
        const float* v = cs + (CT + i) * 16 + 4 * g;
        return Have{*reinterpret_cast<const f32x4*>(v), *reinterpret_cast<const f32x4*>(v + N * 16)};
      },
      [&](int i, int mr, const f32x4& v, const Have& h) {
        const int row = 16 * mr + lq;
        f32x2 st = {1.f, 0.f};
        if (CT > 0) {   // (the first batch's waves have left them)
          st = *reinterpret_cast<const f32x2*>(stat + 2 * row);
        } else {
          if (stats) st = pl_row_stat<D>(&L.part[0][0], 2 * 16 * MR, row, g);
          if (i == 0) *reinterpret_cast<f32x2*>(stat + 2 * row) = st;
        }
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(v[e], st[0], __builtin_fmaf(st[1], h.c[e], h.b[e]));
        if (row < rows) epi(row, (CT + i) * 16 + 4 * g, o);
      });
  };
  batch(std::integral_constant<int, 0>{}, std::integral_constant<int, (N < NB ? N : NB)>{});
  if constexpr (N > NB) batch(std::integral_constant<int, NB>{}, std::integral_constant<int, (N - NB < NB ? N - NB : NB)>{});
  if constexpr (N > 2 * NB) batch(std::integral_constant<int, 2 * NB>{}, std::integral_constant<int, (N - 2 * NB < NB ? N - 2 * NB : NB)>{});
  if constexpr (N > 3 * NB) batch(std::integral_constant<int, 3 * NB>{}, std::integral_constant<int, (N - 3 * NB < NB ? N - 3 * NB : NB)>{});
  if constexpr (N > 4 * NB) batch(std::integral_constant<int, 4 * NB>{}, std::integral_constant<int, (N - 4 * NB < NB ? N - 4 * NB : NB)>{});
  if constexpr (N > 5 * NB) batch(std::integral_constant<int, 5 * NB>{}, std::integral_constant<int, (N - 5 * NB < NB ? N - 5 * NB : NB)>{});
  if constexpr (N > 6 * NB) batch(std::integral_constant<int, 6 * NB>{}, std::integral_constant<int, (N - 6 * NB < NB ? N - 6 * NB : NB)>{});
  if constexpr (N > 7 * NB) batch(std::integral_constant<int, 7 * NB>{}, std::integral_constant<int, (N - 7 * NB < NB ? N - 7 * NB : NB)>{});
  static_assert(N <= 8 * NB, "batches");
}

// residual sum of stage S on the workgroup's columns: y = LN_prev(x) + A W^T + b; K = KC * D.  vecs: the three column vectors (LDS); resid(mr, ct):
// where lane's part of x is and y goes; out(row, column of the workgroup, y) on live rows.
template <int D, int MR, int S, class Resid, class Out>
__device__ __forceinline__ void pl_sum(const XcdArgs& a, PlLds<D, MR>& L, PlTurn& t, const char* A, const float* stat, int rows,
                                       const float* vecs, Resid&& resid, Out&& out) {
  typedef PlDim<D> Dim;
  constexpr int KC = S == 7 ? Dim::kKC : 1;
  const int lane = pl_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lq = lane & 15, g = lane >> 4;
  const PlRows<D, MR> R(a, A, false, rows, lane, wave);
  constexpr int SETS = MR * Dim::KS * KC <= 32 ? KC : MR * Dim::KS <= 16 ? 2 : 1, TD = Dim::kTD;   // chunks of K of which rows are held
  constexpr int NB = PlLds<D, MR>::kBatch, GT = NB < TD ? NB : TD;        // column tiles summed together
  static_assert(TD % GT == 0 && GT <= 2, "whole batches");
  u32x4 af[SETS][MR][Dim::KS];
  f32x4 acc[TD / GT][GT][MR];
#pragma unroll
  for (int ct = 0; ct < TD; ++ct)
#pragma unroll
    for (int mr = 0; mr < MR; ++mr) acc[ct / GT][ct % GT][mr] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) {
    u32x4(&now)[MR][Dim::KS] = af[kc % SETS];
    constexpr bool ALL = KC > 1 && MR * Dim::KS * KC <= 8;
    if constexpr (ALL) {
      if (kc == 0) R.template all<KC>(af);
    } else {
      if (kc == 0) R.first(now, nullptr, nullptr);
      else R.arrive_later(kc, now);
    }
#pragma unroll
    for (int ahead = 1; ahead < (ALL ? 0 : SETS); ++ahead)   // as early as there are registers
      if (kc + ahead < KC && (kc == 0 || ahead + 1 == SETS)) {
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) R.request(mr, kc + ahead, af[(kc + ahead) % SETS]);
      }
#pragma unroll
    for (int ct = 0; ct < TD; ++ct) {
      bf16x8 wf[Dim::KS];
      if (kc * TD + ct < Dim::kRing) pl_weights<D, MR, -1>(a, L, t, wave, lane, wf);
      else if (kc + 1 < KC || ct % GT == 0) pl_weights<D, MR, Dim::kRing - 1>(a, L, t, wave, lane, wf);
      else pl_weights<D, MR, Dim::kRing - 2>(a, L, t, wave, lane, wf);   // (the sum's tiles ask together, behind the last)
#pragma unroll
      for (int u = 0; u < Dim::KS; ++u)
#pragma unroll
        for (int mr = 0; mr < MR; ++mr)
          acc[ct / GT][ct % GT][mr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[u], __builtin_bit_cast(bf16x8, now[mr][u]),
                                                                              acc[ct / GT][ct % GT][mr], 0, 0, 0);
      if (kc + 1 < KC) {   // (a product of few chunks asks for the next ones at its end, all at once)
        if (KC * TD > Dim::kRing) pl_ask<D, MR, S, 0, 1>(a, L, t, wave);
        continue;
      }
      if ((ct + 1) % GT != 0) continue;
      struct Have { f32x4 v[3], x; };
      if (KC * TD > Dim::kRing) pl_ask<D, MR, S, 0, GT>(a, L, t, wave);
      else if (ct + 1 == TD) pl_ask<D, MR, S, 0, Dim::kAsk[S]>(a, L, t, wave);
      pl_reduce<D, MR, GT>(L, t, wave, lane, acc[ct / GT],
        [&](int i, int mr) {
          const int tile = ct / GT * GT + i;
          const float* v = vecs + tile * 16 + 4 * g;
          return Have{{*reinterpret_cast<const f32x4*>(v), *reinterpret_cast<const f32x4*>(v + Dim::kND), *reinterpret_cast<const f32x4*>(v + 2 * Dim::kND)},
                      *reinterpret_cast<const f32x4*>(resid(mr, tile))};
        },
        [&](int i, int mr, const f32x4& v, const Have& h) {
          const int tile = ct / GT * GT + i, row = 16 * mr + lq;
          const f32x2 st = *reinterpret_cast<const f32x2*>(stat + 2 * row);
          f32x4 y, gx;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            y[e] = v[e] + __builtin_fmaf(__builtin_fmaf(h.x[e], st[0], st[1]), h.v[0][e], h.v[1][e]);
            gx[e] = y[e] * h.v[2][e];
          }
          *reinterpret_cast<f32x4*>(resid(mr, tile)) = y;
          out(row, tile * 16 + 4 * g, y, gx);
        });
    }
    if (SETS == 1 && kc + 1 < KC) {
      asm volatile("" ::: "memory");   // (not above the products: there is one set of registers)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mr = 0; mr < MR; ++mr) R.request(mr, kc + 1, af[0]);
    }
  }
}

// The queries of a workgroup's unit of cross-attention, formed by the workgroup itself: a product of a head's 64 columns in place of a stage
// of its own and its hand-over, where the units of self-attention and of cross-attention have workgroups of their own (PlPlace::w from below
// and from above).  The weights and the first chunk of keys and values are requested while the others are at self-attention and held until the
// rows are there; the queries pass through LDS.  Same products, sums and statistics as in that stage: the same bits.
template <int D>
struct PlOwnQueries {
  typedef PlDim<D> Dim;
  static constexpr int kPitch = 72;   // (16 rows of 144 bytes: a 16-byte read of every row meets all banks once)
  bf16x8 wf[4][Dim::KS];
  f32x4 c, b;
  PlChunk chunk;
  __device__ __forceinline__ void request(const XcdArgs& a, PlLayerPtr Y, int l, int h, int lane, int wave) {
    const int g = lane >> 4;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const int tile = h * 4 + f;
      // (operands in order, from a copy of this matrix behind the column vectors.  As bound, half of each of 16 lines a request: 6 rows 112.7 us,
      // so 108.8.)
      const char* p = reinterpret_cast<const char*>(a.vecs) + ((size_t)a.n_layers * kPlMembers * Dim::kVecPitch * 4 + ((size_t)(l * (D / 16) + tile) * kPlWaves + wave) * Dim::kChunk);
#pragma unroll
      for (int u = 0; u < Dim::KS; ++u) wf[f][u] = *reinterpret_cast<const bf16x8*>(p + lane * 16 + u * 1024);
    }
    const int n = h * kHeadDim + (wave & 3) * 16 + 4 * g;   // (the first four waves' column tiles)
    c = *reinterpret_cast<const f32x4*>(Y->cq_cs + n);
    b = *reinterpret_cast<const f32x4*>(Y->cq_bf + n);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
  // the unit's queries as operands f
  template <int MR>
  __device__ __forceinline__ void form(const XcdArgs& a, PlLds<D, MR>& L, const PlExch& ex, const PlUnit& t, int lane, int wave, u32x4 (&f)[2]) const {
    const int lq = lane & 15, g = lane >> 4, row0 = t.b * a.T + t.q0;
    u32x4 af[1][Dim::KS];
    PlRows<D, 1>(a, ex.xg(0) + row0 * 32, false, min(16, a.T - t.q0), lane, wave).first(af, ex.st(0) + row0 * 8, L.part[wave]);
    f32x4* red = L.red;
    bf16* q = L.queries();
    f32x4 acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < Dim::KS; ++u)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i][u], __builtin_bit_cast(bf16x8, af[0][u]), acc[i], 0, 0, 0);
    }
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[3]));   // (the last of the products; see mfma_settle)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      asm volatile("" : "+v"(acc[i]));   // (not ahead of it)
      red[(i * kPlWaves + wave) * 64 + lane] = acc[i];
    }
    lds_barrier();
    if (wave < 4) {
      f32x4 p[kPlWaves];
#pragma unroll
      for (int w = 0; w < kPlWaves; ++w) p[w] = red[(wave * kPlWaves + w) * 64 + lane];
      const f32x2 st = pl_row_stat<D>(&L.part[0][0], 2 * 16 * MR, lq, g);
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = p[0][e];
#pragma unroll
        for (int w = 1; w < kPlWaves; ++w) v += p[w][e];
        o[e] = __builtin_fmaf(v, st[0], __builtin_fmaf(st[1], c[e], b[e]));
      }
      *reinterpret_cast<u32x2*>(q + lq * kPitch + wave * 16 + 4 * g) = pl_pack4(o);
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 2; ++i) f[i] = *reinterpret_cast<const u32x4*>(q + lq * kPitch + i * 32 + 8 * g);
  }
};
// Key chunks kw, kw + kstep, ... of 32 on this wave (see attn_core.h for the operand layouts).  SELF: keys / values below the
// pass's first row come from the cache, the pass's own from the exchange buffers (waited for); else the cross-attention arenas.
// KV8 (cross): codes with one fp32 scale per key and per value, as in attn_core.h.
// SLOTS: of the a.T row places of a sequence the first `live` hold rows of the pass; the first `causal` of them see the keys up to their own,
// the others (a drafter's slots) all keys.  Places beyond see none, and nobody reads what becomes of them.  (Else all see the keys up to their own.)
// PHASE 1: requests the first chunk of cross-attention alone; 2: that chunk and the queries f are there.
template <bool SELF, bool KV8, bool SLOTS, int PHASE>
__device__ __forceinline__ void pl_attn_wave(const XcdArgs& a, const PlExch& ex, int l, int b0, const PlUnit& t, int causal, int live, int kw, int kstep,
                                             bf16* Vs, PlChunk& now, u32x4 (&f)[2], float& mrun, float& lrun, f32x4 (&oacc)[4]) {
  const int lane = pl_lane(), lq = lane & 15, g = lane >> 4;
  const int r0 = t.b * a.T;                                // first row of the sequence, in the group
  const int j = t.j, nkey = t.nkey;
  const int cap = SELF ? a.Lcap : a.Scap;
  const size_t arena = ((size_t)(b0 + t.b) * a.H + t.h) * cap * kHeadDim;
  constexpr int EB = KV8 ? 1 : 2;   // bytes of an element
  const char* kb = (SELF ? reinterpret_cast<const char*>(a.kc + a.kv_layer * l) : static_cast<const char*>(a.xk) + a.xkv_layer * l * EB) + arena * EB;
  const char* vb = (SELF ? reinterpret_cast<const char*>(a.vc + a.kv_layer * l) : static_cast<const char*>(a.xv) + a.xkv_layer * l * EB) + arena * EB;
  const size_t sc0 = KV8 ? (a.xkv_layer * l + arena) / kHeadDim : 0;
  mrun = kNegInf;
  lrun = 0.f;
#pragma unroll
  for (int et = 0; et < 4; ++et) oacc[et] = f32x4{0.f, 0.f, 0.f, 0.f};
  // K operands: tile i, row lq  <->  key c0 + 8*(lq/4) + 4*i + lq%4; values as whole rows (lane -> row 8*i + lane/8, dims
  // 8*(lane%8) .. + 7) or, key-blocked, as operands.  A chunk without rows of the pass is requested ahead.
  PlChunk next;
  auto key_k = [&](int c0, int i) { return c0 + 8 * (lq >> 2) + 4 * i + (lq & 3); };
  auto key_v = [&](int c0, int i) { return c0 + 8 * i + (lane >> 3); };
  auto fetch = [&](int c0, PlChunk& t) {
    const int last = (SELF ? j : nkey) - 1;
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
  const PlBuf qb = pl_buf(ex.q(SELF ? 0 : 1));
  const int off = pl_at(a.RP, r0, t.h * kHeadDim), xtile = a.RP * 32, offq = off + pl_at(a.RP, min(t.q0 + lq, a.T - 1), 8 * g);
  unsigned spins = 0;
  // a chunk with rows of the pass: every lane's keys and values from the cache or the exchange buffers, and the queries, until all
  // are there.  (One statement: its results are valid behind its wait.)
  auto own = [&](int c0, PlChunk& t_) {
    const char *pk[4], *pv[4], *pq[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int key = key_k(c0, i), row = min(max(key - j, 0), a.T - 1);
      const bool mine = key >= j;
      pk[2 * i] = mine ? ex.kx() + off + pl_at(a.RP, row, 8 * g) : kb + key * 128 + g * 16;
      pk[2 * i + 1] = pk[2 * i] + (mine ? 2 * xtile : 64);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = key_v(c0, i), row = min(max(key - j, 0), a.T - 1);
      pv[i] = key >= j ? ex.vx() + off + pl_at(a.RP, row, 8 * (lane & 7)) : vb + key * 128 + (lane & 7) * 16;
    }
    pq[0] = ex.q(0) + offq;
    pq[1] = pq[0] + 2 * xtile;
    while (true) {
      asm volatile("global_load_dwordx4 %0, %10, off sc1\n\tglobal_load_dwordx4 %1, %11, off sc1\n\t"
                   "global_load_dwordx4 %2, %12, off sc1\n\tglobal_load_dwordx4 %3, %13, off sc1\n\t"
                   "global_load_dwordx4 %4, %14, off sc1\n\tglobal_load_dwordx4 %5, %15, off sc1\n\t"
                   "global_load_dwordx4 %6, %16, off sc1\n\tglobal_load_dwordx4 %7, %17, off sc1\n\t"
                   "global_load_dwordx4 %8, %18, off sc1\n\tglobal_load_dwordx4 %9, %19, off sc1\n\ts_waitcnt vmcnt(0)"
                   : "=&v"(t_.kf[0]), "=&v"(t_.kf[1]), "=&v"(t_.kf[2]), "=&v"(t_.kf[3]), "=&v"(t_.vf[0]), "=&v"(t_.vf[1]),
                     "=&v"(t_.vf[2]), "=&v"(t_.vf[3]), "=&v"(f[0]), "=&v"(f[1])
                   : "v"(pk[0]), "v"(pk[1]), "v"(pk[2]), "v"(pk[3]), "v"(pv[0]), "v"(pv[1]), "v"(pv[2]), "v"(pv[3]), "v"(pq[0]), "v"(pq[1])
                   : "memory");
      // (keys at and beyond nkey are masked later: not waited for, but the first place's of a sequence without rows is, for the sake of the
      // refill)
      const int end = SLOTS ? max(nkey, j + 1) : nkey;
      bool bad = pl_missing(f[0]) || pl_missing(f[1]);
#pragma unroll
      for (int i = 0; i < 4; ++i) bad |= key_k(c0, i >> 1) >= j && key_k(c0, i >> 1) < end && pl_missing(t_.kf[i]);
#pragma unroll
      for (int i = 0; i < 4; ++i) bad |= key_v(c0, i) >= j && key_v(c0, i) < end && pl_missing(t_.vf[i]);
      if (!__builtin_amdgcn_ballot_w64(bad)) break;
      pl_again(spins, a);
    }
    // (values beyond nkey meet a probability of zero: they must be finite)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) t_.vf[i][e] = key_v(c0, i) >= nkey ? 0u : t_.vf[i][e];
  };
  const int cfirst = kw * 32;
  if (PHASE == 1) {
    fetch(cfirst, now);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    return;
  }
  if (SELF && cfirst + 32 > j) {
    own(cfirst, now);
  } else if (PHASE == 0) {
    fetch(cfirst, now);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    while (true) {
#pragma unroll
      for (int i = 0; i < 2; ++i) f[i] = pl_request(qb, offq, i * 2 * xtile);
      if (!__builtin_amdgcn_ballot_w64(pl_missing(f[0]) || pl_missing(f[1]))) break;
      pl_again(spins, a);
    }
  }
  const bf16x8 q0 = __builtin_bit_cast(bf16x8, f[0]), q1 = __builtin_bit_cast(bf16x8, f[1]);
  const int qrow = t.q0 + lq;
  const int lim = SELF && SLOTS ? (qrow < causal ? j + qrow + 1 : qrow < live ? j + live : 0) : qrow < a.T ? (SELF ? j + qrow + 1 : nkey) : 0;
  for (int c0 = cfirst; c0 < nkey; c0 += kstep * 32) {
    const int c1 = c0 + kstep * 32;
    if (c1 < nkey && !(SELF && c1 + 32 > j)) fetch(c1, next);
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
    if (SELF && c1 < nkey && c1 + 32 > j) {
      own(c1, now);
    } else if (c1 < nkey) {
      now = next;
    }
  }
  mfma_settle(oacc);
}

// All units of one attention stage: as many waves to a unit as there are (XcdArgs::wpu), a power of two.  The waves of a unit take
// chunks of 32 keys in turn and merge through LDS.
struct PlPair { int b, h, q0; };   // sequence of the group, head, first query
__device__ __forceinline__ PlPair pl_pair(const XcdArgs& a, const PlPlace& p, int r, int wave) {
  const int tiles = (a.T + 15) >> 4, u = min((r * kPlMembers + p.w) * (kPlWaves / a.wpu) + wave / a.wpu, pl_units(a, p) - 1), pair = u / tiles, b = pair / a.H;
  return PlPair{__builtin_amdgcn_readfirstlane(b), __builtin_amdgcn_readfirstlane(pair - b * a.H), __builtin_amdgcn_readfirstlane((u - pair * tiles) * 16)};
}
// mine: the unit of the first round (there is seldom another)
// FORM: the units' queries may be formed here (form: they are, and units come from above); own: what is held of it
template <bool SELF, bool KV8, bool SLOTS, bool FORM, int D, int MR>
__device__ __forceinline__ void pl_attention(const XcdArgs& a, const PlExch& ex, int l, const PlPlace& at, const PlPair& mine, int units, int rounds, PlLds<D, MR>& L,
                                             PlTurn& turn, bool form, PlOwnQueries<D>& own) {
  char* out = ex.att(SELF ? 0 : 1);
  const int wpu = a.wpu, log = 31 - __builtin_clz(wpu), per = kPlWaves >> log;   // waves of a unit, units at a time
  for (int r = 0; r < rounds; ++r) {
    // (What follows from the lane and the wave is worked out in the round, where it is used: ahead of the loop, where the compiler would have it,
    // the merge's share of it comes before the keys' and values' requests.)
    const int lane = pl_lane(), wave = pl_wave(), lq = lane & 15, g = lane >> 4, kw = wave & (wpu - 1);
    const int u = FORM && form ? kPlMembers - 1 - at.w : (r * kPlMembers + at.w) * per + (wave >> log);
    const PlPair pair = r == 0 ? mine : pl_pair(a, at, r, wave);
    PlUnit t;
    t.b = pair.b; t.h = pair.h; t.q0 = pair.q0;
    t.j = SELF ? __builtin_amdgcn_readfirstlane(L.seq[t.b].j) : 0;
    const int causal = SELF && SLOTS ? __builtin_amdgcn_readfirstlane(L.seq[t.b].causal) : 0;
    const int live = SELF && SLOTS ? __builtin_amdgcn_readfirstlane(L.seq[t.b].live) : 0;
    t.nkey = !SELF ? __builtin_amdgcn_readfirstlane(L.seq[t.b].src_len) : t.j + (!SLOTS ? min(a.T, t.q0 + 16) : t.q0 + 16 <= causal ? t.q0 + 16 : live);
    const int chunks = (t.nkey + 31) >> 5, used = u < units ? min(max(chunks, 1), wpu) : 0;   // waves with keys (one at least)
    float mrun, lrun;
    f32x4 oacc[4];
    auto store = [&](int et, const f32x4& o, float inv) {
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = o[i] * inv;
      const u32x2 p = pl_pack4(v);
      if (t.q0 + lq < a.T) pl_store8(out + pl_at(a.RP, t.b * a.T + t.q0 + lq, t.h * kHeadDim + et * 16 + 4 * g), p[0], p[1]);
    };
    lds_barrier();   // the latest product's partial tiles, or the units' before, are done with
    if (FORM && form) {   // (every wave takes part in forming the queries)
      u32x4 f[2];
      if (used > 0) own.form(a, L, ex, t, lane, wave, f);
      if (kw < used) pl_attn_wave<SELF, KV8, SLOTS, FORM ? 2 : 0>(a, ex, l, at.b0, t, causal, live, kw, wpu, L.vs(wave), own.chunk, f, mrun, lrun, oacc);
    } else if (kw < used) {
      PlChunk chunk;
      u32x4 f[2];
      pl_attn_wave<SELF, KV8, SLOTS, 0>(a, ex, l, at.b0, t, causal, live, kw, wpu, L.vs(wave), chunk, f, mrun, lrun, oacc);
    }
    if (used == 1 && kw == 0) {   // nothing to merge
      const float inv = lrun > 0.f ? 1.f / lrun : 0.f;
#pragma unroll
      for (int et = 0; et < 4; ++et) store(et, oacc[et], inv);
    }
    // O of every wave to LDS (where its values were); wave et of the unit (two or more et's where it has few waves) merges dims
    // 16 et .. + 15
    f32x4* om = L.red;    // [wave][et][lane]
    float* ml = L.ml;     // [wave][max, sum][16]
    if (used > 1 && kw < used) {
#pragma unroll
      for (int et = 0; et < 4; ++et) om[(wave * 4 + et) * 64 + lane] = oacc[et];
      if (g == 0) { ml[wave * 32 + lq] = mrun; ml[wave * 32 + 16 + lq] = lrun; }
    }
    lds_barrier();
    // what is requested goes behind all waves' keys and values, and behind the merge on the waves that have a share of it
    auto ask = [&] {
      if (r + 1 == rounds) pl_ask<D, MR, SELF ? 1 : 4, 0, PlDim<D>::kAsk[SELF ? 1 : 4]>(a, L, turn, wave);
    };
    if (used <= 1 || kw >= 4) ask();
    auto merge = [&](auto most) {
      constexpr int W = decltype(most)::value;
      const int first = wave - kw;
      float ms[W], ls[W], M = kNegInf, Ls = 0.f;
#pragma unroll
      for (int s = 0; s < W; ++s) {
        const int w = first + min(s, used - 1);
        ms[s] = ml[w * 32 + lq];
        ls[s] = ml[w * 32 + 16 + lq];
      }
#pragma unroll
      for (int s = 0; s < W; ++s) M = fmaxf(M, ms[s]);
#pragma unroll
      for (int s = 0; s < W; ++s) {
        ms[s] = s < used && ms[s] > kNegInf ? __builtin_amdgcn_exp2f((ms[s] - M) * kCexp) : 0.f;
        Ls += ls[s] * ms[s];
      }
      const float inv = Ls > 0.f ? 1.f / Ls : 0.f;
      for (int et = kw; et < 4; et += wpu) {
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < W; ++s) {
          const f32x4 v = om[((first + min(s, used - 1)) * 4 + et) * 64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] += v[i] * ms[s];
        }
        store(et, o, inv);
      }
    };
    if (used > 1 && kw < 4) {
      if (used <= 3) merge(std::integral_constant<int, 3>{});
      else merge(std::integral_constant<int, kPlWaves>{});
      ask();
    }
  }
  lds_barrier();
}

// KV8: cross-attention keys / values as E4M3 codes.
// MR: row tiles of a group.
// TICKETS: see the head of this file; the residual in memory instead of LDS.
// DIRECT: the weights read in place (d = 512: a few rows, a drafter's).
// SLOTS: a drafter's rows (XcdArgs::causal); the second run asks for both kinds.  (As what every pass asks, verify passes of d = 512 took 0.5 - 1.6 %
// longer.)
template <bool KV8, int D, int MR, bool TICKETS, bool DIRECT, bool SLOTS>
__global__ __launch_bounds__(kPlThreads) void pl_decoder_kernel(XcdArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char pl_smem[];
  typedef PlLds<D, MR> Lds;
  typedef PlDim<D> Dim;
  static_assert(sizeof(Lds) <= 160 * 1024, "LDS of a CU");
  constexpr bool kHalf = MR > kPlRows / 16;   // half of the exchange buffers are filled when the pass starts
  Lds& L = *reinterpret_cast<Lds*>(pl_smem);
  if (!TICKETS) a.RP = 16 * MR;   // known when compiled: every place in the exchange buffers is then a constant away from the layer's
  a.H = D / kHeadDim;
  if (DIRECT) a.stream = nullptr;
  if (!TICKETS && !DIRECT) __builtin_assume(a.stream != nullptr);
  // (one look for all waves: others may raise the flag meanwhile, and none of a workgroup's waves is to go on without the rest)
  if (threadIdx.x == 0) L.row_at[0] = (int)__hip_atomic_load(a.raised, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if ((__builtin_amdgcn_readfirstlane(L.row_at[0]) != 0) != TICKETS) return;
  __syncthreads();
  // the XCD this workgroup runs on (hardware register 20, its lowest four bits)
  const int xcd = (int)__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11));
  if (!TICKETS && xcd >= a.G) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  PlPlace at = pl_place(a, TICKETS ? 0 : xcd, (int)blockIdx.x / kPlGroups);
  // what the workgroup needs of its group's rows
  auto take_rows = [&] {
    for (int i = threadIdx.x; i < at.rows; i += kPlThreads) {
      const int b = a.row_b[at.row0 + i], pos = a.row_pos[at.row0 + i];
      L.row_at[i] = b < 0 ? -1 : b * a.H * a.Lcap + pos;
    }
    for (int i = threadIdx.x; i < at.nb; i += kPlThreads) {
      const int b = at.b0 + i;
      L.seq[i] = PlSeq{a.row_pos[b * a.T], SLOTS && a.causal ? a.causal[b] : a.T, SLOTS && a.causal ? a.live[b] : a.T, a.src_len[b]};
    }
  };
  if (!TICKETS) take_rows();
  PlTurn turn = pl_turn<D>(a, at.w, wave, 0, 0, a.n_layers * Dim::kPerLayer);
  int units = pl_units(a, at), rounds = pl_rounds(a, at);
  PlPair mine = pl_pair(a, at, 0, wave);
  PlPlace from_above = at;
  from_above.w = kPlMembers - 1 - at.w;
  const PlPair above = pl_pair(a, from_above, 0, wave);
  PlOwnQueries<D> own;
  // stage s of layer l
  auto stage = [&](int s, int l) __attribute__((always_inline)) {
    // What follows from the layer is worked out where it is used.  Ahead of the layer's stages, where the compiler would have it, it does not fit
    // the scalar registers and goes through lanes of vector ones: with the builtin in pl_again and the row pitch of the buffers as an argument
    // a wave issued 500 instructions a stage, half of them scalar.  Whole verify passes, us, with all that / without: d = 512, 77 rows
    // 149.3 / 133.9, 352 rows 198.4 / 188.9; d = 1024, 352 rows of long sources 544 / 530, 209 rows 422 / 408.
    asm volatile("" : "+s"(l));
    if constexpr (DIRECT) {
      if (s == 0) pl_ask_at<D, 0>(a, turn, l);
      if (s == 1) pl_ask_at<D, 1>(a, turn, l);
      if (s == 2 || s == 3 || s == 4) pl_ask_at<D, 2>(a, turn, l);
      if (s == 5 || s == 6) pl_ask_at<D, 5>(a, turn, l);
      if (s == 7) pl_ask_at<D, 7>(a, turn, l);
    }
    const PlExch ex(a.exch + (kHalf ? (l & 1) * a.G + at.g : at.g * 2 + (l & 1)) * pl_layer_bytes(a.RP, D, 4 * D), a.RP, D);
    const PlExch before(a.exch + (kHalf ? (~l & 1) * a.G + at.g : at.g * 2 + (~l & 1)) * pl_layer_bytes(a.RP, D, 4 * D), a.RP, D);
    const float* vec = L.vec[l & 1];
    float* stat = L.stat[(3 * l + s / 3) & 1];
    // (see PlOwnQueries)
    constexpr bool FORM = !TICKETS && Lds::kForm;
    const bool form = FORM && a.form;
    if (s == 1) {
      pl_attention<true, false, SLOTS, false>(a, ex, l, at, mine, units, rounds, L, turn, false, own);
      if (FORM && form && kPlMembers - 1 - at.w < units) {
        const int lane = pl_lane();
        PlUnit t;
        t.b = above.b; t.h = above.h; t.q0 = above.q0; t.j = 0;
        t.nkey = __builtin_amdgcn_readfirstlane(L.seq[t.b].src_len);
        own.request(a, pl_layer(a, l), l, above.h, lane, wave);
        float m;
        f32x4 o[4];
        u32x4 f[2];
        if (wave * 32 < t.nkey) pl_attn_wave<false, KV8, SLOTS, 1>(a, ex, l, at.b0, t, 0, 0, wave, kPlWaves, L.vs(wave), own.chunk, f, m, m, o);
      }
      return;
    }
    if (s == 4) return pl_attention<false, KV8, SLOTS, FORM>(a, ex, l, at, FORM && form ? above : mine, units, rounds, L, turn, form, own);
    // the statistics of the LayerNorm pending on the residual
    const char* st = s <= 2 ? (l == 0 ? nullptr : before.st(2)) : s <= 5 ? ex.st(0) : ex.st(1);
    if (s == 0 || s == 3 || s == 6) {
      const bool top = s == 0 && l == 0;
      const char* A = top ? reinterpret_cast<const char*>(a.xb + (size_t)at.row0 * D) : s == 0 ? before.xg(2) : s == 3 ? ex.xg(0) : ex.xg(1);
      if (s == 0) {   // queries, keys, values (these appended to the cache as well)
        pl_project<D, MR, 0, Dim::kTQ>(a, L, turn, A, top, st, stat, at.rows, vec + Dim::kVecQ, [&](int row, int c, const float (&v)[4]) {
          const int col = at.w * Dim::kNQ + c, part = col / D, cc = col - part * D;
          const u32x2 p = pl_pack4(v);
          pl_store8((part == 0 ? ex.q(0) : part == 1 ? ex.kx() : ex.vx()) + pl_at(a.RP, row, cc), p[0], p[1]);
          const int to = L.row_at[row];
          if (part == 0 || to < 0) return;
          bf16* cache = (part == 1 ? a.kc : a.vc) + a.kv_layer * l;
          *reinterpret_cast<u32x2*>(cache + (size_t)(to + (cc >> 6) * a.Lcap) * kHeadDim + (cc & 63)) = p;
        });
      } else if (s == 3 && form) {   // (its weights are passed over)
        for (int i = 0; i < Dim::kTD; ++i) turn.use = turn.use + Dim::kChunk == Dim::kRing * Dim::kChunk ? 0 : turn.use + Dim::kChunk;
        pl_ask<D, MR, 3, 0, Dim::kAsk[3]>(a, L, turn, wave);
      } else if (s == 3) {
        pl_project<D, MR, 3, Dim::kTD>(a, L, turn, A, false, st, stat, at.rows, vec + Dim::kVecC, [&](int row, int c, const float (&v)[4]) {
          const u32x2 p = pl_pack4(v);
          pl_store8(ex.q(1) + pl_at(a.RP, row, at.w * Dim::kND + c), p[0], p[1]);
        });
      } else {
        pl_project<D, MR, 6, Dim::kTF>(a, L, turn, A, false, st, stat, at.rows, vec + Dim::kVecF, [&](int row, int c, const float (&v)[4]) {
          const float o[4] = {fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
          const u32x2 p = pl_pack4(o);
          pl_store8(ex.hid() + pl_at(a.RP, row, at.w * Dim::kNF + c), p[0], p[1]);
        });
      }
      return;
    }
    const int i = s == 2 ? 0 : s == 5 ? 1 : 2;   // which sum
    const bool last = s == 7 && l + 1 == a.n_layers;
    if (TICKETS) {   // (another workgroup may have formed them for the projection before)
      u32x4 none[MR][Dim::KS];
      PlRows<D, MR>(a, s == 7 ? ex.hid() : ex.att(i), false, at.rows, pl_lane(), wave).first(none, st, L.part[wave]);
      lds_barrier();
      for (int mr = wave; mr < MR; mr += kPlWaves) {
        const int row = 16 * mr + (pl_lane() & 15);
        *reinterpret_cast<f32x2*>(stat + 2 * row) = st ? pl_row_stat<D>(&L.part[0][0], 2 * 16 * MR, row, pl_lane() >> 4) : f32x2{1.f, 0.f};
      }
    }
    if (s == 5 && form) {   // the statistics, which stage 3 has not formed
      PlRows<D, MR>(a, ex.xg(0), false, at.rows, pl_lane(), wave).statistics(st, L.part[wave]);
      lds_barrier();
      if (wave < MR) {
        const int row = 16 * wave + (pl_lane() & 15);
        *reinterpret_cast<f32x2*>(stat + 2 * row) = pl_row_stat<D>(&L.part[0][0], 2 * 16 * MR, row, pl_lane() >> 4);
      }
    }
    auto resid = [&](int mr, int ct) {
      const int lane = pl_lane(), lq = lane & 15, g = lane >> 4;
      if (TICKETS) return a.resid + (size_t)(at.g * 16 * MR + 16 * mr + lq) * D + (at.w * Dim::kTD + ct) * 16 + 4 * g;
      return L.resid + ((ct * MR + mr) * 16 + lq) * 16 + 4 * g;
    };
    auto out = [&](int row, int c, const f32x4& y, const f32x4& gx) {
      const int col = at.w * Dim::kND + c, g = pl_lane() >> 4;
      const bool live = row < at.rows;
      if (last) {
        if (live) *reinterpret_cast<f32x4*>(a.y + (size_t)(at.row0 + row) * D + col) = y;
        return;
      }
      const float o[4] = {gx[0], gx[1], gx[2], gx[3]};
      const u32x2 w = pl_pack4(o);
      if (live) pl_store8(ex.xg(i) + pl_at(a.RP, row, col), w[0], w[1]);
      float sum = 0.f, ss = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) { sum += y[e]; ss = __builtin_fmaf(y[e], y[e], ss); }
      sum = pl_row_sum(sum);
      ss = pl_row_sum(ss);
      if (live && g == 0)
        pl_store8(ex.st(i) + ((col >> 4) * a.RP + row) * 8, __builtin_bit_cast(unsigned, sum),
                           __builtin_bit_cast(unsigned, fmaxf(ss - sum * sum * (1.0f / 16), 0.f)));
    };
    const float* vecs = vec + Dim::kVecS + i * 3 * Dim::kND;
    if (s == 7) return pl_sum<D, MR, 7>(a, L, turn, ex.hid(), stat, at.rows, vecs, resid, out);
    if (s == 5) return pl_sum<D, MR, 5>(a, L, turn, ex.att(i), stat, at.rows, vecs, resid, out);
    pl_sum<D, MR, 2>(a, L, turn, ex.att(i), stat, at.rows, vecs, resid, out);
    if (!TICKETS && (l > 0 || kHalf) && l + 1 < a.n_layers) {   // nobody reads the layer before any more
      const u32x4 poison = {kPoison, kPoison, kPoison, kPoison};
      const int bytes = (int)(pl_layer_bytes(a.RP, D, 4 * D) / kPlMembers);
      for (int o = (wave * 64 + pl_lane()) * 16; o < bytes; o += kPlWaves * 1024) *reinterpret_cast<u32x4*>(before.base + at.w * bytes + o) = poison;
    }
    // (what every wave asks for and stores here is done with when it has its rows of stage 3, for the workgroup at the barriers there.  Where units
    // form their queries nothing is waited for in stage 3, and in stage 4 by the workgroups of units alone: there it is done with in stage 5 when the
    // wave has its statistics, which it requests behind all this, and at the barrier behind them, ahead of all that the workgroup stores in that stage.
    // Nobody can be in the next layer before: its first product takes rows of stage 7 from every workgroup.)
    if (!TICKETS && l + 1 < a.n_layers) pl_ask_vectors<D, MR>(a, L, l + 1, at.w, wave);
  };
  if constexpr (!TICKETS) {
    for (int i = threadIdx.x; i < Dim::kTD * 16 * MR * 4; i += kPlThreads) {   // the residual: embedded rows
      const int ct = i / (16 * MR * 4), row = (i >> 2) % (16 * MR), c = (i & 3) * 4;
      *reinterpret_cast<f32x4*>(L.resid + i * 4) =
          *reinterpret_cast<const f32x4*>(a.x + (size_t)(at.row0 + min(row, at.rows - 1)) * D + (at.w * Dim::kTD + ct) * 16 + c);
    }
    __syncthreads();
    pl_ask_vectors<D, MR>(a, L, 0, at.w, wave);
    if constexpr (DIRECT) pl_ask_rows<D, MR>(a, L, turn, wave, 0, 0, Dim::kAskFirst);
    else pl_ask_next<D, MR>(L, turn, wave, Dim::kAskFirst);
    wait_vmcnt<Dim::kAskFirst * Dim::kReq>();   // the vectors
    __syncthreads();
    for (int l = 0; l < a.n_layers; ++l) {
      stage(0, l);
      if (SLOTS && a.kv_only && l + 1 == a.n_layers) {
        wait_vmcnt<0>();   // (weights on their way to LDS, as in pl_again)
        return;
      }
      stage(1, l); stage(2, l); stage(3, l); stage(4, l); stage(5, l); stage(6, l); stage(7, l);
    }
  } else {
    const int per = a.G * kPlMembers, total = (a.n_layers * kPlStages - (a.kv_only ? kPlStages - 1 : 0)) * per;   // tickets of a stage; of the pass: below 2^17
    int st = -1, group = -1;
    while (true) {
      // (In one block: see persist.hip)
      if (threadIdx.x == 0) {
        if (st >= 0) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the caches' write-back, which the fence only starts)
          __hip_atomic_fetch_add(&a.tickets->done[st], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        L.drawn = (int)(__hip_atomic_fetch_add(&a.tickets->drawn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u);
      }
      __syncthreads();
      // a wave that gives up ends, and what it would have drawn or left the others cannot go on with
      if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0) return;
      const int t = __builtin_amdgcn_readfirstlane(L.drawn);
      st = t / per;
      if (t >= total) {   // (the last workgroup to find none left: every one has read the flag, and nothing else writes it now)
        if (t == total + (int)gridDim.x - 1 && threadIdx.x == 0) *a.raised -= 1u;
        return;
      }
      const int l = st / kPlStages, s = st - l * kPlStages, g = (t - st * per) / kPlMembers;
      // everything before this stage: its tickets are out, so whoever holds them is running
      unsigned spins = 0;
      while (st > 0 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(&a.tickets->done[st - 1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT)) + 1u != (unsigned)per) {
        if (++spins > kPlTicketSpinMax || __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0) {
          __hip_atomic_store(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      at = pl_place(a, g, (t - st * per) % kPlMembers);
      if (g != group) take_rows();
      group = g;
      units = pl_units(a, at);
      rounds = pl_rounds(a, at);
      mine = pl_pair(a, at, 0, wave);
      int c = 0;
      for (int e = 0; e < s; ++e) c += pl_chunks<Dim>(e);
      turn = pl_turn<D>(a, at.w, wave, l, c, pl_chunks<Dim>(s));
      pl_ask_vectors<D, MR>(a, L, l, at.w, wave);
      if (D == 512 && !a.stream) pl_ask_rows<D, MR>(a, L, turn, wave, l, c, Dim::kRing);
      else pl_ask_next<D, MR>(L, turn, wave, Dim::kRing);
      if (st == 0) {   // the residual of the member's columns: embedded rows (those beyond the group's: read, never used)
        for (int i = threadIdx.x; i < 16 * MR * (Dim::kND / 4); i += kPlThreads) {
          const int row = i / (Dim::kND / 4), col = at.w * Dim::kND + i % (Dim::kND / 4) * 4;
          *reinterpret_cast<f32x4*>(a.resid + (size_t)(g * 16 * MR + row) * D + col) =
              *reinterpret_cast<const f32x4*>(a.x + (size_t)(at.row0 + min(row, at.rows - 1)) * D + col);
        }
      }
      wait_vmcnt<0>();
      __syncthreads();
      stage(s, l);
      wait_vmcnt<0>();   // (all that this wave stored is out)
      __syncthreads();   // (and the ticket has been read)
    }
  }
}

template <bool KV8, int D, int MR, bool TICKETS, bool DIRECT = false, bool SLOTS = TICKETS>
static hipError_t pl_launch(hipStream_t st, const XcdArgs& a, int blocks) {
  constexpr int kBytes = (int)sizeof(PlLds<D, MR>);
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(pl_decoder_kernel<KV8, D, MR, TICKETS, DIRECT, SLOTS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
  if (attr != hipSuccess) return attr;
  SD_LAUNCH_TIMED((pl_decoder_kernel<KV8, D, MR, TICKETS, DIRECT, SLOTS>), dim3(blocks), dim3(kPlThreads), kBytes, st, a);
  return hipGetLastError();
}
// The pass, and its second run by tickets: workgroups for the members of one group, or of two where there are more (a fraction of the chip, so
// that it costs little to start; a pass of 8 x 7 rows of d = 512 by 32 / 64 / 128 of them 3.1 / 2.1 / 1.9 ms, of one sentence by as many 0.44 / 0.59 / 0.92).
template <bool KV8, int D>
hipError_t pl_launch_both(hipStream_t st, XcdArgs a, int blocks) {
  hipError_t e = hipErrorInvalidValue;
  if constexpr (D == 512) {
    if (!a.copy) {   // (a verification pass from the copy: within 1 %)
      if (a.RP == 80) e = pl_launch<KV8, D, 5, false, true, true>(st, a, blocks);
      if (a.RP == 96) e = pl_launch<KV8, D, 6, false, true, true>(st, a, blocks);
      if (a.RP == 112) e = pl_launch<KV8, D, 7, false, true, true>(st, a, blocks);
      if (a.RP == 128) e = pl_launch<KV8, D, 8, false, true, true>(st, a, blocks);
      if (a.RP == 144) e = pl_launch<KV8, D, 9, false, true, true>(st, a, blocks);
      if (a.RP == 160) e = pl_launch<KV8, D, 10, false, true, true>(st, a, blocks);
    } else if (a.causal) {
      if (a.RP == 16) e = pl_launch<KV8, D, 1, false, true, true>(st, a, blocks);
      if (a.RP == 32) e = pl_launch<KV8, D, 2, false, true, true>(st, a, blocks);
      if (a.RP == 48) e = pl_launch<KV8, D, 3, false, true, true>(st, a, blocks);
      if (a.RP == 64) e = pl_launch<KV8, D, 4, false, true, true>(st, a, blocks);
    } else if (!a.stream) {   // (63 rows at most: 32 of a group)
      if (a.RP == 16) e = pl_launch<KV8, D, 1, false, true>(st, a, blocks);
      if (a.RP == 32) e = pl_launch<KV8, D, 2, false, true>(st, a, blocks);
    } else if (a.RP == 16) {   // (128 rows at most: with d = 1024 the decoder over the whole GPU takes them)
      e = pl_launch<KV8, D, 1, false>(st, a, blocks);
    }
  }
  if (a.stream) {
    if (a.RP == 32) e = pl_launch<KV8, D, 2, false>(st, a, blocks);
    if (a.RP == 48) e = pl_launch<KV8, D, 3, false>(st, a, blocks);
    if (a.RP == 64) e = pl_launch<KV8, D, 4, false>(st, a, blocks);
    if constexpr (D == 1024) {
      if (a.RP == 80) e = pl_launch<KV8, D, 5, false>(st, a, blocks);
      if (a.RP == 96) e = pl_launch<KV8, D, 6, false>(st, a, blocks);
    }
  }
  if (e != hipSuccess) return e;
  a.raised = a.err;
  a.err += 1;
  // (either kernel writes all of its row tiles of the residual, pl_resid_rows of them a group)
  constexpr int kTall = pl_resid_rows(pl_rows_most(D), D), kShort = pl_resid_rows(kPlRows, D);
  if (pl_resid_rows(a.RP, D) == kTall) return pl_launch<KV8, D, kTall / 16, true>(st, a, kPlMembers * std::min(a.G, 2));
  return pl_launch<KV8, D, kShort / 16, true>(st, a, kPlMembers * std::min(a.G, 2));
}
}  // namespace xcd
}  // namespace sd
