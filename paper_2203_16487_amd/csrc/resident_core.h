// What the two decoders that run as one kernel share (persist.hip: over the whole GPU; xcd_core.h: each XCD on sequences of its own):
// words that are their own flags, and the buffers workgroups exchange them through.
#pragma once
#include "attn_core.h"
#include "xcd_room.h"

namespace sd {

constexpr unsigned kPoison = 0xffffffffu;   // "not there yet", in every 32-bit word of the exchange buffers when a pass starts
__device__ __forceinline__ unsigned not_poison(unsigned u) { return u == kPoison ? 0x7fc07fc0u : u; }   // (a NaN for a NaN)

// The kernels behind them, which run a pass given up by tickets (PlTickets).
constexpr unsigned kPlTicketSpinMax = 1u << 24;
constexpr unsigned kPlTicketPasses = 64;    // passes that go to it once waits were given up (a wait in vain then costs 2 - 5 ms a pass)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Coherent 16-byte load (past the L1; from memory, past this XCD's L2, where the stores go there): the buffer form with sc1.  (An inline-asm
// load would leave the compiler free to copy its result before it has arrived.)
typedef __amdgpu_buffer_rsrc_t PlBuf;
__device__ __forceinline__ PlBuf pl_buf(const void* p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffff, 0x00027000); }
constexpr int kPlSc1 = 16;
__device__ __forceinline__ u32x4 pl_request(PlBuf b, int voff, int soff) { return __builtin_amdgcn_raw_buffer_load_b128(b, voff, soff, kPlSc1); }

__device__ __forceinline__ u32x2 pl_pack4(const float (&v)[4]) {
  bf16x4 t;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = (bf16)v[i];
  return __builtin_bit_cast(u32x2, t);
}

// sums over the four 16-lane rows (lanes lq + 16 g), result in all of them
__device__ __forceinline__ float pl_row_sum(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return half_add(__builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]));
}

// The lane, as a value the compiler cannot carry over from an earlier stage: otherwise every stage's addresses are computed
// ahead of the layer loop and held (or spilled) throughout.
__device__ __forceinline__ int pl_lane() {
  int t = threadIdx.x & 63;
  asm volatile("" : "+v"(t));
  return t;
}

// The wave, likewise (the same for all of its lanes).
__device__ __forceinline__ int pl_wave() {
  int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  asm volatile("" : "+s"(w));
  return w;
}

// Exchange buffers of one layer (and group), all in tiles of 16 columns, [column / 16][RP][16]: what one item produces lies together and
// shares no line with another workgroup's stores (with rows of all columns side by side the 8- and 32-byte pieces of up to 16
// workgroups met in every line, and a residual sum took 3 us to become visible through memory instead of 1).  Statistics likewise,
// [chunk][RP] pairs.  (pl_layer_bytes of them.)
struct PlExch {   // (only the layer's base stays in registers)
  char* base;
  int row;        // bytes of a buffer of RP rows of d
  __device__ __forceinline__ PlExch(char* b, int RP, int d) : base(b), row(RP * 2 * d) {}
  __device__ __forceinline__ char* xg(int i) const { return base + i * row; }
  __device__ __forceinline__ char* q(int i) const { return base + (3 + i) * row; }
  __device__ __forceinline__ char* kx() const { return base + 5 * row; }
  __device__ __forceinline__ char* vx() const { return base + 6 * row; }
  __device__ __forceinline__ char* att(int i) const { return base + (7 + i) * row; }
  __device__ __forceinline__ char* st(int i) const { return base + 9 * row + i * (row >> 2); }
  __device__ __forceinline__ char* hid() const { return base + 9 * row + 3 * (row >> 2); }
};
// element (row, k) of a buffer, bytes
__device__ __forceinline__ int pl_at(int RP, int row, int k) { return ((k >> 4) * RP + row) * 32 + (k & 15) * 2; }

// Attention of one unit: 16 queries (the last ones of a sequence: fewer) of one (sequence, head) pair.
struct PlUnit {
  int b, h, q0, j, nkey;   // sequence (of the group), head, first query; keys cached before the pass (self-attention), all keys
};
// 1 / sqrt(64) and log2(e) meet the scores in the exponent.
constexpr float kCexp = 0.125f * 1.44269504088896341f;

// A chunk of 32 keys of one pair on a wave.  (What is done with it stands in both files: as functions shared here, in four ways, the same
// instructions came in another order, and a pass of 26 rows of d = 1024 with 8-bit weights took 229 - 233 us in place of 227.)
struct PlChunk {   // (one of the two forms)
  u32x4 kf[4], vf[4];
  fp8x8 kf8[4], vf8[4];
  f32x4 sck[2], scv[2];
};

}  // namespace sd
