// What a pass of the per-XCD decoder (xcd_core.h) takes of a workspace, and what a workspace holds for the largest one within the limits of a
// context.  Arithmetic alone, without HIP, so that the two can be compared on any machine.
#pragma once
#include <algorithm>
#include <cstddef>

namespace sd {

// What the kernels that run a pass given up by tickets count with, ahead of the exchange buffers (all words ~0 when a pass
// starts): tickets drawn, and per stage the virtual workgroups that have finished it.
constexpr int kPlLayers = 32, kPlStages = 8;
struct PlTickets { unsigned drawn, done[kPlStages * kPlLayers]; };
constexpr size_t kPlTicketBytes = (sizeof(PlTickets) + 255) & ~size_t(255);
// Exchange buffers of one layer, rows padded to RP (PlExch)
constexpr size_t pl_layer_bytes(int RP, int d, int F) {
  return (size_t)RP * (3 * (2 * d + d / 2) + 6 * 2 * d + 2 * F);
}

namespace xcd {
constexpr int kPlGroups = 8;   // XCDs, and groups of sequences
// Rows of a group: what registers and LDS hold; of d = 512 from a copy of the weights (more are read in place); what the second run's smaller
// kernel takes.
constexpr int pl_rows_most(int d) { return d == 512 ? 160 : 96; }
constexpr int pl_copy_rows_most(int d) { return d == 512 ? 64 : 96; }
constexpr int kPlRows = 64;
inline int pl_group_rows(int B, int T) { return ((B + kPlGroups - 1) / kPlGroups * T + 15) & ~15; }
// Rows to a group of the second run's residual, all of which it writes: those of its kernel (of two, see pl_launch_both), not of the pass.
constexpr int pl_resid_rows(int RP, int d) { return RP > kPlRows ? pl_rows_most(d) : kPlRows; }
// Tickets, and exchange buffers of some layers (the pass uses those of two in turn) for every group.
inline size_t pl_exch_bytes(int B, int RP, int d, int F, int layers) { return kPlTicketBytes + (size_t)std::min(B, kPlGroups) * layers * pl_layer_bytes(RP, d, F); }
}  // namespace xcd

// T: places of a sequence; exch: bytes of exchange buffers; rows: of d floats each, twice, the last sum and the residual.
struct XcdRoom { int T; size_t exch; int rows; };

// Of a pass of B sequences of T places (rows 0: too many for it).
inline XcdRoom xcd_needs(int B, int T, int d, int F) {
  const int RP = xcd::pl_group_rows(B, T);
  if (RP > xcd::pl_rows_most(d)) return XcdRoom{T, 0, 0};
  return XcdRoom{T, xcd::pl_exch_bytes(B, RP, d, F, 2), std::min(B, xcd::kPlGroups) * xcd::pl_resid_rows(RP, d)};
}

// Of every pass within the limits: at d = 512 verification, drafting and prefill, else verification alone.  What a pass takes grows with its
// sequences and with its places, as far as there is a pass; it is asked for of the groups' rows, which a pass of few rows may have as many of
// as one of many (one sequence of 80 has as many as eight).
inline XcdRoom xcd_room(int max_batch, int k_max, int max_tgt, int d, int F) {
  const int most = xcd::pl_rows_most(d);
  XcdRoom r;
  r.T = d == 512 ? std::max(2 * k_max + 1, std::min(max_tgt + 1, most)) : k_max + 1;
  const int RP = std::min(xcd::pl_group_rows(max_batch, r.T), most);
  r.exch = xcd::pl_exch_bytes(max_batch, RP, d, F, 2);
  r.rows = std::min(max_batch, xcd::kPlGroups) * xcd::pl_resid_rows(RP, d);
  return r;
}

// Rows that the activation buffers of a decoder pass hold.  A prefill pass takes as many rows as make its products large (8192 rows: 150 MB of
// activations for the big model), never more than the streams can hold and never fewer than a verify / draft pass needs.
inline long decoder_pass_rows(int max_batch, int k_max, int max_tgt) {
  return std::max(std::min(max_batch * (long)(max_tgt + 1), 8192L), max_batch * (long)(2 * k_max + 1));
}

// Prefill of B streams of which at most `uncached` tokens each (no stream has more than max_tgt + 1, whatever the bound) are not cached: as few
// passes as the buffers allow, all of the same number of places.
struct PrefillPasses { int passes, T; };
inline PrefillPasses prefill_passes(int uncached, long pass_rows, int B, int max_tgt) {
  const int rows = std::min(uncached, max_tgt + 1), most = (int)(pass_rows / B);
  if (rows <= 0) return PrefillPasses{0, 0};
  const int passes = (rows + most - 1) / most;
  return PrefillPasses{passes, (rows + passes - 1) / passes};
}

}  // namespace sd
