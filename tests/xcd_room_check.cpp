// Host check of csrc/xcd_room.h, compiled and run by test_xcd_room.py: walks limits and passes and prints the first pass that takes more of a
// workspace than one made for the limits holds.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2203_16487_amd/csrc/xcd_room.h"

static long checked = 0;

static void check(const char* what, const sd::XcdRoom& room, int max_batch, int k_max, int max_tgt, int B, int T, int d, int F) {
  const sd::XcdRoom n = sd::xcd_needs(B, T, d, F);
  if (n.rows == 0) return;   // (launches)
  ++checked;
  // the second run writes every row of its kernel's tiles, of every group, and the last sum has the pass's rows
  const int groups = B < 8 ? B : 8, in_group = (B + 7) / 8 * T, written = groups * (in_group > 64 ? d == 512 ? 160 : 96 : 64);
  if (n.rows < written || n.rows < B * T || room.rows < n.rows || room.exch < n.exch) {
    printf("%s, d = %d, limits (%d, %d, %d), %d sequences of %d places: rows %d of %d, written %d, exchange %zu of %zu\n", what, d, max_batch, k_max,
           max_tgt, B, T, n.rows, room.rows, written, n.exch, room.exch);
    exit(1);
  }
}

int main() {
  std::vector<int> batches, tgts;
  for (int i = 1; i <= 40; ++i) batches.push_back(i);
  for (int i : {48, 63, 64, 65, 80, 96, 128, 129, 200, 1300}) batches.push_back(i);
  for (int i = 1; i <= 170; ++i) tgts.push_back(i);
  for (int i : {255, 256, 1024}) tgts.push_back(i);
  for (int d : {512, 1024})
    for (int max_batch : batches)
      for (int k_max : {1, 2, 3, 7, 10, 16, 25, 31})
        for (int max_tgt : tgts) {
          const sd::XcdRoom room = sd::xcd_room(max_batch, k_max, max_tgt, d, 4 * d);
          for (int B = 1; B <= max_batch && B <= 1280; B += B < 64 ? 1 : 61) {
            for (int T = 1; T <= k_max + 1; ++T) check("verify", room, max_batch, k_max, max_tgt, B, T, d, 4 * d);
            if (d != 512) continue;
            for (int T = k_max + 2; T <= 2 * k_max + 1; ++T) check("draft", room, max_batch, k_max, max_tgt, B, T, d, 4 * d);
            // (the bound on what is not cached grows with every commit, beyond what a stream can have)
            const long pass_rows = sd::decoder_pass_rows(max_batch, k_max, max_tgt);
            for (int uncached = 1; uncached <= 2 * max_tgt + 160; uncached += uncached < 200 ? 1 : 37) {
              const sd::PrefillPasses p = sd::prefill_passes(uncached, pass_rows, B, max_tgt);
              if (p.T < 1 || (long)p.T * B > pass_rows || p.T > max_tgt + 1 || p.T * p.passes < (uncached < max_tgt + 1 ? uncached : max_tgt + 1)) {
                printf("prefill of %d, limits (%d, %d, %d), %d sequences: %d passes of %d\n", uncached, max_batch, k_max, max_tgt, B, p.passes, p.T);
                exit(1);
              }
              check("prefill", room, max_batch, k_max, max_tgt, B, p.T, d, 4 * d);
            }
          }
        }
  printf("%ld passes\n", checked);
  return checked > 1000000 ? 0 : 1;
}
