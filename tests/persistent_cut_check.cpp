// Every shape that takes the one-launch decode step: its workgroups share out all the work there is.  Compiled and run by
// test_persistent_turn.py; exits non-zero at the first shape that does not hold.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "persistent_cut.h"

using namespace mtmc::bf16;

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (nt_d %d ks %d nb %d bt %d)\n", __LINE__, #x, s.nt_d, s.ks_down, s.down_nb, s.m_tiles); std::exit(1); } } while (0)

// The (row tile, split) pairs of the down projection, as its workgroups take them: once each.
static void down_projection(const PersistShape& s) {
  const int dn = persist_dn_ranges(s.down_nb), tiles = persist_dn_tiles(dn);
  std::vector<int> taken((size_t)s.nt_d * s.ks_down);
  for (int wg = 0; wg < kPersistGrid; ++wg)
    for (int j = 0; j < tiles; ++j) {
      const int split = dn == 5 ? wg & 7 : wg % s.ks_down;
      const int tile = dn == 5 ? (wg >> 3) + kPersistGrid / 8 * j : wg / s.ks_down * tiles + j;
      if (tile >= s.nt_d) continue;
      CHECK(split < s.ks_down);
      ++taken[(size_t)tile * s.ks_down + split];
    }
  for (int n : taken) CHECK(n == 1);
}

int main() {
  long fits = 0, all = 0;
  for (int nt_d = 90; nt_d <= 260; ++nt_d)
    for (int down_nb = 2; down_nb <= 4; ++down_nb)
      for (int ks = 1; ks <= 40; ++ks)
        for (int nt_gu : {32, 1024, 1026, 1536, 1538, 2560, 2562})
          for (int bt = 1; bt <= 5; ++bt) {
            const PersistShape s{bt, 128, nt_d / 2, nt_d, nt_d + 32, nt_gu, 1, 16 * bt, down_nb, ks};
            ++all;
            if (!decode_persistent_fits(s)) continue;
            ++fits;
            down_projection(s);
            const int gu = persist_gu_tiles(nt_gu);
            CHECK(gu * kPersistGrid >= nt_gu && nt_d <= kPersistGrid && bt <= 4);
            if (bt > 1) {  // the O projection has a unit per workgroup
              const int o_tiles = bt == 2 && gu == 6 ? 1 : 2;
              CHECK((nt_d + o_tiles - 1) / o_tiles * bt <= kPersistGrid);
            }
          }
  const PersistShape s{};
  CHECK(fits > 1000 && fits < all / 2);
  // the shapes that are there: 1.5 B class (64 and 32 rows, one row), 7 B class (32 rows); and with the splits of 128 rows
  CHECK(decode_persistent_fits({4, 128, 48, 96, 128, 1120, 2, 128, 3, 8}) && decode_persistent_fits({1, 128, 48, 96, 128, 1120, 8, 2, 3, 8}));
  CHECK(decode_persistent_fits({2, 128, 112, 224, 288, 2368, 1, 128, 4, 4}));
  CHECK(!decode_persistent_fits({1, 128, 48, 96, 128, 1120, 1, 2, 4, 21}) && !decode_persistent_fits({2, 128, 112, 224, 288, 2368, 1, 128, 4, 9}));
  // row tiles of a workgroup and ranges of the down projection of the widths that test_gpu_persistent_given_up.py names after them
  struct { int gu, dn, F, down_nb; } named[] = {{4, 5, 6144, 3}, {4, 4, 8192, 4}, {6, 8, 11008, 2}, {6, 4, 12288, 4}, {10, 5, 16384, 3}, {10, 8, 14336, 2}};
  for (auto& n : named) CHECK(persist_gu_tiles(n.F / 8) == n.gu && persist_dn_ranges(n.down_nb) == n.dn);
  std::printf("ok\n");
  return 0;
}
