// What the one-launch step of few rows hands from phase to phase: every buffer in its place, none over another, all on 128 bytes.
// Compiled and run by test_few_rows.py; exits non-zero at the first shape that does not hold.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "persistent_cut.h"

using namespace mtmc::bf16;

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s (B %d kt_d %d)\n", __LINE__, #x, B, kt_d); std::exit(1); } } while (0)

int main() {
  for (int B = 1; B <= kPersistAskRows; ++B)
    for (int kt_d : {48, 50, 112, 128})
      for (int kt_F : {1, 16, 35, 280, 640})
        for (int kv : {1, 4, 32})
          for (int chunks = 1; chunks <= 8; ++chunks)
            for (int ks : {1, 4, 8, 40}) {
              const int heads = 32, kt_nq = heads * 4, nt_qkv = (heads + 2 * kv) * 8;
              const PersistHand h = persist_hand(B, kt_d, kt_F, nt_qkv, kt_nq, heads, chunks, ks);
              const long need[][2] = {{h.x, (long)kPersistCopies * h.x_copy}, {h.xo, (long)kPersistCopies * h.x_copy}, {h.act, B * kt_F * 64L},
                                      {h.qkv, B * nt_qkv * 64L}, {h.o, (long)chunks * h.o_chunk}, {h.ml, B * heads * chunks * 8L},
                                      {h.part, (long)ks * B * kt_d * 32 * 4}, {h.ss0, (long)kPersistCopies * h.ss_copy},
                                      {h.ss1, (long)kPersistCopies * h.ss_copy}};
              CHECK(h.x_copy >= B * kt_d * 64 && h.o_chunk == B * kt_nq * 64 && h.ss_copy >= B * kPersistGrid * 4);
              long end = 0;
              for (auto& n : need) {
                CHECK(n[0] % 128 == 0 && n[0] >= end);
                end = n[0] + n[1];
              }
              CHECK(kPersistPieces == 3 && end <= h.bytes && h.bytes % 128 == 0 && h.x_copy % 128 == 0 && h.o_chunk % 16 == 0 && h.ss_copy % 4 == 0);
            }
  for (int bt = 1; bt <= 4; ++bt)
    for (int kt_d : {48, 50, 112, 128})
      for (int ks : {1, 4, 8, 40}) {
        const int B = bt * 16, nt_qkv = 2 * kt_d + 32;
        const PersistHand h = persist_hand_rows(bt, kt_d, nt_qkv, ks);
        CHECK(h.qkv == 0 && h.qkv_copy >= B * nt_qkv * 16 * 4 && h.part >= 2 * h.qkv_copy && h.part % 128 == 0 && h.qkv_copy % 128 == 0);
        CHECK(h.bytes >= h.part + ks * B * kt_d * 32 * 4);
      }
  // one tile of rows always has memory for readers that ask, several with the cuts whose readers do
  for (int bt = 1; bt <= 4; ++bt)
    for (int gu : {4, 6, 10}) {
      const int B = 0, kt_d = gu;
      CHECK(persist_some_ask(bt, gu) == (bt == 1 || gu == 6));
    }
  std::printf("ok\n");
  return 0;
}
