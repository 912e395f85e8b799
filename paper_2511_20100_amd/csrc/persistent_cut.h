// Which decode steps run as one launch, and how that one is cut.  Host code only.
#pragma once

#include <stddef.h>

namespace mtmc {
namespace bf16 {

constexpr int kPersistGrid = 256;        // workgroups, all resident at once: one per CU

struct PersistShape {
  int m_tiles, head_dim, kt_d, nt_d, nt_qkv, nt_gu, n_chunks, pairs;  // pairs: sequences x kv heads
  int down_nb, ks_down;  // the down projection's own launch: row tiles per workgroup (2, 3 or 4), which tells its ranges of K, and splits
};

// Gate / up row tiles per workgroup: one round on the 256 CUs with the ranges of K of the launch of its own.
inline int persist_gu_tiles(int nt_gu) { return nt_gu <= 4 * 256 ? 4 : nt_gu <= 6 * 256 ? 6 : nt_gu <= 10 * 256 ? 10 : 0; }
// Ranges of K of the down projection, and the row tiles that a workgroup has of one of its splits.
inline int persist_dn_ranges(int down_nb) { return down_nb == 3 ? 5 : down_nb == 2 ? 8 : 4; }
inline int persist_dn_tiles(int dn_ranges) { return dn_ranges == 5 ? 3 : dn_ranges == 8 ? 2 : 4; }

// More than one tile of rows: 6 row tiles x 64 rows or 10 x 32 are what the accumulators hold.  Each cut is an instance of its own,
// and these are built: d 1536 with feed-forward widths of 8208 to 12288, and to 32 rows those of 10 gate / up tiles with 4 ranges of
// the down projection (d 3584, F 18944).  Other widths that would fit the registers (d 2048, F 11008: 6 tiles and 8 ranges) run
// separate launches from 17 rows on.
inline bool persist_rows_fit(int bt, int gu_tiles, int dn_ranges) {
  return bt == 2 ? (gu_tiles == 6 && dn_ranges == 5) || (gu_tiles == 10 && dn_ranges == 4)
                 : (bt == 3 || bt == 4) && gu_tiles == 6 && dn_ranges == 5;
}

inline bool decode_persistent_fits(const PersistShape& s) {
  const int gu = persist_gu_tiles(s.nt_gu), dn = persist_dn_ranges(s.down_nb), tiles = persist_dn_tiles(dn);
  // 16 ranges of K in the QKV projection (d from 1536), matrices within a descriptor's reach, a row tile of the sum of the
  // splits per workgroup, a unit of the attention per workgroup
  if (s.head_dim != 128 || s.kt_d < 48 || s.nt_d > kPersistGrid || s.nt_qkv > 4096 || s.n_chunks > 8 ||
      s.pairs * s.n_chunks > kPersistGrid || gu == 0)
    return false;
  // one (group of row tiles, split) of the down projection per workgroup: not so in the smaller last group of a call of many
  // sequences, which keeps the splits that were chosen for 128 rows
  const bool down = dn == 5 ? s.ks_down == 8 && s.nt_d <= 96 : s.ks_down * ((s.nt_d + tiles - 1) / tiles) <= kPersistGrid;
  return down && (s.m_tiles == 1 || persist_rows_fit(s.m_tiles, gu, dn));
}

// Steps of so few rows hand their data to readers that ask for them (decode_persistent.hip).
constexpr int kPersistAskRows = 2;
// Steps of more rows in which readers ask for some of it (persist_hand_rows()): not with 10 gate / up tiles and several tiles of rows
// (decode_persistent_rows.hip, kAsks), which need no memory for that.
constexpr bool persist_some_ask(int bt, int gu_tiles) { return bt == 1 || gu_tiles == 6; }
// What the phases of such a step hand on: a piece of memory per block (block l: l % kPersistPieces), in which every buffer has the
// rows of the batch and no others (bytes from the piece's start).  What all workgroups ask for is there kPersistCopies times, a copy
// for the workgroups of a die.
//
// Readers ask until a word is no longer the one that says that nobody has written it.  The first two pieces are filled with that word
// before the step.  Later, who writes a place in one block (always the same wavefront) first puts the word into the place of the
// block behind it and waits for that store.  So
//   - whoever asks for a place has seen what was written to it in the block before, and with that the word was there;
//   - what the word goes over is of three blocks before, and its readers are done.  Every writer has asked for something in the
//     same phase one block earlier (a unit of the attention without a part of the context, too), and each phase's data come, one
//     phase after the other, of all that was read in the phases of a whole block before.  x, ss0 and the ss1 of the block before are
//     read one block later than the others: x and ss0 are marked at the end of a block, behind an O projection that came of them
//     all, ss1 behind the sum of the splits.
// The second point needs a store of the workgroup behind everything that one of its wavefronts has asked for, in the same phase: of its
// own, or behind a barrier that it takes part in.
constexpr int kPersistCopies = 8, kPersistPieces = 3;
// A unit of the attention whose chunk holds no part of the context stores zeros, 16 threads per query head, without such a barrier: only
// wavefronts that store ask for the rows of qkv.
constexpr bool persist_empty_unit_asks(int wave, int heads) { return wave * 64 < heads * 16; }
struct PersistHand {
  int x, xo, act, qkv, o, ml, part, ss0, ss1;  // x, ss0: of the block before it; o, ml: chunk by chunk, o_chunk bytes apart
  int x_copy, ss_copy, qkv_copy, o_chunk, bytes;
};
// What a step of more rows hands to readers that ask for it: the rows of qkv (block l: buffer l % 2) and the sums of
// the splits.  Filled with the word before the step.  Whoever writes a row of qkv marks its place in the other buffer a block ahead,
// whoever adds up the splits marks what it has read; several waits of all workgroups lie between either and the next write.
inline PersistHand persist_hand_rows(int bt, int kt_d, int nt_qkv, int ks_down) {
  PersistHand h{};
  h.qkv_copy = bt * 16 * nt_qkv * 64;
  h.part = 2 * h.qkv_copy;
  h.bytes = h.part + bt * 16 * kt_d * 128 * ks_down;
  return h;
}
inline PersistHand persist_hand(int B, int kt_d, int kt_F, int nt_qkv, int kt_nq, int heads, int n_chunks, int ks_down) {
  PersistHand h{};
  auto take = [&](int n) {
    const int at = h.bytes;
    h.bytes += (n + 127) / 128 * 128;
    return at;
  };
  h.x_copy = (B * kt_d * 64 + 4095) / 4096 * 4096;
  h.ss_copy = B * kPersistGrid * 4;
  h.x = take(kPersistCopies * h.x_copy);
  h.xo = take(kPersistCopies * h.x_copy);
  h.act = take(B * kt_F * 64);
  h.qkv = take(B * nt_qkv * 64);
  h.o_chunk = B * kt_nq * 64;
  h.o = take(n_chunks * h.o_chunk);
  h.ml = take(B * heads * n_chunks * 8);
  h.part = take(B * kt_d * 128 * ks_down);
  h.ss0 = take(kPersistCopies * h.ss_copy);
  h.ss1 = take(kPersistCopies * h.ss_copy);
  return h;
}

}  // namespace bf16
}  // namespace mtmc
