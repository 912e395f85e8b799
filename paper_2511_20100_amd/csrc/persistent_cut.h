// Which decode steps run as one launch, and how that one is cut.  Host code only.
#pragma once

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

}  // namespace bf16
}  // namespace mtmc
