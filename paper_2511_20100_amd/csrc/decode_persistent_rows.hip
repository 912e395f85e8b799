// The persistent decode step for two to four tiles of 16 rows (17 to 64 rows); see decode_persistent.hip for the one-tile form,
// for what a persistent step saves and for what it asks of the device.
//
// What bounds it: a CU takes in about 50 GB/s, weights from memory or operand from the cache.  At 64 rows the gate / up phase
// needs 192 KB of operand beside 288 KB of weights per CU, 9 of a block's 56 us; in all a block spends 20 us on its six
// hand-overs (stores drained 1 us, counters 1.5, stragglers), 10 on sums and epilogues, 26 on streams.  So the operand is
// taken in as seldom as registers allow: the gate / up projection holds 6 row tiles x 64 rows in accumulators, which takes 256
// registers and hence eight wavefronts in all (with the twelve of the one-tile form, two sets of workgroups per row tile,
// 64 rows took 133 ms).  They stream, multiply, sum and store; one of them watches the counters, and asks for its share of
// the next weights behind that (loads return in order).  Two or three k tiles in flight make no difference at 64 rows.
//
// (Since the rows of qkv and the sums of the splits are asked for, kAsks below, it is 51 of which four hand-overs are counted.)
//
// 63 steps of the 1.5 B shape, separate launches -> this, all counted: 32 rows 100.2 -> 94.2 ms, 64 rows 120.5 -> 114.8; 31 steps of 48
// rows 62.2 -> 56.6; cached step of the 7 B shape (4 blocks, 8192 tokens, 32 rows, 47 steps) 46.5 -> 44.0.
#include <type_traits>

#include "decode_persistent.h"
#include "kernels.h"

namespace mtmc {
namespace bf16 {
namespace persist {
namespace {

constexpr int kWaves = AW, kThreads = kWaves * 64;
constexpr int kWatch = kWaves - 1;  // the wavefront that counts the workgroup in and watches the counters
// sums of 16 x 16 values that a phase hands over at once, by what the LDS holds beside them
template <int GU_TILES>
constexpr int kItems = GU_TILES == 6 ? 96 : 80;

// BT tiles of 16 rows.  A unit of the QKV projection is kQkvTiles row tiles and kUnit tiles of rows; one of the O projection
// kOTiles row tiles and one tile of rows: the attention's output comes past the caches, in several chunks.  Such that the
// units are one round on the 256 CUs (d 1536: 128 and 96 row tiles; d 3584: 288 and 224).
template <int BT, int GU_TILES>
constexpr int kQkvTiles = GU_TILES == 6 ? 1 : 2;
template <int BT, int GU_TILES>
constexpr int kUnit = GU_TILES == 6 ? (BT + 1) / 2 : BT;
template <int BT, int GU_TILES>
constexpr int kOTiles = BT == 2 && GU_TILES == 6 ? 1 : 2;

template <int BT, int GU_TILES, int NT>
struct Shared {
  union {
    v4f red[kItems<GU_TILES>][64];  // sums per range of K, as the accumulators lie in the lanes
    AttnLds at;
  };
  int table[ATAB];  // page ids of the attention unit
  float squares[16 * BT][NT + 4];  // sums of squares of a row's tiles
  union {
    float squares_old[16 * BT][NT + 4];  // ... of the residual that the operand was divided by
    struct {
      float ml[kWaves][2][8][16];     // O projection: per wavefront, head in hand, chunk and row: the chunk's rescaled sum
      float share[kWaves][2][8][16];  // ... and its share
    };
  };
  float total[2][16 * BT];  // sums of the rows' squares: now, and of the older residual
  int stop;
};

// The sums of ROWS rows' squares by one wavefront, as a launch of W wavefronts per workgroup makes them: such a launch (64 W
// threads over 16 BT rows) adds P = 64 W / (16 BT) partial sums of the row's tiles (part p: tiles p, p + P, ...) in order.
// load() asks for all tiles at once (they lie side by side, kPersistGrid floats a row), finish() adds.
template <int ROWS, int NT>
struct RowSums {
  static constexpr int L = 64 / ROWS, N = (NT / 4 + L - 1) / L;  // lanes a row, loads a lane
  v4f v[N];

  __device__ __forceinline__ static int quad(int j, int lane) { return min(lane % L + L * j, NT / 4 - 1); }
  __device__ __forceinline__ void load(const float* ss, int row0, int lane) {
    const Rsrc r = rsrc_of(ss);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = ld16f(r, ((row0 + lane / L) * kPersistGrid + quad(j, lane) * 4) * 4, 0);
  }
  __device__ __forceinline__ void finish(float (*squares)[NT + 4], float* total, int row0, int nt_d, int P, int lane) {
    float* row = squares[row0 + lane / L];
#pragma unroll
    for (int j = 0; j < N; ++j) *reinterpret_cast<v4f*>(&row[quad(j, lane) * 4]) = v[j];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows are the wavefront's own
    for (int p = lane % L; p < min(P, nt_d); p += L) {
      float part = 0.f;
#pragma unroll 4
      for (int t = p; t < nt_d; t += P) part += row[t];
      row[p] = part;  // nobody else reads tile p
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    float sum = 0.f;
#pragma unroll 8
    for (int p = 0; p < min(P, nt_d); ++p) sum += row[p];
    if (lane % L == 0) total[row0 + lane / L] = sum;
  }
};

// Whether the attention asks for the rows of qkv and whoever adds up the splits for their sums, each of which has few readers, until they
// are there: two of six times that a block does not drain stores and count (23 steps of the 1.5 B shape behind 200 tokens: 64 rows
// 43.3 -> 41.0 ms, 48 rows 39.6 -> 38.0, 32 rows 35.3 -> 32.9).  Not with 10 gate / up tiles, whose registers are full: the loops
// cost 10 more in scratch, and four 7 B blocks with 32 rows took 17.76 ms instead of 17.58.
template <int GU_TILES>
constexpr bool kAsks = persist_some_ask(2, GU_TILES);
// The rows of qkv in block l, and the sums of the splits (persist_hand_rows()).
template <bool ASK>
__device__ __forceinline__ float* qkv_of(const PersistArgs& a, int l) {
  return ASK ? (float*)(a.hand + (l & 1) * a.at_hand.qkv_copy) : a.qkv;
}
template <bool ASK>
__device__ __forceinline__ float* part_of(const PersistArgs& a) { return ASK ? (float*)(a.hand + a.at_hand.part) : a.part; }

// An attention unit that asks for its rows of qkv; enter() as in CountedUnit.
template <class Enter>
struct AskingUnit : CountedUnit<Enter> {
  int l;
  int* stop;
  __device__ __forceinline__ AskingUnit(int Mpad, Enter e, int l_, int* stop_) : CountedUnit<Enter>{Mpad, e}, l(l_), stop(stop_) {}
  __device__ __forceinline__ const float* qkv(const PersistArgs& a) const { return keep(qkv_of<true>(a, l)); }
  template <class Load>
  __device__ __forceinline__ bool operator()(const PersistArgs& a, Load load) const {
    if (!this->enter()) return false;
    Asker{a, stop}(load);
    return true;
  }
};

// wait_grid() behind the first phase: the roll call.  The watch's first look comes back behind its keys and values: if that took longer
// than the limit, callers who have set one are told, also where all are there by then.
__device__ __forceinline__ bool answer_roll(const Ctx& c) {
  const Word mine = word_of(c.a, c.wg % kPersistTops), ended = word_of(c.a, kPersistEnded), before = {c.a.sync + kPersistGaveUp};
  const long long t0 = wall_clock64();
  long long limit = c.a.roll_ticks;
  for (int i = 0;; ++i) {
    const bool there = look(mine) >= kPersistGroups;
    if (wall_clock64() - t0 <= limit) {
      if (there) break;
      if (i % 16 == 15) {
        if (look(ended)) return false;
        if (look(before)) limit = min(limit, kAgainTicks);
      }
      continue;
    }
    if (give_up(c)) return false;
    limit = kWaitTicks;  // every group is full: the last of them are about to say so
  }
  asm volatile("" ::: "memory");
  return true;
}

// GU_TILES row tiles of the gate / up projection per workgroup, 8 ranges of K, one per wavefront; the sums go over in rounds of
// kGroup tiles of 16 rows.
template <int BT, int GU_TILES>
struct GuCut {
  static constexpr int kGroup = kItems<GU_TILES> / (8 * GU_TILES) < BT ? kItems<GU_TILES> / (8 * GU_TILES) : BT;
  static constexpr int kRounds = (BT + kGroup - 1) / kGroup;
  // weights and operand ahead, in k tiles
  static constexpr int kAhead = BT == 2 ? (GU_TILES == 6 ? 4 : 2) : BT == 3 ? 3 : 2;
};

template <int BT, int GU_TILES, int DN_RANGES, int NT>
__device__ __forceinline__ void step(Shared<BT, GU_TILES, NT>& sh, int wave) {
  constexpr int MU = kUnit<BT, GU_TILES>, NP = (BT + MU - 1) / MU, QT = kQkvTiles<BT, GU_TILES>, OT = kOTiles<BT, GU_TILES>;
  using Gu = GuCut<BT, GU_TILES>;
  constexpr bool ASK = kAsks<GU_TILES>;
  const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
  const bool watches = wave == kWatch;
  uint32_t phase = 0;
  // Into the next phase: the watch waits until every workgroup has left the last one.  prefetch() asks for what does not depend on
  // it; false: the launch ends here.
  auto enter = [&](auto prefetch) {
    if (watches && phase > 0 && !wait_grid(fresh(wave), phase)) sh.stop = 1;
    prefetch();
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(sh.stop) == 0;
  };
  // Out of it: what the workgroup has stored is where others see it, and that has been counted before anybody asks for more (a
  // CU's memory requests are served in order).
  auto leave = [&] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (watches) {
      const Ctx c = fresh(wave);
      if (c.lane == 0) count_in(c, phase);
    }
    lds_barrier();
    ++phase;
  };
  // Out of a phase whose readers ask for what it gives.
  auto leave_asked = [&] {
    if constexpr (ASK) lds_barrier();
    else leave();
  };
  const v4u none = v4u{kNotThere, kNotThere, kNotThere, kNotThere};
  auto loads_done = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  const int n_layers = fresh(wave).a.n_layers;
  const Ctx first = fresh(wave);
  const AttnHeld unit(first.a, first.wg, wave, first.lane, sh.table, 16 * BT);
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection: 16 (or 8) ranges of K, two (or one) per wavefront
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, lane = c.lane, rq = (lane >> 4) * 4;
      const h16_t* const W = a.wqkv + (size_t)l * a.layer_stride / sizeof(h16_t);
      const h16_t* const x = keep(x_of(a, l));
      const Rsrc out = rsrc_of(keep(qkv_of<ASK>(a, l))), behind = rsrc_of(keep(qkv_of<ASK>(a, l + 1)));
      const int kt_d = keep(a.kt_d), nt_qkv = keep(a.nt_qkv), nt_d = keep(a.nt_d), B = keep(a.B), ranges = keep(a.qkv_ranges);
      const int units = (nt_qkv + QT - 1) / QT * NP, per = (kt_d + ranges - 1) / ranges;
      Stream<QT, MU, 3, 3> s0, s1;
      int u = c.wg;
      auto start = [&] {
        int rows[QT];
#pragma unroll
        for (int i = 0; i < QT; ++i) rows[i] = min(min(u, units - 1) / NP * QT + i, nt_qkv - 1) * kt_d * 1024;
        s0.start(rsrc_of(W), rows, w * per, min(per, kt_d - w * per), 0, 0, kt_d - 1, lane);
        s1.start(rsrc_of(W), rows, (w + 8) * per, min(per, kt_d - (w + 8) * per), 0, 0, kt_d - 1, lane);  // empty with 8 ranges
      };
      if (!enter(start)) return;
      for (int i = 0; u < units;) {
        const int mt0 = u % NP * MU, base = (i & 1) * ranges * QT * MU;
        const auto xr = Operand<MU>::tiled(x, BT, mt0, lane, B);
        // the rows' sums: of the residual that is (wavefronts 0 .. 3) and of the one that x was divided by
        RowSums<4 * MU, NT> rs;
        const int row0 = mt0 * 16 + w % 4 * (4 * MU);
        const bool sums = l > 0 && row0 < 16 * BT;  // the second half of three tiles is one
        if (sums) rs.load(a.ss_in[w / 4], row0, lane);
        s0.operands(xr);
        s1.operands(xr);
        if (sums) rs.finish(w / 4 ? sh.squares_old : sh.squares, sh.total[w / 4], row0, nt_d, 4 * ranges / BT, lane);
        v4f a0[QT][MU], a1[QT][MU];
        clear(a0);
        clear(a1);
        s0.run(xr, 0, s0.n, a0);
        s1.run(xr, 0, s1.n, a1);
#pragma unroll
        for (int t = 0; t < QT * MU; ++t) sh.red[base + w * (QT * MU) + t][lane] = a0[t / MU][t % MU];
        if (ranges > 8) {
#pragma unroll
          for (int t = 0; t < QT * MU; ++t) sh.red[base + (w + 8) * (QT * MU) + t][lane] = a1[t / MU][t % MU];
        }
        lds_barrier();
        if (w < QT * MU) {
          const int m = (mt0 + w % MU) * 16 + (lane & 15), nt = u / NP * QT + w / MU;
          v4f sum = zero;
          if (ranges == 8) add_ranges<8>(sum, sh.red, base + w, QT * MU, lane);
          else add_ranges<16>(sum, sh.red, base + w, QT * MU, lane);
          const int row = min(m, 16 * BT - 1);
          const float sc = l > 0 ? scale_of(sh.total[0][row], sh.total[1][row], true, a.inv_d, a.eps) : 1.f;
          if (m < B && nt < nt_qkv) {
            const int off = ((m * nt_qkv + nt) * 16 + rq) * 4;
            st16(out, off, 0, written(sum * sc));
            if (ASK) st16(behind, off, 0, none);  // the units of the block before have read it
          }
        }
        u += kPersistGrid;
        ++i;
        if (u >= units) break;
        start();
      }
      if (l == 0) leave();
      else leave_asked();
    }
    // ---- attention; the first one is behind the roll call
    auto enter_attention = [&] {
      if (ASK && l > 0) return true;
      if (watches) {
        const Ctx c = fresh(wave);
        if (!(l == 0 ? answer_roll(c) : wait_grid(c, phase))) sh.stop = 1;
      }
      lds_barrier();
      return __builtin_amdgcn_readfirstlane(sh.stop) == 0;
    };
    if (!unit.active) {
      if (!enter_attention()) return;
    } else {
      if constexpr (ASK) {
        if (!attend<true>(unit, sh.at, sh.table, l, wave, AskingUnit<decltype(enter_attention)>(16 * BT, enter_attention, l, &sh.stop))) return;
      } else {
        if (!attend<true>(unit, sh.at, sh.table, l, wave, counted_unit(16 * BT, enter_attention))) return;
      }
    }
    leave();
    // ---- O projection: at most one unit per workgroup
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, lane = c.lane, rq = (lane >> 4) * 4, kt_nq = keep(a.kt_nq), B = keep(a.B), nt_d = keep(a.nt_d);
      const int units = (nt_d + OT - 1) / OT * BT, u = min(c.wg, units - 1), nt0 = u / BT * OT, mt = u % BT;
      const h16_t* const W = a.wo + (size_t)l * a.layer_stride / sizeof(h16_t);
      const h16_t* const o = keep(a.at.o);
      const float* const ml = keep(a.at.ml);
      const TileOut to(a, a.xo + (size_t)l * a.x_stride, 1, l + 1 == n_layers);
      const float* const gp = (const float*)((const char*)a.ffn_norm + l * a.layer_stride);
      const int R = keep(a.o_ranges), NC = keep(a.at.n_chunks), n_heads = keep(a.at.Hq);
      const int chunk_bytes = (int)(a.at.o_chunk_stride * sizeof(h16_t));
      // this wavefront's list of heads behind a split context: range v takes heads v, v + R, ...; ranges w and (12 ranges) w + 8
      const int per0 = max((n_heads - w + R - 1) / R, 0);
      const int per1 = (R > 8 && w + 8 < R) ? max((n_heads - (w + 8) + R - 1) / R, 0) : 0;
      const int n_e = per0 + per1, per = (kt_nq + R - 1) / R;
      auto head_of = [&](int e0) {  // entry e0 of the list; past its end the last one again
        const int e = min(e0, n_e - 1);
        return max(0, e < per0 ? w + e * R : w + 8 + (e - per0) * R);
      };
      v4f h_old = zero, gain = zero;
      auto preload = [&] {  // wavefronts 0 .. OT - 1 finish a tile each
        const int m = mt * 16 + (lane & 15), nt = min(nt0 + min(w, OT - 1), nt_d - 1);
        h_old = ld16f(to.h, (min(m, B - 1) * to.d + nt * 16 + rq) * 4, 0);
        gain = *reinterpret_cast<const v4f*>(gp + nt * 16 + rq);
      };
      auto row_sums = [&] {  // two rows per wavefront
        RowSums<2, NT> rs;
        rs.load(a.ss_in[0], mt * 16 + w * 2, lane);
        rs.finish(sh.squares, sh.total[0], mt * 16 + w * 2, nt_d, 4 * R / BT, lane);
      };
      auto finish = [&] {
        lds_barrier();
        if (w < OT && nt0 + w < nt_d) {
          loads_done();
          v4f sum = zero;
          if (R == 16) add_ranges<16>(sum, sh.red, w, OT, lane);
          else if (R == 12) add_ranges<12>(sum, sh.red, w, OT, lane);
          else add_ranges<8>(sum, sh.red, w, OT, lane);
          residual_tile<BT>(to, nt0 + w, mt, lane, sum, h_old, gain,
                            scale_of(sh.total[0][mt * 16 + (lane & 15)], 0.f, false, a.inv_d, a.eps));
        }
      };
      auto row_tile = [&](int i) { return min(nt0 + i, nt_d - 1) * kt_nq; };  // its first k tile
      const auto xr = Operand<1, kDeviceScope>::tiled(o, BT, mt, lane, B);
      if (c.wg >= units) {
        if (!enter([] {})) return;
      } else if (NC == 1) {
        Stream<OT, 1, 3, 3> s0, s1;
        auto start = [&] {
          int rows[OT];
#pragma unroll
          for (int i = 0; i < OT; ++i) rows[i] = row_tile(i) * 1024;
          preload();
          s0.start(rsrc_of(W), rows, w * per, min(per, kt_nq - w * per), 0, 0, kt_nq - 1, lane);
          s1.start(rsrc_of(W), rows, (w + 8) * per, min(per, kt_nq - (w + 8) * per), 0, 0, kt_nq - 1, lane);  // empty with 8 ranges
        };
        if (!enter(start)) return;
        v4f a0[OT][1], a1[OT][1];
        clear(a0);
        clear(a1);
        s0.operands(xr);
        s1.operands(xr);
        row_sums();
        s0.run(xr, 0, s0.n, a0);
        s1.run(xr, 0, s1.n, a1);
#pragma unroll
        for (int k = 0; k < OT; ++k) {
          sh.red[w * OT + k][lane] = a0[k][0];
          sh.red[(w + 8) * OT + k][lane] = a1[k][0];
        }
        finish();
      } else {
        // The chunks of the context are combined here, head by head: out += sum_chunk share * (W_head . o_chunk), share =
        // l exp(m - max m) / sum l exp(m - max m); two heads in hand at a time, 4 or 6 (head, chunk) operands on their way.
        constexpr int kItemsAhead = OT == 1 ? 6 : 4;
        const int col = lane & 15, lg = lane >> 4;
        const Rsrc wr = rsrc_of(W);
        v8h wf[2][4][OT];
        auto load_heads = [&](int e0) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
              for (int k = 0; k < OT; ++k)
                wf[i][t][k] = load_weight(wr, e0 + i < n_e ? lane * 16 : kReach, (row_tile(k) + head_of(e0 + i) * 4 + t) * 1024);
        };
        auto start = [&] {
          preload();
          load_heads(0);
        };
        if (!enter(start)) return;
        v4f acc[OT];
#pragma unroll
        for (int k = 0; k < OT; ++k) acc[k] = zero;
        for (int e0 = 0; e0 < n_e; e0 += 2) {
          if (e0) load_heads(e0);
          // chunk statistics of the two heads: lane (row, lg) has chunks lg and lg + 4
          uint2 st[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k)
              st[i][k] = ld8(ml + (((size_t)min(mt * 16 + col, B - 1) * n_heads + head_of(e0 + i)) * NC + min(lg + 4 * k, NC - 1)) * 2);
          const int n_items = min(2, n_e - e0) * NC;
          v8h xf[kItemsAhead][4];
          auto load_items = [&](int i0) {
#pragma unroll
            for (int q = 0; q < kItemsAhead; ++q) {
              const int i = min(i0 + q, n_items - 1), h = i >= NC ? 1 : 0;
              const int off = (i - h * NC) * chunk_bytes + head_of(e0 + h) * 4 * xr.step;
              auto x = xr;
              if (i0 + q >= n_items) x.off[0] = kReach;  // nothing to fetch
#pragma unroll
              for (int t = 0; t < 4; ++t) xf[q][t] = x.load(0, off + t * xr.step);
            }
          };
          load_items(0);
          if (e0 == 0) row_sums();
          float cl[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const bool row = mt * 16 + col < B, live0 = lg < NC && row, live1 = lg + 4 < NC && row;
            const float m0 = live0 ? __uint_as_float(st[i][0].x) : -INFINITY, m1 = live1 ? __uint_as_float(st[i][1].x) : -INFINITY;
            const float l0 = live0 ? __uint_as_float(st[i][0].y) : 0.f, l1 = live1 ? __uint_as_float(st[i][1].y) : 0.f;
            float mx = fmaxf(m0, m1);
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            cl[i][0] = l0 > 0.f ? l0 * expf(m0 - mx) : 0.f;
            cl[i][1] = 0.f;
            if (NC > 4) cl[i][1] = l1 > 0.f ? l1 * expf(m1 - mx) : 0.f;
            sh.ml[w][i][lg][col] = cl[i][0];
            sh.ml[w][i][lg + 4][col] = cl[i][1];
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            float den = 0.f;  // in chunk order
#pragma unroll
            for (int k = 0; k < 8; ++k) den += sh.ml[w][i][k][col];
            sh.share[w][i][lg][col] = den > 0.f ? cl[i][0] / den : 0.f;
            sh.share[w][i][lg + 4][col] = den > 0.f ? cl[i][1] / den : 0.f;
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          for (int i0 = 0; i0 < n_items; i0 += kItemsAhead) {
            if (i0) load_items(i0);
#pragma unroll
            for (int q = 0; q < kItemsAhead; ++q) {
              const int i = i0 + q;
              if (i < n_items) {
                const int h = i >= NC ? 1 : 0, k = i - h * NC;
                if (k == 0 && e0 + h == per0) {  // range w is complete
#pragma unroll
                  for (int j = 0; j < OT; ++j) {
                    sh.red[w * OT + j][lane] = acc[j];
                    acc[j] = zero;
                  }
                }
                const float share = sh.share[w][h][k][col];
#pragma unroll
                for (int j = 0; j < OT; ++j) {
                  v4f part = zero;
                  if (h == 0) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) part = mfma16(wf[0][t][j], xf[q][t], part);
                  } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t) part = mfma16(wf[1][t][j], xf[q][t], part);
                  }
                  acc[j] = acc[j] + part * share;
                }
              }
            }
          }
        }
        if (n_e == 0) row_sums();
#pragma unroll
        for (int j = 0; j < OT; ++j) {
          if (per1 > 0) {
            sh.red[(w + 8) * OT + j][lane] = acc[j];
          } else {
            sh.red[w * OT + j][lane] = acc[j];
            if (w + 8 < R) sh.red[(w + 8) * OT + j][lane] = zero;
          }
        }
        finish();
      }
      leave();
    }
    // ---- gate / up projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, lane = c.lane, rq = (lane >> 4) * 4, first_tile = (kPersistGrid - 1 - c.wg) * GU_TILES;
      const int kt_d = keep(a.kt_d), nt_gu = keep(a.nt_gu), nt_d = keep(a.nt_d), B = keep(a.B), per = (kt_d + 7) / 8;
      const h16_t* const W = a.wgu + (size_t)l * a.layer_stride / sizeof(h16_t);
      h16_t* const act = keep(a.act + (size_t)l * a.act_stride);
      int* const err_flag = keep(a.err_flag);
      if (first_tile >= nt_gu) {
        if (!enter([] {})) return;
      } else {
        Stream<GU_TILES, BT, Gu::kAhead, Gu::kAhead> st;
        auto start = [&] {
          int rows[GU_TILES];
#pragma unroll
          for (int i = 0; i < GU_TILES; ++i) rows[i] = min(first_tile + i, nt_gu - 1) * kt_d * 1024;
          st.start(rsrc_of(W), rows, w * per, min(per, kt_d - w * per), 0, 0, kt_d - 1, lane);
        };
        if (!enter(start)) return;
        const auto xr = Operand<BT>::tiled(keep(a.xo + (size_t)l * a.x_stride), BT, 0, lane, B);
        constexpr int kRows = BT == 2 ? 8 : 16, kOf = 16 * BT / kRows;
        if (w < 2 * kOf) {
          RowSums<kRows, NT> rs;
          const int row0 = w % kOf * kRows;
          rs.load(a.ss_in[1 - w / kOf], row0, lane);
          rs.finish(w / kOf ? sh.squares_old : sh.squares, sh.total[w / kOf], row0, nt_d, 4 * 8 / BT, lane);
        }
        v4f acc[GU_TILES][BT];
        clear(acc);
        st.operands(xr);
        st.run(xr, 0, st.n, acc);
        bool out_of_range = false;
#pragma unroll
        for (int r = 0; r < Gu::kRounds; ++r) {
          if (r > 0) lds_barrier();  // the round before has been read
#pragma unroll
          for (int i = 0; i < GU_TILES; ++i)
#pragma unroll
            for (int g = 0; g < Gu::kGroup; ++g)
              if (r * Gu::kGroup + g < BT) sh.red[(i * Gu::kGroup + g) * 8 + w][lane] = acc[i][(r * Gu::kGroup + g) % BT];
          lds_barrier();
          // a wavefront per (pair of row tiles, tile of 16 rows)
          for (int t = w; t < GU_TILES / 2 * Gu::kGroup; t += kWaves) {
            const int p = t / Gu::kGroup, g = t % Gu::kGroup, mt = r * Gu::kGroup + g, m = mt * 16 + (lane & 15);
            const int tile = first_tile + 2 * p;
            if (mt >= BT || tile >= nt_gu) continue;
            v4f gs = zero, us = zero;
            add_ranges<8>(gs, sh.red, (2 * p * Gu::kGroup + g) * 8, 1, lane);
            add_ranges<8>(us, sh.red, ((2 * p + 1) * Gu::kGroup + g) * 8, 1, lane);
            const float sc = scale_of(sh.total[0][m], sh.total[1][m], true, a.inv_d, a.eps);
            gs = gs * sc;
            us = us * sc;
            uint2 pk;
            bool far = false;
            pk.x = pack_h16x2_track(silu_p(gs[0]) * us[0], silu_p(gs[1]) * us[1], far);
            pk.y = pack_h16x2_track(silu_p(gs[2]) * us[2], silu_p(gs[3]) * us[3], far);
            if (m < B) {
              st8(act + act_off(m, (tile >> 1) * 16 + rq, 16 * BT), pk);
              out_of_range |= far;
            }
          }
        }
        if (out_of_range) atomicOr(err_flag, kErrFp16Range);
      }
      leave();
    }
    // ---- down projection: sums per split of K
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane, rq = (lane >> 4) * 4;
      const h16_t* const W = a.wdown + (size_t)l * a.layer_stride / sizeof(h16_t);
      const Rsrc out = rsrc_of(keep(part_of<ASK>(a)));
      const int kt_F = keep(a.kt_F), d = keep(a.d), nt_d = keep(a.nt_d), ks = keep(a.ks_down), B = keep(a.B);
      const int per_split = (kt_F + ks - 1) / ks, split = DN_RANGES == 5 ? wg & 7 : wg % ks;
      const int kbeg = split * per_split, kend = min(kt_F, kbeg + per_split);
      const int per = (max(kend - kbeg, 0) + DN_RANGES - 1) / DN_RANGES;
      // 8 splits of 5 ranges: split = workgroup % 8, three row tiles, a range per wavefront (the others have none); else groups
      // of four tiles and 4 ranges, two tiles per wavefront, one (group, split) per workgroup
      constexpr int kTiles = DN_RANGES == 5 ? 3 : 4, kMine = DN_RANGES == 5 ? 3 : 2;
      constexpr int PF = DN_RANGES == 5 ? 6 : 4, PFX = DN_RANGES == 5 ? 3 : 4;
      const int s = DN_RANGES == 5 ? w : w % 4, j0 = DN_RANGES == 5 ? 0 : w / 4 * 2;
      auto tile_of = [&](int j) { return DN_RANGES == 5 ? (wg >> 3) + kPersistGrid / 8 * j : wg / ks * kTiles + j; };
      const bool works = s < DN_RANGES && tile_of(0) < nt_d;
      Stream<kMine, BT, PF, PFX> st;
      auto start = [&] {
        int rows[kMine];
#pragma unroll
        for (int i = 0; i < kMine; ++i) rows[i] = min(tile_of(j0 + i), nt_d - 1) * kt_F * 1024;
        const int k0 = kbeg + s * per;
        st.start(rsrc_of(W), rows, k0, works ? min(per, kend - k0) : 0, 0, 0, kt_F - 1, lane);
      };
      if (!enter(start)) return;
      const auto xr = Operand<BT>::tiled(keep(a.act + (size_t)l * a.act_stride), BT, 0, lane, B);
      v4f acc[kMine][BT];
      clear(acc);
      if (works) {
        st.operands(xr);
        st.run(xr, 0, st.n, acc);
      }
      if (s < DN_RANGES) {
#pragma unroll
        for (int i = 0; i < kMine; ++i)
#pragma unroll
          for (int mt = 0; mt < BT; ++mt) sh.red[((j0 + i) * BT + mt) * DN_RANGES + s][lane] = acc[i][mt];
      }
      lds_barrier();
      for (int t = w; t < kTiles * BT; t += kWaves) {  // a wavefront per (row tile, tile of 16 rows)
        const int j = t / BT, mt = t % BT, m = mt * 16 + (lane & 15), tile = tile_of(j);
        if (tile >= nt_d) continue;
        v4f sum = zero;
        add_ranges<DN_RANGES>(sum, sh.red, t * DN_RANGES, 1, lane);
        if (m < B) st16(out, ((split * 16 * BT + m) * d + tile * 16 + rq) * 4, 0, written(sum));
      }
      leave_asked();
    }
    // ---- sum of the splits, residual, operand of the next block: row tile wg, a wavefront per tile of 16 rows
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane, rq = (lane >> 4) * 4, m = min(w, BT - 1) * 16 + (lane & 15);
      const int nt_d = keep(a.nt_d);
      const TileOut to(a, x_behind(a, l), 0, l + 1 == n_layers);
      const Rsrc part = rsrc_of(keep(part_of<ASK>(a)));
      const int ks = keep(a.ks_down), at = (min(m, to.B - 1) * to.d + min(wg, nt_d - 1) * 16 + rq) * 4;
      const float* gp = l + 1 == n_layers ? a.final_norm : (const float*)((const char*)a.attn_norm + (l + 1) * a.layer_stride);
      const bool mine = wg < nt_d && w < BT;
      v4f gain = zero, h_old = zero;
      auto prepare = [&] {  // what does not depend on the splits: the residual and the sums of the rows
        constexpr int kRows = BT == 2 ? 4 : 8;
        if (wg < nt_d && w * kRows < 16 * BT) {
          RowSums<kRows, NT> rs;
          rs.load(a.ss_in[1], w * kRows, lane);
          rs.finish(sh.squares, sh.total[0], w * kRows, nt_d, 4 * DN_RANGES / BT, lane);
        }
        if (mine) {
          gain = *reinterpret_cast<const v4f*>(gp + wg * 16 + rq);
          h_old = ld16f(to.h, at, 0);
        }
      };
      if constexpr (ASK) {
        prepare();
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(sh.stop)) return;
      } else {
        if (!enter(prepare)) return;
      }
      if (mine) {
        const std::conditional_t<ASK, Asker, Known> asker = [&] {
          if constexpr (ASK) return Asker{a, &sh.stop};
          else return Known{};
        }();
        v4f sum = zero;
        for (int s0 = 0; s0 < ks; s0 += 8) {
          v4f v[8];
          asker([&] {
            uint32_t top = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = ld16f(part, at, min(s0 + k, ks - 1) * 64 * BT * to.d);
#pragma unroll
            for (int k = 0; k < 8; ++k) top = max(top, largest(__builtin_bit_cast(v4u, v[k])));
            return top;
          });
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (s0 + k < ks) sum = sum + v[k];
        }
        loads_done();
        residual_tile<BT>(to, wg, w, lane, sum, h_old, gain, scale_of(sh.total[0][m], 0.f, false, a.inv_d, a.eps));
      }
      leave();
      if (ASK && mine && m < to.B)
        for (int s = 0; s < ks; ++s) st16(part, at, s * 64 * BT * to.d, none);
    }
  }
}

template <int BT, int GU_TILES, int DN_RANGES>
__global__ __launch_bounds__(kThreads, 2) void k_decode_layers_rows(PersistArgs) {  // read through the kernel argument segment: fresh()
  constexpr int NT = DN_RANGES == 5 ? 96 : kPersistGrid;  // row tiles of the residual at most
  __shared__ Shared<BT, GU_TILES, NT> sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) sh.stop = 0;
  __syncthreads();
  step<BT, GU_TILES, DN_RANGES, NT>(sh, wave);
}

}  // namespace

void launch_rows(const PersistArgs& a, int bt, int gu_tiles, hipStream_t st) {
  if (persist_some_ask(bt, gu_tiles)) launch_fill_u32(reinterpret_cast<uint32_t*>(a.hand), kNotThere, (size_t)a.at_hand.bytes / 4, st);
  if (bt == 2 && gu_tiles == 6) k_decode_layers_rows<2, 6, 5><<<kPersistGrid, kThreads, 0, st>>>(a);
  else if (bt == 2) k_decode_layers_rows<2, 10, 4><<<kPersistGrid, kThreads, 0, st>>>(a);
  else if (bt == 3) k_decode_layers_rows<3, 6, 5><<<kPersistGrid, kThreads, 0, st>>>(a);
  else k_decode_layers_rows<4, 6, 5><<<kPersistGrid, kThreads, 0, st>>>(a);
}

}  // namespace persist
}  // namespace bf16
}  // namespace mtmc
