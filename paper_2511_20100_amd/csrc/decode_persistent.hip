// The residual blocks of a decode step as ONE launch (MTMC_OPT_PERSISTENT_DECODE): one tile of 16 rows here, two to four tiles
// in decode_persistent_rows.hip.
//
// What bounds a step of few rows as six launches per block is not its bytes: a dependent launch costs 4 to 5 us before its
// first weight arrives, and a block's 93 MB (1.5 B shape, 15 us at the rate of a plain read) took 48 us as six launches.  Here
// one workgroup per CU stays for the whole step.  Between two dependent phases the grid waits on counters in memory (1.5 us
// from the last arrival), and the weights of the next phase are on their way to registers while it waits: they depend on
// nothing.  One row 47.7 -> 31 us per block (63 steps 89.5 -> 63.1 ms), 16 rows 51 -> 37 (96.6 -> 74.0 ms).
//
// What is left of a block's 31 us are six dependent phases (the sixth adds up the splits) of about 1 us to the first operand, 0.5
// for sums and epilogue, 0.5 to 1 for the stores to drain and 1.5 for the counters, and the 10 us in which the gate / up and
// down weights come at 5 TB/s.
//
//   wavefronts 0 .. 7    stream weights and multiply; their sums per range of K go to LDS.  They ask for the next weights only
//                        when the workgroup has been counted in: ahead of its stores in the CU's queue to memory they
//                        held these up by 2 to 3 us.
//   wavefronts 8 .. 11   add up the ranges in order, run the epilogues, drain their stores, count the workgroup in and (one
//                        of them) watch the counters.  They hold no weights in flight: loads return in order, and a
//                        look at a counter would come back behind them.
//
// What one workgroup writes and another reads goes past the caches that are not coherent between the dies: device-scope
// (sc1) stores and loads, stores drained before the workgroup is counted.  Everything else (weights, tables, pages of
// earlier steps) is read as usual.  Every sum has the ranges and the order of the launches of decode_bf16.hip, so the
// results are theirs bit for bit.
//
// All kPersistGrid workgroups have to be resident at once: one per CU, and no second persistent launch of the process under way
// (PersistentTurn).  What else holds a CU, and for how long, nobody here knows.  So the first wait of a launch is its roll call
// (roll_call.h): the phase before it changes nothing that a step starts from, and where not all workgroups come within the limit, the
// launch ends there and decode_persistent_some.hip does the step.
#include <type_traits>

#include "decode_persistent.h"

namespace mtmc {
namespace bf16 {
namespace persist {
namespace {

constexpr int kComputeWaves = AW, kControlWaves = 4, kThreads = (kComputeWaves + kControlWaves) * 64;
constexpr int kItems = 48;  // sums of 16 x 16 values that a phase hands over at once

struct Shared {
  union {
    v4f red[kItems][64];  // sums per range of K, as the accumulators lie in the lanes
    AttnLds at;
  };
  int table[ATAB];                       // page ids of the attention unit
  float ml[kComputeWaves][2][8][16];     // per wavefront, head in hand, chunk and row: the chunk's rescaled sum
  float share[kComputeWaves][2][8][16];  // ... and its share
  float part[2][16][68];                 // partial sums of a row's squares
  float scale[16];
  int arrived, stop;
};

// Each control wavefront drains its own stores, the last one of the four counts the workgroup in.
__device__ __forceinline__ void arrive(const Ctx& c, int* arrived, uint32_t phase) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  if (c.lane == 0) {
    const int n = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (n % kControlWaves == kControlWaves - 1) count_in(c, phase);
  }
}

// The row scales of a phase.  The sums of squares of a row's tiles lie side by side (kPersistGrid floats per row).  P partial sums
// of them (part p: tiles p, p + P, ...), then those in order: the order of a launch of 16 P threads.  The four control
// wavefronts take four rows each, 16 lanes to a row, all loads in one go; what they leave in sh.scale is read behind a barrier.
template <int P, bool TWO>
__device__ __forceinline__ void row_scales(Shared& sh, const Ctx& c, const float* cur, const float* old) {
  const PersistArgs& a = c.a;
  const int cw = c.wave - kComputeWaves, m = cw * 4 + (c.lane >> 4), q = c.lane & 15;
  if (cw * 4 >= a.B) return;
  // lane q: parts q, q + G, ... (PP of them), part p's tiles p + P k (K of them)
  constexpr int G = P == 20 ? 10 : 16, PP = P / G, K = P == 20 ? 5 : (kPersistGrid + P - 1) / P;
  float va[PP][K], vb[PP][K];
  if (P != 20 || q < G) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < PP; ++i) {
        const int t = m * kPersistGrid + min(q + G * i + P * k, a.nt_d - 1);
        va[i][k] = ld4(cur + t);
        if (TWO) vb[i][k] = ld4(old + t);
      }
#pragma unroll
    for (int i = 0; i < PP; ++i) {
      float sa = 0.f, sb = 0.f;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool there = q + G * i + P * k < a.nt_d;
        sa += there ? va[i][k] : 0.f;
        if (TWO) sb += there ? vb[i][k] : 0.f;
      }
      sh.part[0][m][q + G * i] = sa;
      if (TWO) sh.part[1][m][q + G * i] = sb;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows are the wavefront's own
  if (q == 0) {
    float ta = 0.f, tb = 0.f;
    v4f pa[P / 4], pb[P / 4];
#pragma unroll
    for (int p = 0; p < P / 4; ++p) {
      pa[p] = *reinterpret_cast<const v4f*>(&sh.part[0][m][4 * p]);
      if (TWO) pb[p] = *reinterpret_cast<const v4f*>(&sh.part[1][m][4 * p]);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
      ta += pa[p / 4][p % 4];
      if (TWO) tb += pb[p / 4][p % 4];
    }
    sh.scale[m] = scale_of(ta, tb, TWO, a.inv_d, a.eps);
  }
}

// wait_grid() behind the first phase: the roll call.
__device__ __forceinline__ bool answer_roll(const Ctx& c) {
  const Word mine = word_of(c.a, c.wg % kPersistTops), ended = word_of(c.a, kPersistEnded), before = {c.a.sync + kPersistGaveUp};
  const long long t0 = wall_clock64();
  long long limit = c.a.roll_ticks;
  for (int i = 0; look(mine) < kPersistGroups; ++i) {
    if (i % 16 == 15) {
      if (look(ended)) return false;
      if (look(before)) limit = min(limit, kAgainTicks);
    }
    if (wall_clock64() - t0 <= limit) continue;
    if (give_up(c)) return false;
    limit = kWaitTicks;  // every group is full: the last of them are about to say so
  }
  asm volatile("" ::: "memory");
  return true;
}

// ---- which workgroup does what.  The O projection and the sum of the splits have a row tile for workgroups 0 .. nt_d - 1; the
// QKV tiles go to the others first (from the top down), the attention to those that start behind nt_d, and of the gate / up
// tiles a workgroup with an O tile takes one pair where the others can take the rest: it comes to them last.
__device__ __forceinline__ int qkv_place(int wg) { return kPersistGrid - 1 - wg; }
__device__ __forceinline__ int attn_place(const PersistArgs& a, int wg) { return (wg - a.nt_d) & (kPersistGrid - 1); }
template <int GU_TILES>
struct GuShare {
  int first, tiles;  // row tiles of this workgroup
  __device__ __forceinline__ GuShare(const PersistArgs& a, int wg) {
    const int others = kPersistGrid - a.nt_d;
    if (a.nt_gu <= others * GU_TILES + 2 * a.nt_d) {
      tiles = wg < a.nt_d ? 2 : GU_TILES;
      first = wg < a.nt_d ? others * GU_TILES + 2 * wg : (wg - a.nt_d) * GU_TILES;
    } else {
      tiles = GU_TILES;
      first = wg * GU_TILES;
    }
  }
};

template <int S>
__device__ __forceinline__ v4f sum_ranges(const Shared& sh, int first, int lane) {
  v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
  add_ranges<S>(sum, sh.red, first, 1, lane);
  return sum;
}

template <int GU_TILES, int DN_RANGES>
__device__ __forceinline__ void control(Shared& sh, int wave) {
  const int cw = wave - kComputeWaves;
  const bool lead = cw == 0;
  constexpr int kGuRanges = GU_TILES == 6 ? 8 : 4;
  uint32_t phase = 0;
  // lets the compute wavefronts into the phase; false: the launch ends here
  auto go = [&](const Ctx& c) {
    if (lead && phase > 0 && !wait_grid(c, phase)) sh.stop = 1;
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(sh.stop) == 0;
  };
  auto arrive_lead = [&](const Ctx& c) {  // phases whose stores are the lead's own, or drained before a barrier
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (lead && c.lane == 0) count_in(c, phase);
  };
  // behind the barrier: what was loaded before is there, so that no store has to be waited for on its behalf
  auto loads_done = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  const int n_layers = fresh(wave).a.n_layers;
  bool attends, attn_active;
  {
    const Ctx c = fresh(wave);
    const AttnUnit u(c.a, attn_place(c.a, c.wg));
    attends = u.there;
    attn_active = u.active;
  }
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const int place = qkv_place(wg);
      const Rsrc out = rsrc_of(keep(a.qkv));
      const int nt_qkv = keep(a.nt_qkv), B = keep(a.B);
      if (!go(c)) return;
      if (l == 0) {
        if (lane < 4) sh.scale[cw * 4 + lane] = 1.f;
      } else if (place < nt_qkv) {
        row_scales<64, true>(sh, c, a.ss_in[0], a.ss_in[1]);
      }
      for (int u = 0; place + u * kPersistGrid < nt_qkv; ++u) {
        lds_barrier();
        if ((u & 3) == cw) {
          const int nt = place + u * kPersistGrid;
          const v4f sum = sum_ranges<16>(sh, (u & 1) * 16, lane);
          if (m < B) st16(out, ((m * nt_qkv + nt) * 16 + rq) * 4, 0, __builtin_bit_cast(v4u, sum * sh.scale[m]));
        }
      }
      arrive(c, &sh.arrived, phase);
      lds_barrier();
      ++phase;
    }
    // ---- attention
    {
      const Ctx c = fresh(wave);
      if (lead && l == 0 && !answer_roll(c)) sh.stop = 1;
      if (!go(c)) return;
      if (attends) {
        if (attn_active) {
          lds_barrier();
          lds_barrier();
        }
        lds_barrier();
      }
      arrive_lead(c);
      lds_barrier();
      ++phase;
    }
    // ---- O projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const bool has_tile = wg < a.nt_d;
      const TileOut to(a, a.xo + (size_t)l * a.x_stride, 1, l + 1 == n_layers);
      const int ranges = keep(a.o_ranges);
      v4f h_old = v4f{0.f, 0.f, 0.f, 0.f}, gain = h_old;
      if (lead && has_tile) {
        h_old = ld16f(to.h, (min(m, to.B - 1) * to.d + wg * 16 + rq) * 4, 0);
        gain = *reinterpret_cast<const v4f*>((const float*)((const char*)a.ffn_norm + l * a.layer_stride) + wg * 16 + rq);
      }
      if (!go(c)) return;
      if (has_tile) {
        if (ranges == 16) row_scales<64, false>(sh, c, a.ss_in[0], a.ss_in[0]);
        else if (ranges == 12) row_scales<48, false>(sh, c, a.ss_in[0], a.ss_in[0]);
        else row_scales<32, false>(sh, c, a.ss_in[0], a.ss_in[0]);
        lds_barrier();
        if (lead) {
          loads_done();
          const v4f sum = ranges == 16 ? sum_ranges<16>(sh, 0, lane) : ranges == 12 ? sum_ranges<12>(sh, 0, lane) : sum_ranges<8>(sh, 0, lane);
          residual_tile<1>(to, wg, 0, lane, sum, h_old, gain, sh.scale[m]);
        }
      }
      arrive_lead(c);
      lds_barrier();
      ++phase;
    }
    // ---- gate / up projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      h16_t* const act = keep(a.act + (size_t)l * a.act_stride);
      const int nt_gu = keep(a.nt_gu), B = keep(a.B);
      int* const err_flag = keep(a.err_flag);
      if (!go(c)) return;
      const GuShare<GU_TILES> share(a, wg);
      if (share.first < nt_gu) {
        row_scales<4 * kGuRanges, true>(sh, c, a.ss_in[1], a.ss_in[0]);
        lds_barrier();
        bool out_of_range = false;
        for (int p = cw; p < share.tiles / 2; p += kControlWaves) {
          const int j = share.first + 2 * p;
          if (j >= nt_gu) break;
          const float sc = sh.scale[m];
          const v4f g = sum_ranges<kGuRanges>(sh, 2 * p * kGuRanges, lane) * sc;
          const v4f u = sum_ranges<kGuRanges>(sh, (2 * p + 1) * kGuRanges, lane) * sc;
          uint2 pk;
          bool far = false;
          pk.x = pack_h16x2_track(silu_p(g[0]) * u[0], silu_p(g[1]) * u[1], far);
          pk.y = pack_h16x2_track(silu_p(g[2]) * u[2], silu_p(g[3]) * u[3], far);
          if (m < B) {
            st8(act + act_off(m, (j >> 1) * 16 + rq, 16), pk);
            out_of_range |= far;
          }
        }
        if (out_of_range) atomicOr(err_flag, kErrFp16Range);
      }
      arrive(c, &sh.arrived, phase);
      lds_barrier();
      ++phase;
    }
    // ---- down projection: sums per split of K
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const Rsrc out = rsrc_of(keep(a.part));
      const int d = keep(a.d), nt_d = keep(a.nt_d), B = keep(a.B), ks = keep(a.ks_down);
      if (!go(c)) return;
      if (wg < nt_d) row_scales<4 * DN_RANGES, false>(sh, c, a.ss_in[1], a.ss_in[1]);
      lds_barrier();
      constexpr int kTiles = DN_RANGES == 5 ? 3 : DN_RANGES == 8 ? 2 : 4;
      const int split = DN_RANGES == 5 ? wg & 7 : wg % ks;
      const int tile = DN_RANGES == 5 ? (wg >> 3) + kPersistGrid / 8 * cw : wg / ks * kTiles + cw;
      if (cw < kTiles && tile < nt_d) {
        const v4f sum = sum_ranges<DN_RANGES>(sh, cw * DN_RANGES, lane);
        if (m < B) st16(out, ((split * 16 + m) * d + tile * 16 + rq) * 4, 0, __builtin_bit_cast(v4u, sum));
      }
      arrive(c, &sh.arrived, phase);
      lds_barrier();
      ++phase;
    }
    // ---- sum of the splits, residual, operand of the next block: the lead alone
    if (lead) {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const bool has_tile = wg < a.nt_d;
      const TileOut to(a, x_behind(a, l), 0, l + 1 == n_layers);
      const Rsrc part = rsrc_of(keep(a.part));
      const int ks = keep(a.ks_down), at = (min(m, to.B - 1) * to.d + wg * 16 + rq) * 4;
      const float* gp = l + 1 == n_layers ? a.final_norm : (const float*)((const char*)a.attn_norm + (l + 1) * a.layer_stride);
      v4f gain = v4f{0.f, 0.f, 0.f, 0.f}, h_old = gain;
      if (has_tile) {
        gain = *reinterpret_cast<const v4f*>(gp + wg * 16 + rq);
        h_old = ld16f(to.h, at, 0);
      }
      if (!wait_grid(c, phase)) {
        sh.stop = 1;
      } else if (has_tile) {
        v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < ks; s0 += 8) {
          v4f v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = ld16f(part, at, min(s0 + u, ks - 1) * 64 * to.d);
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (s0 + u < ks) sum = sum + v[u];
        }
        loads_done();
        residual_tile<1>(to, wg, 0, lane, sum, h_old, gain, sh.scale[m]);
      }
      arrive_lead(c);
    }
    ++phase;
  }
}

// ======================================================================================
// compute wavefronts
// ======================================================================================
template <int GU_TILES, int DN_RANGES>
__device__ __forceinline__ void compute(Shared& sh, int wave) {
  auto go = [&] {
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(sh.stop) == 0;
  };
  // the control wavefronts have stored what the phase gave and counted the workgroup in: only then the next weights, which
  // would be ahead of those stores in the CU's queue to memory
  auto counted_in = [] { lds_barrier(); };
  const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
  const int n_layers = fresh(wave).a.n_layers;
  const Ctx first = fresh(wave);
  const AttnHeld unit(first.a, attn_place(first.a, first.wg), wave, first.lane, sh.table, 16);
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection: one row tile at a time, 16 ranges of K, two per wavefront
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane;
      const h16_t* const W = a.wqkv + (size_t)l * a.layer_stride / sizeof(h16_t);
      const h16_t* const x = keep(x_of(a, l));
      const int kt_d = keep(a.kt_d), nt_qkv = keep(a.nt_qkv), B = keep(a.B), per = (kt_d + 15) / 16;
      const Operand<1> xr = Operand<1>::tiled(x, 1, 0, lane, B);
      Stream<1, 1, 4, 4> s0, s1;
      auto start = [&](int nt) {
        int rows[1] = {nt * kt_d * 1024};
        s0.start(rsrc_of(W), rows, w * per, min(per, kt_d - w * per), 0, 0, kt_d - 1, lane);
        s1.start(rsrc_of(W), rows, (w + 8) * per, min(per, kt_d - (w + 8) * per), 0, 0, kt_d - 1, lane);
      };
      int nt = qkv_place(wg);
      if (nt < nt_qkv) {
        start(nt);
        if (!go()) return;
        for (int u = 0;; ++u) {
          v4f a0[1][1] = {{zero}}, a1[1][1] = {{zero}};
          s0.operands(xr);
          s1.operands(xr);
          s0.run(xr, 0, s0.n, a0);
          s1.run(xr, 0, s1.n, a1);
          sh.red[(u & 1) * 16 + w][lane] = a0[0][0];
          sh.red[(u & 1) * 16 + w + 8][lane] = a1[0][0];
          lds_barrier();
          nt += kPersistGrid;
          if (nt >= nt_qkv) break;
          start(nt);
        }
      } else if (!go()) {
        return;
      }
    }
    counted_in();
    // ---- attention
    if (!unit.active) {
      if (!go()) return;
      if (unit.there) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
      }
    } else {
      if (!attend<false>(unit, sh.at, sh.table, l, wave, 16, go)) return;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_barrier();
    }
    counted_in();
    // ---- O projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane, kt_nq = keep(a.kt_nq), B = keep(a.B);
      const h16_t* const W = a.wo + (size_t)l * a.layer_stride / sizeof(h16_t) + (size_t)wg * kt_nq * 512;
      const h16_t* const o = keep(a.at.o);
      const int R = keep(a.o_ranges), NC = keep(a.at.n_chunks);
      if (wg >= a.nt_d) {
        if (!go()) return;
      } else if (NC == 1) {
        const int per = (kt_nq + R - 1) / R;
        int rows[1] = {0};
        const auto xr = Operand<1, kDeviceScope>::tiled(o, 1, 0, lane, B);
        Stream<1, 1, 4, 4> s0, s1;
        s0.start(rsrc_of(W), rows, w * per, min(per, kt_nq - w * per), 0, 0, kt_nq - 1, lane);
        s1.start(rsrc_of(W), rows, (w + 8) * per, min(per, kt_nq - (w + 8) * per), 0, 0, kt_nq - 1, lane);  // empty with 8 ranges
        if (!go()) return;
        v4f a0[1][1] = {{zero}}, a1[1][1] = {{zero}};
        s0.operands(xr);
        s1.operands(xr);
        s0.run(xr, 0, s0.n, a0);
        s1.run(xr, 0, s1.n, a1);
        sh.red[w][lane] = a0[0][0];
        sh.red[w + 8][lane] = a1[0][0];
        lds_barrier();
      } else {
        // The chunks of the context are combined here, head by head: out += sum_chunk share * (W_head . o_chunk), share =
        // l exp(m - max m) / sum l exp(m - max m).  Range v takes heads v, v + R, ...; this wavefront ranges w and (12
        // ranges) w + 8: its list of heads, two in hand at a time, up to five (head, chunk) operands on their way at once (six do not
        // fit the registers).
        constexpr int kItemsAhead = 5;
        const int n_heads = keep(a.at.Hq), col = lane & 15, lg = lane >> 4;
        const auto xr = Operand<1, kDeviceScope>::tiled(o, 1, 0, lane, B);
        const float* const ml = keep(a.at.ml);
        const int chunk_bytes = (int)(a.at.o_chunk_stride * sizeof(h16_t));
        const int per0 = max((n_heads - w + R - 1) / R, 0);                                    // heads of range w
        const int per1 = (R > 8 && w + 8 < R) ? max((n_heads - (w + 8) + R - 1) / R, 0) : 0;  // of range w + 8
        const int n_e = per0 + per1;
        auto head_of = [&](int e0) {  // entry e0 of the list; past its end the last one again
          const int e = min(e0, n_e - 1);
          return max(0, e < per0 ? w + e * R : w + 8 + (e - per0) * R);
        };
        v8h wf[2][4];
        auto load_heads = [&](int e0) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) wf[i][t] = load_weight(W + (size_t)(head_of(e0 + i) * 4 + t) * 512, lane);
        };
        load_heads(0);
        if (!go()) return;
        v4f acc = zero;
        for (int e0 = 0; e0 < n_e; e0 += 2) {
          if (e0) load_heads(e0);
          // chunk statistics of the two heads: lane (row, lg) has chunks lg and lg + 4
          uint2 st[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k)
              st[i][k] = ld8(ml + (((size_t)min(col, B - 1) * n_heads + head_of(e0 + i)) * NC + min(lg + 4 * k, NC - 1)) * 2);
          const int n_items = min(2, n_e - e0) * NC;
          v8h xf[kItemsAhead][4];
          auto load_items = [&](int i0) {
#pragma unroll
            for (int q = 0; q < kItemsAhead; ++q) {
              const int i = min(i0 + q, n_items - 1), h = i >= NC ? 1 : 0;
              const int off = (i - h * NC) * chunk_bytes + head_of(e0 + h) * 4096;
#pragma unroll
              for (int t = 0; t < 4; ++t) xf[q][t] = xr.load(0, off + t * 1024);
            }
          };
          load_items(0);
          float cl[2][2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const bool live0 = lg < NC && col < B, live1 = lg + 4 < NC && col < B;
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
                  sh.red[w][lane] = acc;
                  acc = zero;
                }
                v4f part = zero;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                  if (h == 0) part = mfma16(wf[0][t], xf[q][t], part);
                if (h == 1) {
#pragma unroll
                  for (int t = 0; t < 4; ++t) part = mfma16(wf[1][t], xf[q][t], part);
                }
                acc = acc + part * sh.share[w][h][k][col];
              }
            }
          }
        }
        if (per1 > 0) {
          sh.red[w + 8][lane] = acc;
        } else {
          sh.red[w][lane] = acc;
          if (w + 8 < R) sh.red[w + 8][lane] = zero;
        }
        lds_barrier();
      }
    }
    counted_in();
    // ---- gate / up projection: 8 ranges of K over all the tiles, or 4 over half of them
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, lane = c.lane;
      constexpr int kRanges = GU_TILES == 6 ? 8 : 4;
      const GuShare<GU_TILES> share(a, c.wg);
      const int kt_d = keep(a.kt_d), nt_gu = keep(a.nt_gu), B = keep(a.B), first = keep(share.first);
      const int per = (kt_d + kRanges - 1) / kRanges, s = w % kRanges;
      const h16_t* const W = a.wgu + (size_t)l * a.layer_stride / sizeof(h16_t);
      const Operand<1> xr = Operand<1>::tiled(keep(a.xo + (size_t)l * a.x_stride), 1, 0, lane, B);
      // kTiles row tiles of this wavefront from tile first + j0 on
      auto multiply = [&](auto tiles_per_wave, auto depth) {
        constexpr int kTiles = decltype(tiles_per_wave)::value, PF = decltype(depth)::value;
        const int j0 = (w / kRanges) * kTiles;
        int rows[kTiles];
#pragma unroll
        for (int i = 0; i < kTiles; ++i) rows[i] = min(first + j0 + i, nt_gu - 1) * kt_d * 1024;
        Stream<kTiles, 1, PF, PF> st;
        st.start(rsrc_of(W), rows, s * per, min(per, kt_d - s * per), 0, 0, kt_d - 1, lane);
        if (!go()) return false;
        v4f acc[kTiles][1];
        clear(acc);
        st.operands(xr);
        st.run(xr, 0, st.n, acc);
#pragma unroll
        for (int i = 0; i < kTiles; ++i) sh.red[(j0 + i) * kRanges + s][lane] = acc[i][0];
        lds_barrier();
        return true;
      };
      constexpr int kFull = GU_TILES * kRanges / 8, kPair = 2 * kRanges / 8;
      if (first >= nt_gu) {
        if (!go()) return;
      } else if (share.tiles == GU_TILES) {
        if (!multiply(std::integral_constant<int, kFull>{}, std::integral_constant<int, kFull >= 5 ? 4 : 6>{})) return;
      } else {
        if (!multiply(std::integral_constant<int, kPair>{}, std::integral_constant<int, 6>{})) return;
      }
    }
    counted_in();
    // ---- down projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane;
      const h16_t* const W = a.wdown + (size_t)l * a.layer_stride / sizeof(h16_t);
      const h16_t* const x = keep(a.act + (size_t)l * a.act_stride);
      const int kt_F = keep(a.kt_F), nt_d = keep(a.nt_d), ks = keep(a.ks_down), B = keep(a.B);
      const int per_split = (kt_F + ks - 1) / ks, split = DN_RANGES == 5 ? wg & 7 : wg % ks;
      const int kbeg = split * per_split, kend = min(kt_F, kbeg + per_split);
      const int per = (max(kend - kbeg, 0) + DN_RANGES - 1) / DN_RANGES;
      if constexpr (DN_RANGES == 5) {
        // 8 splits, split = workgroup % 8; three row tiles, 15 (tile, range) items over 8 wavefronts
        Stream<1, 1, 7, 7> s0, s1;
        auto start = [&](Stream<1, 1, 7, 7>& s, int item) {
          const int i = item / 5, r = item - i * 5, tile = (wg >> 3) + kPersistGrid / 8 * i;
          int rows[1] = {min(tile, nt_d - 1) * kt_F * 1024};
          const int k0 = kbeg + r * per;
          s.start(rsrc_of(W), rows, k0, item < 15 && tile < nt_d ? min(per, kend - k0) : 0, 0, 0, kt_F - 1, lane);
        };
        start(s0, w);
        start(s1, w + 8);
        if (!go()) return;
        const Operand<1> xr = Operand<1>::tiled(x, 1, 0, lane, B);
        v4f a0[1][1] = {{zero}}, a1[1][1] = {{zero}};
        s0.operands(xr);
        s1.operands(xr);
        s0.run(xr, 0, s0.n, a0);
        s1.run(xr, 0, s1.n, a1);
        sh.red[w][lane] = a0[0][0];
        if (w + 8 < 15) sh.red[w + 8][lane] = a1[0][0];
        lds_barrier();
      } else {
        // groups of 2 tiles and 8 ranges or of 4 tiles and 4 ranges, one (group, split) per workgroup
        constexpr int kTiles = DN_RANGES == 8 ? 2 : 4, PF = 6;
        const int t0 = wg / ks * kTiles, s = w % DN_RANGES, j0 = (w / DN_RANGES) * 2, k0 = kbeg + s * per;
        int rows[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) rows[i] = min(t0 + j0 + i, nt_d - 1) * kt_F * 1024;
        Stream<2, 1, PF, PF> st;
        st.start(rsrc_of(W), rows, k0, t0 < nt_d ? min(per, kend - k0) : 0, 0, 0, kt_F - 1, lane);
        if (!go()) return;
        const Operand<1> xr = Operand<1>::tiled(x, 1, 0, lane, B);
        v4f acc[2][1];
        clear(acc);
        st.operands(xr);
        st.run(xr, 0, st.n, acc);
#pragma unroll
        for (int i = 0; i < 2; ++i) sh.red[(j0 + i) * DN_RANGES + s][lane] = acc[i][0];
        lds_barrier();
      }
    }
    counted_in();
  }
}

template <int GU_TILES, int DN_RANGES>
__global__ __launch_bounds__(kThreads, 3) void k_decode_layers(PersistArgs) {  // read through the kernel argument segment: fresh()
  __shared__ Shared sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) {
    sh.arrived = 0;
    sh.stop = 0;
  }
  __syncthreads();
  if (wave < kComputeWaves) compute<GU_TILES, DN_RANGES>(sh, wave);
  else control<GU_TILES, DN_RANGES>(sh, wave);
}

template <int GU_TILES>
void launch_gu(const PersistArgs& a, int dn, hipStream_t st) {
  switch (dn) {
    case 5: k_decode_layers<GU_TILES, 5><<<kPersistGrid, kThreads, 0, st>>>(a); break;
    case 8: k_decode_layers<GU_TILES, 8><<<kPersistGrid, kThreads, 0, st>>>(a); break;
    default: k_decode_layers<GU_TILES, 4><<<kPersistGrid, kThreads, 0, st>>>(a); break;
  }
}

}  // namespace

void launch_one_tile(const PersistArgs& a, int gu_tiles, int dn_ranges, hipStream_t st) {
  if (gu_tiles == 4) launch_gu<4>(a, dn_ranges, st);
  else if (gu_tiles == 6) launch_gu<6>(a, dn_ranges, st);
  else launch_gu<10>(a, dn_ranges, st);
}

}  // namespace persist

void decode_persistent(const PersistArgs& args, int m_tiles, int down_nb, hipStream_t st) {
  const int gu = persist_gu_tiles(args.nt_gu), dn = persist_dn_ranges(down_nb);
  PersistArgs a = args;
  a.gu_ranges = m_tiles > 1 || gu == 6 ? 8 : 4;
  a.dn_ranges = dn;
  if (m_tiles == 1) persist::launch_one_tile(a, gu, dn, st);
  else persist::launch_rows(a, m_tiles, gu, st);
  persist::launch_some(a, m_tiles, st);
}

}  // namespace bf16
}  // namespace mtmc
