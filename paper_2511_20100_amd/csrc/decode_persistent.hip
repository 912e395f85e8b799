// The residual blocks of a decode step of up to 16 rows as ONE launch (MTMC_OPT_PERSISTENT_DECODE).
//
// What bounds a step of few rows as six launches per block is not its bytes: a dependent launch costs 4 to 5 us before its
// first weight arrives, and a block's 93 MB (1.5 B shape, 15 us at the rate of a plain read) took 48 us as six launches.  Here
// one workgroup per CU stays for the whole step.  Between two dependent phases the grid waits on counters in memory (1.5 us
// from the last arrival), and the weights of the next phase are on their way to registers while it waits: they depend on
// nothing.  One row 47.7 -> 31 us per block (63 steps 89.5 -> 63.1 ms), 16 rows 51 -> 37 (96.6 -> 74.0 ms).
//
// What is left of a block's 31 us are five dependent phases of about 1 us to the first operand, 0.5 for sums and epilogue, 0.5
// to 1 for the stores to drain and 1.5 for the counters, the sum of the splits, and the 10 us in which the gate / up and
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
// All kPersistGrid workgroups have to be resident at once.  The host sees to that: one workgroup per CU, no second persistent launch
// under way on the device (PersistentTurn), and a wait that outlasts its limit ends the launch with MTMC_DATA_STALLED.
#include <type_traits>

#include "attention_decode.h"
#include "bf16_kernels.h"
#include "device_utils.h"
#include "frag.h"

namespace mtmc {
namespace bf16 {

namespace {

constexpr int kComputeWaves = AW, kControlWaves = 4, kThreads = (kComputeWaves + kControlWaves) * 64;
constexpr int kItems = 48;     // sums of 16 x 16 values that a phase hands over at once
constexpr int kMaxParts = 64;  // partial sums of a row's squares
constexpr int kHeadDim = 128;

// ---- device-scope accesses: past the caches that other dies do not see
using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr int kDeviceScope = 16;  // sc1
constexpr int kReach = 0x40000000;  // bytes that a descriptor covers; every buffer of a step is smaller
__device__ __forceinline__ Rsrc rsrc_of(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kReach, 0x00027000);
}
// Where a lane finds its part of an operand tile: lanes of rows that hold nothing point past the end of the descriptor, which
// gives zeros without a trip to memory (one row of 16: a tile is 64 bytes instead of 1 KiB).
__device__ __forceinline__ int operand_offset(int lane, int B) { return (lane & 15) < B ? lane * 16 : kReach; }
__device__ __forceinline__ v4u ld16(Rsrc r, int lane_off, int off) {
  return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, kDeviceScope));
}
__device__ __forceinline__ v4f ld16f(Rsrc r, int lane_off, int off) { return __builtin_bit_cast(v4f, ld16(r, lane_off, off)); }
__device__ __forceinline__ void st16(Rsrc r, int lane_off, int off, v4u v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, lane_off, off, kDeviceScope);
}
__device__ __forceinline__ float ld4(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st4(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint2 ld8(const void* p) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void st8(void* p, uint2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), (uint64_t)v.y << 32 | v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Weights: read once per step, past what the caches hold for the rest (one row: 64.0 -> 62.7 ms of 63 steps, 16 rows 77.0 ->
// 74.9, together with the fourth k tile in flight of the gate / up stream).
__device__ __forceinline__ v8h load_weight(const h16_t* tile, int lane) {
  return __builtin_bit_cast(v8h, __builtin_nontemporal_load(reinterpret_cast<const v4u*>(tile + lane * 8)));
}
// A uniform value that is to be in a register from here on.
template <class T>
__device__ __forceinline__ T keep(T v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Workgroup barrier that orders LDS only: weight loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct Shared {
  v4f red[kItems][64];  // sums per range of K, as the accumulators lie in the lanes
  struct {              // attention: rotated queries, this position's key and value, the wavefronts' results, the page ids
    __attribute__((aligned(16))) h16_t q[16][kHeadDim], k[kHeadDim], v[kHeadDim];
    float o[AW][AGMAX][kHeadDim + 1];
    float m[AW][16], l[AW][16];
    int table[ATAB];
  } at;
  float ml[kComputeWaves][2][8][16];     // per wavefront, head in hand, chunk and row: the chunk's rescaled sum
  float share[kComputeWaves][2][8][16];  // ... and its share
  float part[2][16][kMaxParts + 4];
  float scale[16];
  int arrived, stop;
};

// ---- the weight stream of one wavefront: NB row tiles and one tile of 16 rows over k tiles [k0, k1), PF k tiles ahead.
// start() takes the weights only and may run before the operand exists.  An empty range loads a tile that nobody multiplies
// (last: the last k tile there is): with a branch around the loads their registers would be taken for live everywhere.
template <int NB, int PF>
struct Stream {
  const h16_t* wp[NB];
  int k0, k1, top, lane, xoff;
  v8h wr[PF][NB], xr[PF];

  __device__ __forceinline__ void start(const h16_t* const (&rows)[NB], int k0_, int k1_, int last, int lane_, int B) {
    xoff = operand_offset(lane_, B);
    k0 = k0_;
    k1 = k1_;
    top = min(max(k0, k1 - 1), last);
    lane = lane_;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wp[nb] = rows[nb];
#pragma unroll
    for (int s = 0; s < PF; ++s) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) wr[s][nb] = load_weight(wp[nb] + (size_t)min(k0 + s, top) * 512, lane);
    }
  }
  __device__ __forceinline__ v8h operand(Rsrc x, int k) const { return __builtin_bit_cast(v8h, ld16(x, xoff, k * 1024)); }
  __device__ __forceinline__ void operands(Rsrc x) {
#pragma unroll
    for (int s = 0; s < PF; ++s) xr[s] = operand(x, min(k0 + s, top));
  }
  __device__ __forceinline__ void run(Rsrc x, v4f (&acc)[NB]) {
    int ks = k0;
    for (; ks + 2 * PF <= k1; ks += PF) {  // every slot that is multiplied is refilled (no load behind a branch)
#pragma unroll
      for (int s = 0; s < PF; ++s) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma16(wr[s][nb], xr[s], acc[nb]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) wr[s][nb] = load_weight(wp[nb] + (size_t)(ks + s + PF) * 512, lane);
        xr[s] = operand(x, ks + s + PF);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    for (; ks < k1; ks += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        if (ks + s < k1) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma16(wr[s][nb], xr[s], acc[nb]);
          const int kn = ks + s + PF;
          if (kn < k1) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) wr[s][nb] = load_weight(wp[nb] + (size_t)kn * 512, lane);
            xr[s] = operand(x, kn);
          }
        }
      }
    }
  }
};

__device__ __forceinline__ float silu_p(float g) { return g / (1.0f + expf(-g)); }

// Sum of S ranges of a tile, in range order.
template <int S>
__device__ __forceinline__ v4f sum_ranges(const Shared& sh, int first, int lane) {
  v4f v[S], sum = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < S; ++s) v[s] = sh.red[first + s][lane];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[r] += v[s][r];
  return sum;
}

// What a wavefront knows of the launch.
struct Ctx {
  const PersistArgs& a;
  Shared& sh;
  int wg, wave, lane;
};
// The same as new to the compiler: it would otherwise work out the addresses of all phases ahead of the loop over the blocks
// and keep them, a thousand registers of them.
using KernArgs = const __attribute__((address_space(4))) PersistArgs*;
__device__ __forceinline__ Ctx fresh(Shared& sh, int wave) {
  KernArgs k = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
  int lane = threadIdx.x & 63, wg = blockIdx.x;
  asm volatile("" : "+s"(k), "+s"(wg), "+s"(wave), "+v"(lane));
  return Ctx{*(const PersistArgs*)k, sh, wg, wave, lane};
}

// ======================================================================================
// control wavefronts
// ======================================================================================
// Counts the workgroup in (one lane): the last of a group of 16 workgroups counts the group in, on eight words of which every
// workgroup watches one.  (Watchers and arrivals on the same words delay each other: with 128 workgroups that come 3 us after
// the others, a flat form of eight counters takes 2.7 us from the last arrival, this one 1.5; all at once 1.5 either way.)
__device__ __forceinline__ void count_in(const Ctx& c, uint32_t phase) {
  uint32_t* group = c.a.sync + (kPersistTops + (c.wg & 15)) * kPersistSyncStride;
  const uint32_t n = __hip_atomic_fetch_add(group, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (n + 1 == (phase + 1) * (kPersistGrid / 16)) {
#pragma unroll
    for (int t = 0; t < kPersistTops; ++t)
      __hip_atomic_fetch_add(c.a.sync + t * kPersistSyncStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
// Each control wavefront drains its own stores, the last one of the four counts the workgroup in.
__device__ __forceinline__ void arrive(const Ctx& c, uint32_t phase) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  if (c.lane == 0) {
    const int n = __hip_atomic_fetch_add(&c.sh.arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (n % kControlWaves == kControlWaves - 1) count_in(c, phase);
  }
}
// One wavefront: until every workgroup has been counted `phase` times, or the wait's limit has passed anywhere (then false).
__device__ __forceinline__ bool wait_grid(const Ctx& c, uint32_t phase) {
  const uint32_t want = phase * 16;
  const uint32_t* p = c.a.sync + (c.wg % kPersistTops) * kPersistSyncStride;
  uint32_t* stalled = c.a.sync + kPersistStalled;
  const long long t0 = wall_clock64();
  bool ok = true;
  for (int i = 0;; ++i) {
    if ((uint32_t)__builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= want) break;
    if (wall_clock64() - t0 > c.a.wait_ticks ||
        (i % 16 == 15 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))) {
      if (c.lane == 0) {
        __hip_atomic_store(stalled, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicOr(c.a.err_flag, kErrStalled);
      }
      ok = false;
      break;
    }
  }
  asm volatile("" ::: "memory");
  return ok;
}
// Sums of squares by (row tile, row): [tile][row] as the other launches have them, or, inside the launch, [row][tile], where a
// row's tiles come with a few requests.
struct Squares {
  float* p;
  int tile, row;
};
__device__ __forceinline__ Squares squares(const PersistArgs& a, int which, bool inside) {
  return inside ? Squares{a.ss_in[which], 1, kPersistGrid} : Squares{a.ss[which], 16, 1};
}
// The row scales of a phase: 1/rms of the current residual and, TWO, times the rms that its operand was divided by.  P partial
// sums of the row's tiles (part p: tiles p, p + P, ...), then those in order: the order of a launch of 16 P threads.  The
// four control wavefronts take four rows each, all loads in one go; what they leave in sh.scale is read behind a barrier.
template <int P, bool TWO>
__device__ __forceinline__ void row_scales(const Ctx& c, Squares cur, Squares old) {
  const PersistArgs& a = c.a;
  const int cw = c.wave - kComputeWaves, m = cw * 4 + (c.lane >> 4), q = c.lane & 15;
  if (cw * 4 >= a.B) return;
  // lane group q: parts q, q + G, ... (PP of them), part p's tiles p + P k (K of them)
  constexpr int G = P == 20 ? 10 : 16, PP = P / G, K = P == 20 ? 5 : (kPersistGrid + P - 1) / P;
  float va[PP][K], vb[PP][K];
  if (P != 20 || q < G) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < PP; ++i) {
        const int t = min(q + G * i + P * k, a.nt_d - 1);
        va[i][k] = ld4(cur.p + t * cur.tile + m * cur.row);
        if (TWO) vb[i][k] = ld4(old.p + t * old.tile + m * old.row);
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
      c.sh.part[0][m][q + G * i] = sa;
      if (TWO) c.sh.part[1][m][q + G * i] = sb;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows are the wavefront's own
  if (q == 0) {
    float ta = 0.f, tb = 0.f;
    v4f pa[P / 4], pb[P / 4];
#pragma unroll
    for (int p = 0; p < P / 4; ++p) {
      pa[p] = *reinterpret_cast<const v4f*>(&c.sh.part[0][m][4 * p]);
      if (TWO) pb[p] = *reinterpret_cast<const v4f*>(&c.sh.part[1][m][4 * p]);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
      ta += pa[p / 4][p % 4];
      if (TWO) tb += pb[p / 4][p % 4];
    }
    float sc = 1.0f / sqrtf(ta * a.inv_d + a.eps);
    if (TWO) sc *= sqrtf(tb * a.inv_d + a.eps);
    c.sh.scale[m] = sc;
  }
}

// Where a tile of the residual goes.
struct TileOut {
  Rsrc h;
  h16_t* x;
  Squares ss;
  float* ss_out;  // the same for the launches that follow, or NULL
  int* err_flag;
  int d, B;
  __device__ __forceinline__ TileOut(const PersistArgs& a, int which, bool last)
      : h(rsrc_of(keep(a.h))), x(keep(a.x)), ss{keep(a.ss_in[which]), 1, kPersistGrid}, ss_out(last ? a.ss[which] : nullptr), err_flag(keep(a.err_flag)), d(keep(a.d)), B(keep(a.B)) {}
};
// h += sum; x' = fp16(h gain r); the squares' sum of the tile.  Lane: row lane % 16, columns 4 (lane / 16) .. of tile nt.
__device__ __forceinline__ void residual_tile(const TileOut& to, int nt, int lane, v4f sum, v4f h_old, v4f gain, float sc) {
  const int m = lane & 15, rq = (lane >> 4) * 4, n = nt * 16 + rq;
  const bool live = m < to.B;
  v4f hv = h_old + sum;
  if (!live) hv = v4f{0.f, 0.f, 0.f, 0.f};
  bool out_of_range = false;
  uint2 pk;
  pk.x = pack_h16x2_track(hv[0] * gain[0] * sc, hv[1] * gain[1] * sc, out_of_range);
  pk.y = pack_h16x2_track(hv[2] * gain[2] * sc, hv[3] * gain[3] * sc, out_of_range);
  if (live) {
    st16(to.h, (m * to.d + n) * 4, 0, __builtin_bit_cast(v4u, hv));
    st8(to.x + act_off(m, n, 16), pk);
  }
  float ss = fmaf(hv[0], hv[0], hv[1] * hv[1]) + fmaf(hv[2], hv[2], hv[3] * hv[3]);  // rounded as in the separate launches
  ss += __shfl_xor(ss, 16, 64);
  ss += __shfl_xor(ss, 32, 64);
  if (lane < 16 && live) {
    st4(to.ss.p + nt * to.ss.tile + m * to.ss.row, ss);
    if (to.ss_out) st4(to.ss_out + nt * 16 + m, ss);
  }
  if (live && out_of_range) atomicOr(to.err_flag, kErrFp16Range);
}

// Which workgroup does what.  The O projection and the sum of the splits have a row tile for workgroups 0 .. nt_d - 1; the QKV
// tiles go to the others first (from the top down), the attention to those that start behind nt_d, and of the gate / up tiles
// a workgroup with an O tile takes one pair where the others can take the rest: it comes to them last.
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

// The unit of a workgroup in the attention phase, the same in every block: (sequence, kv head, chunk) and its place in the cache.
struct AttnUnit {
  int b, g, chunk;
  AttnDecRange r;
  bool there;   // the workgroup has a unit
  bool active;  // ... and its chunk holds a part of the context
  __device__ __forceinline__ AttnUnit(const PersistArgs& a, int wg) {
    const int place = attn_place(a, wg);
    there = place < a.attn_units;
    const int u = there ? place : 0;
    b = u % a.B;
    const int rest = u / a.B;
    g = rest % a.at.Hkv;
    chunk = rest / a.at.Hkv;
    r = attn_dec_pages(a.at, b, chunk);
    attn_dec_position(a.at, b, *a.at.d_step, r);
    r.lo = __builtin_amdgcn_readfirstlane(r.lo);  // the same in all lanes, which the compiler does not see
    r.hi = __builtin_amdgcn_readfirstlane(r.hi);
    r.pos = __builtin_amdgcn_readfirstlane(r.pos);
    active = there && r.lo < r.hi;
  }
};

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
  const int n_layers = fresh(sh, wave).a.n_layers;
  bool attends, attn_active;
  {
    const Ctx c = fresh(sh, wave);
    const AttnUnit u(c.a, c.wg);
    attends = u.there;
    attn_active = u.active;
  }
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection
    {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const int place = qkv_place(wg);
      const Rsrc out = rsrc_of(keep(a.qkv));
      const int nt_qkv = keep(a.nt_qkv), B = keep(a.B);
      if (!go(c)) return;
      if (l == 0) {
        if (lane < 4) sh.scale[cw * 4 + lane] = 1.f;
      } else if (place < nt_qkv) {
        row_scales<64, true>(c, squares(a, 0, true), squares(a, 1, true));
      }
      for (int u = 0; place + u * kPersistGrid < nt_qkv; ++u) {
        lds_barrier();
        if ((u & 3) == cw) {
          const int nt = place + u * kPersistGrid;
          const v4f sum = sum_ranges<16>(sh, (u & 1) * 16, lane);
          if (m < B) st16(out, ((m * nt_qkv + nt) * 16 + rq) * 4, 0, __builtin_bit_cast(v4u, sum * sh.scale[m]));
        }
      }
      arrive(c, phase);
      lds_barrier();
      ++phase;
    }
    // ---- attention
    {
      const Ctx c = fresh(sh, wave);
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
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const bool has_tile = wg < a.nt_d;
      const TileOut to(a, 1, l + 1 == n_layers);
      const int ranges = keep(a.o_ranges);
      v4f h_old = v4f{0.f, 0.f, 0.f, 0.f}, gain = h_old;
      if (lead && has_tile) {
        h_old = ld16f(to.h, (min(m, to.B - 1) * to.d + wg * 16 + rq) * 4, 0);
        gain = *reinterpret_cast<const v4f*>((const float*)((const char*)a.ffn_norm + l * a.layer_stride) + wg * 16 + rq);
      }
      if (!go(c)) return;
      if (has_tile) {
        const Squares cur = squares(a, 0, l > 0);
        if (ranges == 16) row_scales<64, false>(c, cur, cur);
        else if (ranges == 12) row_scales<48, false>(c, cur, cur);
        else row_scales<32, false>(c, cur, cur);
        lds_barrier();
        if (lead) {
          loads_done();
          const v4f sum = ranges == 16 ? sum_ranges<16>(sh, 0, lane) : ranges == 12 ? sum_ranges<12>(sh, 0, lane) : sum_ranges<8>(sh, 0, lane);
          residual_tile(to, wg, lane, sum, h_old, gain, sh.scale[m]);
        }
      }
      arrive_lead(c);
      lds_barrier();
      ++phase;
    }
    // ---- gate / up projection
    {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      h16_t* const act = keep(a.act);
      const int nt_gu = keep(a.nt_gu), B = keep(a.B);
      int* const err_flag = keep(a.err_flag);
      if (!go(c)) return;
      const GuShare<GU_TILES> share(a, wg);
      if (share.first < nt_gu) {
        row_scales<4 * kGuRanges, true>(c, squares(a, 1, true), squares(a, 0, l > 0));
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
      arrive(c, phase);
      lds_barrier();
      ++phase;
    }
    // ---- down projection: sums per split of K
    {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const Rsrc out = rsrc_of(keep(a.part));
      const int d = keep(a.d), nt_d = keep(a.nt_d), B = keep(a.B), ks = keep(a.ks_down), batches = keep(a.dn_batches);
      if (!go(c)) return;
      if (wg < nt_d) row_scales<4 * DN_RANGES, false>(c, squares(a, 1, true), squares(a, 1, true));
      for (int bt = 0; bt < batches; ++bt) {
        lds_barrier();
        const int first = (DN_RANGES == 5 ? (bt & 1) * 16 : 0) + cw * DN_RANGES;
        int split, tile;
        bool mine;
        if (DN_RANGES == 5) {
          const int id = wg + kPersistGrid * (3 * bt + cw);
          split = id & 7;
          tile = id >> 3;
          mine = cw < 3;
        } else {
          constexpr int kTiles = DN_RANGES == 8 ? 2 : 4;
          split = wg % ks;
          tile = wg / ks * kTiles + cw;
          mine = cw < kTiles;
        }
        if (mine && tile < nt_d) {
          const v4f sum = sum_ranges<DN_RANGES>(sh, first, lane);
          if (m < B) st16(out, ((split * 16 + m) * d + tile * 16 + rq) * 4, 0, __builtin_bit_cast(v4u, sum));
        }
      }
      arrive(c, phase);
      lds_barrier();
      ++phase;
    }
    // ---- sum of the splits, residual, operand of the next block: the lead alone
    if (lead) {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const bool has_tile = wg < a.nt_d;
      const TileOut to(a, 0, l + 1 == n_layers);
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
        residual_tile(to, wg, lane, sum, h_old, gain, sh.scale[m]);
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
  const int n_layers = fresh(sh, wave).a.n_layers;
  // what the attention needs and no block changes: the unit, its page ids, the rotation of its position
  int u_b, u_g, u_chunk, u_pos, u_lo, u_hi, id0, id1;
  bool attends, attn_active;
  float rope_c, rope_s;
  {
    const Ctx c = fresh(sh, wave);
    const PersistArgs& a = c.a;
    const AttnUnit u(a, c.wg);
    u_b = u.b; u_g = u.g; u_chunk = u.chunk; u_pos = u.r.pos; u_lo = u.r.lo; u_hi = u.r.hi;
    attends = u.there;
    attn_active = u.active;
    const int* table = a.at.pool.page_table + (size_t)u_b * a.at.pool.max_pages;
    const int tid = wave * 64 + c.lane, last = a.at.pool.max_pages - 1;
    if (attn_active)
      for (int i = tid; i < u_hi - u_lo; i += AW * 64) sh.at.table[i] = table[u_lo + i];
    id0 = __builtin_amdgcn_readfirstlane(table[min(u_lo + 2 * wave, last)]);
    id1 = __builtin_amdgcn_readfirstlane(table[min(u_lo + 2 * wave + 1, last)]);
    const int pos = max(u_pos, 0), half = kHeadDim / 2;
    rope_c = a.at.cos[(size_t)pos * half + c.lane];
    rope_s = a.at.sin[(size_t)pos * half + c.lane];
    if (attends && !attn_active) {
      // a chunk beyond the context contributes nothing, which its consumer learns from a zero sum; its part of the operand
      // is cleared so that stale bits never meet a zero weight.  Once: nobody writes it in this launch.
      const int G = a.at.Hq / a.at.Hkv;
      if (tid < G * (kHeadDim / 8)) {
        const int h = tid / (kHeadDim / 8), d0 = (tid % (kHeadDim / 8)) * 8;
        h16_t* o = a.at.o + u_chunk * a.at.o_chunk_stride + act_off(u_b, (u_g * G + h) * kHeadDim + d0, 16);
        st8(o, make_uint2(0u, 0u));
        st8(o + 4, make_uint2(0u, 0u));
        if (d0 == 0) st8(a.at.ml + (((size_t)u_b * a.at.Hq + u_g * G + h) * a.at.n_chunks + u_chunk) * 2, make_uint2(0xff800000u, 0u));
      }
    }
  }
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection: one row tile at a time, 16 ranges of K, two per wavefront
    {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane;
      const h16_t* W = a.wqkv + (size_t)l * a.layer_stride / sizeof(h16_t);
      const Rsrc xr = rsrc_of(keep(a.x));
      const int kt_d = keep(a.kt_d), nt_qkv = keep(a.nt_qkv), B = keep(a.B), per = (kt_d + 15) / 16;
      Stream<1, 4> s0, s1;
      auto start = [&](int nt) {
        const h16_t* rows[1] = {W + (size_t)nt * kt_d * 512};
        s0.start(rows, w * per, min(kt_d, (w + 1) * per), kt_d - 1, lane, B);
        s1.start(rows, (w + 8) * per, min(kt_d, (w + 9) * per), kt_d - 1, lane, B);
      };
      int nt = qkv_place(wg);
      if (nt < nt_qkv) {
        start(nt);
        if (!go()) return;
        for (int u = 0;; ++u) {
          v4f a0[1] = {zero}, a1[1] = {zero};
          s0.operands(xr);
          s1.operands(xr);
          s0.run(xr, a0);
          s1.run(xr, a1);
          sh.red[(u & 1) * 16 + w][lane] = a0[0];
          sh.red[(u & 1) * 16 + w + 8][lane] = a1[0];
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
    if (!attn_active) {
      if (!go()) return;
      if (attends) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
      }
    } else {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, lane = c.lane, tid = w * 64 + lane, col = lane & 15, lg = lane >> 4;
      const int Hq = a.at.Hq, Hkv = a.at.Hkv, G = Hq / Hkv;
      const KvPool& pool = a.at.pool;
      const h16_t* kbase = dec_page<kHeadDim>(pool, l, 0, 0, u_g);
      const h16_t* vbase = dec_page<kHeadDim>(pool, l, 1, 0, u_g);
      const size_t pstride = (size_t)pool.n_kv_heads * (kPageTokens * kHeadDim);
      const int pg0 = u_lo + 2 * w;
      // the first pair of pages is of earlier steps, but for the current position, which is put in below
      KvFrags<kHeadDim> cur = load_kv<kHeadDim>(kbase + id0 * pstride, kbase + id1 * pstride, vbase + id0 * pstride,
                                                vbase + id1 * pstride, lane);
      const float* row = keep(a.at.qkv) + (size_t)u_b * (Hq + 2 * Hkv) * kHeadDim;
      int* const err_flag = keep(a.err_flag);
      const int n_chunks = keep(a.at.n_chunks);
      h16_t* const out = keep(a.at.o) + u_chunk * a.at.o_chunk_stride;
      float* const ml = keep(a.at.ml);
      if (!go()) return;
      const int cur_page = u_pos / kPageTokens, slot = u_pos % kPageTokens;
      const bool owner = cur_page >= u_lo && cur_page < u_hi;
      const bool appends = owner && w == AW - 1;
      auto rot = [&](float x, float y, float s) { return fmaf(x, rope_c, y * s); };  // rounded as in k_attn_dec
      {
        const float* qp = row + (size_t)(u_g * G + min(w, G - 1)) * kHeadDim;
        const float* kp = row + (size_t)(Hq + u_g) * kHeadDim;
        const float* vp = kp + (size_t)Hkv * kHeadDim;
        const float q0 = ld4(qp + lane), q1 = ld4(qp + lane + 64);
        if (appends) {
          const float x0 = ld4(kp + lane), x1 = ld4(kp + lane + 64), v0 = ld4(vp + lane), v1 = ld4(vp + lane + 64);
          const h16_t k0 = f32_to_h16_flag(rot(x0, x1, -rope_s), err_flag), k1 = f32_to_h16_flag(rot(x1, x0, rope_s), err_flag);
          const h16_t y0 = f32_to_h16_flag(v0, err_flag), y1 = f32_to_h16_flag(v1, err_flag);
          sh.at.k[lane] = k0; sh.at.k[lane + 64] = k1;
          sh.at.v[lane] = y0; sh.at.v[lane + 64] = y1;
          const size_t page = (size_t)sh.at.table[cur_page - u_lo] * pstride;
          h16_t* kd = const_cast<h16_t*>(kbase) + page;
          h16_t* vd = const_cast<h16_t*>(vbase) + page;
          kd[(lane >> 3) * 128 + slot * 8 + (lane & 7)] = k0;
          kd[((lane + 64) >> 3) * 128 + slot * 8 + (lane & 7)] = k1;
          vd[lane * kPageTokens + slot] = y0;
          vd[(lane + 64) * kPageTokens + slot] = y1;
        }
        if (w < G) {
          sh.at.q[w][lane] = f32_to_h16_flag(rot(q0, q1, -rope_s), err_flag);
          sh.at.q[w][lane + 64] = f32_to_h16_flag(rot(q1, q0, rope_s), err_flag);
        }
      }
      lds_barrier();
      v8h qf[kHeadDim / 32];
#pragma unroll
      for (int kb = 0; kb < kHeadDim / 32; ++kb) {
        v4u raw = {0u, 0u, 0u, 0u};
        if (col < G) raw = *reinterpret_cast<const v4u*>(&sh.at.q[col][kb * 32 + 8 * lg]);
        qf[kb] = __builtin_bit_cast(v8h, raw);
      }
      const int qpos = (col < G) ? u_pos : -1;
      AttnState<kHeadDim / 16> st;
      attn_init(st);
      const float scale2 = 0.08838834764831845f * 1.4426950408889634f;  // log2(e) / sqrt(head_dim)
      const int n_st = pg0 < u_hi ? (u_hi - pg0 + 2 * AW - 1) / (2 * AW) : 0;
      auto page_id = [&](int pg) { return (size_t)sh.at.table[min(pg, u_hi - 1) - u_lo] * pstride; };
      // one register set, each half refilled as soon as it is used; a stage that another one follows lies wholly before the
      // position
      int j = 0;
      for (; j + 1 < n_st; ++j) {
        const int pg = pg0 + 2 * AW * (j + 1);
        const size_t o0 = page_id(pg), o1 = page_id(pg + 1);
        const v8h pf = attn_weights1<kHeadDim, false>(cur, (pg0 + 2 * AW * j) * kPageTokens, qf, qpos, scale2, st, lane);
        load_keys<kHeadDim>(cur, kbase + o0, kbase + o1, lane);
        attn_values1<kHeadDim>(cur, pf, st);
        load_values<kHeadDim>(cur, vbase + o0, vbase + o1, lane);
      }
      if (j < n_st) {
        const int pg = pg0 + 2 * AW * j, p = cur_page - pg;
        if (owner && (p == 0 || p == 1)) {
          // the current position's key and value, whatever the load saw of the append
          if (col == slot) {
#pragma unroll
            for (int kb = 0; kb < kHeadDim / 32; ++kb) {
              const v8h k = *reinterpret_cast<const v8h*>(&sh.at.k[kb * 32 + 8 * lg]);
              if (p == 0) cur.k[0][kb] = k;
              else cur.k[1][kb] = k;
            }
          }
          if (lg == slot >> 2) {
            const uint32_t shift = (slot & 1) * 16, mask = 0xffffu << shift;
#pragma unroll
            for (int cb = 0; cb < kHeadDim / 16; ++cb) {
              const uint32_t v = (uint32_t)sh.at.v[cb * 16 + col] << shift;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (e == p * 2 + ((slot & 3) >> 1)) cur.v[cb][e] = (cur.v[cb][e] & ~mask) | v;
            }
          }
        }
        attn_step1<kHeadDim, true>(cur, pg * kPageTokens, qf, qpos, scale2, st, lane);
      }
      float sum_l = st.l;
      sum_l += __shfl_xor(sum_l, 16, 64);
      sum_l += __shfl_xor(sum_l, 32, 64);
      if (col < AGMAX) {
#pragma unroll
        for (int cb = 0; cb < kHeadDim / 16; ++cb)
#pragma unroll
          for (int r = 0; r < 4; ++r) sh.at.o[w][col][cb * 16 + 4 * lg + r] = st.o[cb][r];
      }
      if (lg == 0) {
        sh.at.m[w][col] = st.m;
        sh.at.l[w][col] = sum_l;
      }
      lds_barrier();
      // merge the wavefronts: thread t < 16 G owns (head h, 8 consecutive dims)
      if (tid < G * (kHeadDim / 8)) {
        const int h = tid / (kHeadDim / 8), d0 = (tid % (kHeadDim / 8)) * 8;
        float mm = -INFINITY, ll = 0.f, acc[8] = {};
#pragma unroll
        for (int v = 0; v < AW; ++v) mm = fmaxf(mm, sh.at.m[v][h]);
#pragma unroll
        for (int v = 0; v < AW; ++v) {
          const float f = __builtin_amdgcn_exp2f(sh.at.m[v][h] - mm);
          ll += f * sh.at.l[v][h];
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] += f * sh.at.o[v][h][d0 + e];
        }
        const float inv = 1.0f / ll;  // every page of an active chunk holds at least one visible key
        uint32_t pk[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = pack_h16x2_flag(acc[2 * e] * inv, acc[2 * e + 1] * inv, err_flag);
        h16_t* o = out + act_off(u_b, (u_g * G + h) * kHeadDim + d0, 16);
        st8(o, make_uint2(pk[0], pk[1]));
        st8(o + 4, make_uint2(pk[2], pk[3]));
        if (n_chunks > 1 && d0 == 0)
          st8(ml + (((size_t)u_b * Hq + u_g * G + h) * n_chunks + u_chunk) * 2,
              make_uint2(__float_as_uint(mm * 0.6931471805599453f), __float_as_uint(ll)));  // the consumer works in natural units
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_barrier();
    }
    counted_in();
    // ---- O projection
    {
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane, kt_nq = keep(a.kt_nq), B = keep(a.B);
      const h16_t* W = a.wo + (size_t)l * a.layer_stride / sizeof(h16_t) + (size_t)wg * kt_nq * 512;
      const Rsrc xr = rsrc_of(keep(a.at.o));
      const int R = keep(a.o_ranges), NC = keep(a.at.n_chunks);
      if (wg >= a.nt_d) {
        if (!go()) return;
      } else if (NC == 1) {
        const int per = (kt_nq + R - 1) / R;
        const h16_t* rows[1] = {W};
        Stream<1, 4> s0, s1;
        s0.start(rows, w * per, min(kt_nq, (w + 1) * per), kt_nq - 1, lane, B);
        s1.start(rows, (w + 8) * per, min(kt_nq, (w + 9) * per), kt_nq - 1, lane, B);
        if (!go()) return;
        v4f a0[1] = {zero}, a1[1] = {zero};
        s0.operands(xr);
        s1.operands(xr);
        s0.run(xr, a0);
        s1.run(xr, a1);  // empty with 8 ranges
        sh.red[w][lane] = a0[0];
        sh.red[w + 8][lane] = a1[0];
        lds_barrier();
      } else {
        // The chunks of the context are combined here, head by head: out += sum_chunk share * (W_head . o_chunk), share =
        // l exp(m - max m) / sum l exp(m - max m).  Range v takes heads v, v + R, ...; this wavefront ranges w and (12
        // ranges) w + 8: its list of heads, two in hand at a time, up to five (head, chunk) operands on their way at once (six do not
        // fit the registers).
        constexpr int kItemsAhead = 5;
        const int n_heads = keep(a.at.Hq), col = lane & 15, lg = lane >> 4, xoff = operand_offset(lane, B);
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
              for (int t = 0; t < 4; ++t) xf[q][t] = __builtin_bit_cast(v8h, ld16(xr, xoff, off + t * 1024));
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
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, lane = c.lane;
      constexpr int kRanges = GU_TILES == 6 ? 8 : 4;
      const GuShare<GU_TILES> share(a, c.wg);
      const int kt_d = keep(a.kt_d), nt_gu = keep(a.nt_gu), B = keep(a.B), first = keep(share.first);
      const int per = (kt_d + kRanges - 1) / kRanges, s = w % kRanges;
      const h16_t* W = a.wgu + (size_t)l * a.layer_stride / sizeof(h16_t);
      const Rsrc xr = rsrc_of(keep(a.x));
      // kTiles row tiles of this wavefront from tile first + j0 on
      auto multiply = [&](auto tiles_per_wave, auto depth) {
        constexpr int kTiles = decltype(tiles_per_wave)::value, PF = decltype(depth)::value;
        const int j0 = (w / kRanges) * kTiles;
        const h16_t* rows[kTiles];
#pragma unroll
        for (int i = 0; i < kTiles; ++i) rows[i] = W + (size_t)min(first + j0 + i, nt_gu - 1) * kt_d * 512;
        Stream<kTiles, PF> st;
        st.start(rows, s * per, min(kt_d, (s + 1) * per), kt_d - 1, lane, B);
        if (!go()) return false;
        v4f acc[kTiles];
#pragma unroll
        for (int i = 0; i < kTiles; ++i) acc[i] = zero;
        st.operands(xr);
        st.run(xr, acc);
#pragma unroll
        for (int i = 0; i < kTiles; ++i) sh.red[(j0 + i) * kRanges + s][lane] = acc[i];
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
      const Ctx c = fresh(sh, wave);
      const PersistArgs& a = c.a;
      const int w = c.wave, wg = c.wg, lane = c.lane;
      const h16_t* W = a.wdown + (size_t)l * a.layer_stride / sizeof(h16_t);
      const Rsrc xr = rsrc_of(keep(a.act));
      const int kt_F = keep(a.kt_F), nt_d = keep(a.nt_d), ks = keep(a.ks_down), batches = keep(a.dn_batches), B = keep(a.B);
      const int per_split = (kt_F + ks - 1) / ks;
      if constexpr (DN_RANGES == 5) {
        // 8 splits, split = workgroup % 8; three row tiles at a time: 15 (tile, range) items over 8 wavefronts
        const int kbeg = (wg & 7) * per_split, kend = min(kt_F, kbeg + per_split);
        const int per = (max(kend - kbeg, 0) + 4) / 5;
        Stream<1, 7> s0, s1;
        auto start1 = [&](Stream<1, 7>& s, int item, int bt) {
          const int i = item / 5, r = item - i * 5, id = wg + kPersistGrid * (3 * bt + i), tile = id >> 3;
          const h16_t* rows[1] = {W + (size_t)min(tile, nt_d - 1) * kt_F * 512};
          const bool there = item < 15 && tile < nt_d;
          const int k0 = kbeg + r * per;
          s.start(rows, k0, there ? min(kend, k0 + per) : k0, kt_F - 1, lane, B);
        };
        start1(s0, w, 0);
        start1(s1, w + 8, 0);
        if (!go()) return;
        for (int bt = 0;;) {
          v4f a0[1] = {zero}, a1[1] = {zero};
          s0.operands(xr);
          s1.operands(xr);
          s0.run(xr, a0);
          s1.run(xr, a1);
          sh.red[(bt & 1) * 16 + w][lane] = a0[0];
          sh.red[(bt & 1) * 16 + w + 8][lane] = a1[0];
          lds_barrier();
          if (++bt >= batches) break;
          start1(s0, w, bt);
          start1(s1, w + 8, bt);
        }
      } else {
        // groups of 2 tiles and 8 ranges or of 4 tiles and 4 ranges, one (group, split) per workgroup
        constexpr int kTiles = DN_RANGES == 8 ? 2 : 4;
        const int split = wg % ks, t0 = wg / ks * kTiles, s = w % DN_RANGES, j0 = (w / DN_RANGES) * 2;
        const int kbeg = split * per_split, kend = min(kt_F, kbeg + per_split);
        const int per = (max(kend - kbeg, 0) + DN_RANGES - 1) / DN_RANGES, k0 = kbeg + s * per;
        const h16_t* rows[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) rows[i] = W + (size_t)min(t0 + j0 + i, nt_d - 1) * kt_F * 512;
        Stream<2, 6> st;
        st.start(rows, k0, t0 < nt_d ? min(kend, k0 + per) : k0, kt_F - 1, lane, B);
        if (!go()) return;
        v4f acc[2] = {zero, zero};
        st.operands(xr);
        st.run(xr, acc);
#pragma unroll
        for (int i = 0; i < 2; ++i) sh.red[(j0 + i) * DN_RANGES + s][lane] = acc[i];
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
void launch_gu(const PersistArgs& a, int dn_ranges, hipStream_t st) {
  switch (dn_ranges) {
    case 5: k_decode_layers<GU_TILES, 5><<<kPersistGrid, kThreads, 0, st>>>(a); break;
    case 8: k_decode_layers<GU_TILES, 8><<<kPersistGrid, kThreads, 0, st>>>(a); break;
    default: k_decode_layers<GU_TILES, 4><<<kPersistGrid, kThreads, 0, st>>>(a); break;
  }
}
// Gate / up row tiles per workgroup: one round on the 256 CUs with the ranges of K of the launch of its own (8 from 1025 to
// 1536 tiles, else 4).
int gu_tiles(int nt_gu) { return nt_gu <= 4 * 256 ? 4 : nt_gu <= 6 * 256 ? 6 : nt_gu <= 10 * 256 ? 10 : 0; }

}  // namespace

bool decode_persistent_fits(const PersistShape& s) {
  // one tile of rows; 16 ranges of K in the QKV projection and one O tile per workgroup; a down projection of one unit per
  // workgroup or in batches of three; one attention unit per
  // workgroup
  return s.m_tiles == 1 && s.head_dim == 128 && s.kt_d >= 48 && s.nt_d <= kPersistGrid && gu_tiles(s.nt_gu) > 0 &&
         s.n_chunks <= 8 && s.pairs * s.n_chunks <= kPersistGrid;
}

void decode_persistent(const PersistArgs& a, int down_nb, hipStream_t st) {
  const int dn_ranges = down_nb == 3 ? 5 : down_nb == 2 ? 8 : 4;
  switch (gu_tiles(a.nt_gu)) {
    case 4: launch_gu<4>(a, dn_ranges, st); break;
    case 6: launch_gu<6>(a, dn_ranges, st); break;
    default: launch_gu<10>(a, dn_ranges, st); break;
  }
}

}  // namespace bf16
}  // namespace mtmc
