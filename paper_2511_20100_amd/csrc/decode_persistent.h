// Pieces of the persistent decode step (decode_persistent.hip: one tile of 16 rows; decode_persistent_rows.hip: two to four):
// how its workgroups hand data to each other, how they wait for each other, and the sums that both forms make alike.
//
// What one workgroup writes and another reads goes past the caches that are not coherent between the dies: device-scope (sc1)
// stores, drained before the workgroup is counted in (where readers wait for the counters), and device-scope loads, or plain ones
// where Operand says why.
#pragma once

#include "attention_decode.h"
#include "bf16_kernels.h"
#include "device_scope.h"
#include "device_utils.h"
#include "frag.h"
#include "roll_call.h"

namespace mtmc {
namespace bf16 {
namespace persist {

constexpr int kHeadDim = 128;

using namespace device_scope;  // every buffer of a step is smaller than a descriptor's reach

// Weights: read once per step, past what the caches hold for the rest (one row: 64.0 -> 62.7 ms of 63 steps, 16 rows 77.0 ->
// 74.9, together with the fourth k tile in flight of the gate / up stream).
__device__ __forceinline__ v8h load_weight(const h16_t* tile, int lane) {
  return __builtin_bit_cast(v8h, __builtin_nontemporal_load(reinterpret_cast<const v4u*>(tile + lane * 8)));
}
__device__ __forceinline__ v8h load_weight(Rsrc r, int lane_off, int off) {
  constexpr int kNonTemporal = 2;
  return __builtin_bit_cast(v8h, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, kNonTemporal));
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

// ---- readers that ask for the data themselves.  A word that nobody has written yet holds kNotThere, and a reader asks again, past
// the caches, until no word of what it needs does.  An fp16 pair is never that word (the converters saturate), an fp32 value
// only as a NaN that no instruction makes; written() turns that one into another NaN.
constexpr uint32_t kNotThere = 0xffffffffu;
__device__ __forceinline__ uint32_t written(uint32_t w) { return min(w, kNotThere - 1); }
__device__ __forceinline__ v4u written(v4f v) {
  const v4u w = __builtin_bit_cast(v4u, v);
  return v4u{written(w[0]), written(w[1]), written(w[2]), written(w[3])};
}
__device__ __forceinline__ uint32_t largest(v4u w) { return max(max(w[0], w[1]), max(w[2], w[3])); }

// The operand of MU tiles of 16 rows, fragment-tiled.  The operands of the QKV, gate / up and down projections are read through
// the caches (SCOPE 0): every block of the step has buffers of its own for them, so no line of them is in a cache before it has
// been written, and no line is written by two workgroups (a row tile's 16 columns of 16 rows are 512 bytes).  Past the caches
// (SCOPE kDeviceScope) all CUs together get the 7 TB/s of the memory side.  That is how the attention's output is read: eight
// rows of it, of as many workgroups, share a line.  Lanes of rows that hold nothing point past the end of the descriptor,
// which gives zeros without a trip to memory.
template <int MU, int SCOPE = 0>
struct Operand {
  Rsrc r;
  int off[MU], step;
  // fragment-tiled [k tile][tile of rows][lane]
  __device__ __forceinline__ static Operand tiled(const void* p, int bt, int mt0, int lane, int B) {
    Operand x;
    x.r = rsrc_of(p);
    x.step = bt * 1024;
#pragma unroll
    for (int i = 0; i < MU; ++i) x.off[i] = (mt0 + i) * 16 + (lane & 15) < B ? (mt0 + i) * 1024 + lane * 16 : kReach;
    return x;
  }
  // one tile whose pieces hold `rows` rows (16: as tiled()); rows of fewer lie closer, fewer lines to ask for
  __device__ __forceinline__ static Operand packed(const void* p, int rows, int lane, int B) {
    static_assert(MU == 1, "");
    Operand x;
    x.r = rsrc_of(p);
    x.step = rows * 64;
    x.off[0] = (lane & 15) < B ? (lane >> 4) * (rows * 16) + (lane & 15) * 16 : kReach;
    return x;
  }
  __device__ __forceinline__ v8h load(int i, int at) const {
    return __builtin_bit_cast(v8h, __builtin_amdgcn_raw_buffer_load_b128(r, off[i], at, SCOPE));
  }
  __device__ __forceinline__ v8h tile(int i, int k) const { return load(i, k * step); }
};

// ---- the weight stream of one wavefront: NB row tiles and MU tiles of 16 rows over the steps 0 .. n - 1, step i being k tile
// k0 + i or, from step n0 on, k1 + i - n0 (two ranges of K one after the other); PF steps of weights and PFX of the operand
// ahead.  start() takes the weights only (w: the matrix, rows: where its row tiles begin, bytes) and may run before the operand
// exists.  No load is behind a branch, or its registers would be taken for live everywhere: what start() has no step for points
// past the descriptor, which costs no trip to memory.  last: the last k tile there is.
template <int NB, int MU, int PF, int PFX>
struct Stream {
  static_assert(PF % PFX == 0, "the weight ring must be a multiple of the operand ring");
  static constexpr int kOperandsAhead = PFX;
  Rsrc w;
  int rows[NB];
  int k0, k1, n0, n, last, lane;
  v8h wr[PF][NB], xr[PFX][MU];

  __device__ __forceinline__ int tile_of(int i) const {
    const int j = max(0, min(i, n - 1));
    return min(j < n0 ? k0 + j : k1 + j - n0, last);
  }
  __device__ __forceinline__ void weights(int s, int i, int lane_off) {
    const int k = tile_of(i);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wr[s][nb] = load_weight(w, lane_off, rows[nb] + k * 1024);
  }
  template <int SCOPE>
  __device__ __forceinline__ void operand(const Operand<MU, SCOPE>& x, int s, int i) {
    const int k = tile_of(i);
#pragma unroll
    for (int mu = 0; mu < MU; ++mu) xr[s][mu] = x.tile(mu, k);
  }
  __device__ __forceinline__ void start(Rsrc w_, const int (&rows_)[NB], int k0_, int n0_, int k1_, int n1_, int last_, int lane_) {
    k0 = k0_;
    k1 = k1_;
    n0 = max(n0_, 0);
    n = n0 + max(n1_, 0);
    last = last_;
    lane = lane_;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) rows[nb] = rows_[nb];
    w = w_;
#pragma unroll
    for (int s = 0; s < PF; ++s) weights(s, s, s < n ? lane * 16 : kReach);
  }
  template <int SCOPE>
  __device__ __forceinline__ void operands(const Operand<MU, SCOPE>& x) {
#pragma unroll
    for (int s = 0; s < PFX; ++s) {
      Operand<MU, SCOPE> y = x;
#pragma unroll
      for (int mu = 0; mu < MU; ++mu) y.off[mu] = s < n ? x.off[mu] : kReach;
      operand(y, s, s);
    }
  }
  __device__ __forceinline__ uint32_t largest_of(int s) const {
    uint32_t top = 0;
#pragma unroll
    for (int mu = 0; mu < MU; ++mu) top = max(top, largest(__builtin_bit_cast(v4u, xr[s][mu])));
    return top;
  }
  __device__ __forceinline__ uint32_t largest_ahead() const {
    uint32_t top = 0;
#pragma unroll
    for (int s = 0; s < PFX; ++s) top = max(top, largest_of(s));
    return top;
  }
  // operands() and run() over all steps, of an operand that is asked for until it is there; `asked`: the steps that ask() saw to
  template <int SCOPE, class Asker>
  __device__ __forceinline__ void ask(const Operand<MU, SCOPE>& x, const Asker& asker) {
    asker([&] {
      operands(x);
      return largest_ahead();
    });
  }
  template <int SCOPE, class Asker>
  __device__ __forceinline__ void run_asking(const Operand<MU, SCOPE>& x, const Asker& asker, v4f (&acc)[NB][MU], int asked) {
    auto ready = [&](int s, int i) {
      if (i >= asked && asker.missing(largest_of(s % PFX))) {
        asker([&] {
          operand(x, s % PFX, i);
          return largest_of(s % PFX);
        });
      }
    };
    int i = 0;
    for (; i + 2 * PF <= n; i += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        ready(s, i + s);
        multiply(s, acc);
        __builtin_amdgcn_sched_barrier(0);
        weights(s, i + s + PF, lane * 16);
        operand(x, s % PFX, i + s + PFX);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    for (; i < n; i += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        if (i + s < n) {
          ready(s, i + s);
          multiply(s, acc);
          if (i + s + PF < n) weights(s, i + s + PF, lane * 16);
          if (i + s + PFX < n) operand(x, s % PFX, i + s + PFX);
        }
      }
    }
  }
  __device__ __forceinline__ void multiply(int s, v4f (&acc)[NB][MU]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mu = 0; mu < MU; ++mu) acc[nb][mu] = mfma16(wr[s][nb], xr[s % PFX][mu], acc[nb][mu]);
  }
  // steps i0 .. i1 - 1 (i0 a multiple of PF)
  template <int SCOPE>
  __device__ __forceinline__ void run(const Operand<MU, SCOPE>& x, int i0, int i1, v4f (&acc)[NB][MU]) {
    int i = i0;
    for (; i + 2 * PF <= n && i + PF <= i1; i += PF) {  // every slot that is multiplied is refilled (no load behind a branch)
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        multiply(s, acc);
        __builtin_amdgcn_sched_barrier(0);
        weights(s, i + s + PF, lane * 16);
        operand(x, s % PFX, i + s + PFX);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    for (; i < i1; i += PF) {
#pragma unroll
      for (int s = 0; s < PF; ++s) {
        if (i + s < i1) {
          multiply(s, acc);
          if (i + s + PF < n) weights(s, i + s + PF, lane * 16);
          if (i + s + PFX < n) operand(x, s % PFX, i + s + PFX);
        }
      }
    }
  }
};
template <int NB, int MU>
__device__ __forceinline__ void clear(v4f (&acc)[NB][MU]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int mu = 0; mu < MU; ++mu) acc[nb][mu] = v4f{0.f, 0.f, 0.f, 0.f};
}

__device__ __forceinline__ float silu_p(float g) { return g / (1.0f + expf(-g)); }

// sum += S ranges, in range order; items stride apart
template <int S>
__device__ __forceinline__ void add_ranges(v4f& sum, const v4f (*red)[64], int first, int stride, int lane) {
  v4f v[S];
#pragma unroll
  for (int s = 0; s < S; ++s) v[s] = red[first + s * stride][lane];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[r] += v[s][r];
}

// What a wavefront knows of the launch.
struct Ctx {
  const PersistArgs& a;
  int wg, wave, lane;
};
// The same as new to the compiler: it would otherwise work out the addresses of all phases ahead of the loop over the blocks
// and keep them, a thousand registers of them.  The lane is a statement of its own: together with it the other outputs count as
// different from lane to lane, and every buffer load whose place depends on the wavefront becomes a loop over the lanes' values
// (162 such loops in the one-tile kernels, 294 in the others; 1.5 B blocks, 64 rows: 1533 -> 1521 us a step).
using KernArgs = const __attribute__((address_space(4))) PersistArgs*;
__device__ __forceinline__ Ctx fresh(int wave) {
  KernArgs k = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
  int lane = threadIdx.x & 63, wg = blockIdx.x;
  asm volatile("" : "+s"(k), "+s"(wg), "+s"(wave));
  asm volatile("" : "+v"(lane));
  return Ctx{*(const PersistArgs*)k, wg, wave, lane};
}

constexpr uint32_t kGroupOf = kPersistGrid / kPersistGroups;  // workgroups in a group
constexpr long long kWaitTicks = 60 * 100000000ll;  // what is waited for once all workgroups are there always comes
constexpr long long kAgainTicks = 2000;             // the roll call of a step after one that was given up
__device__ __forceinline__ Word word_of(const PersistArgs& a, int i) { return {a.sync + i * kPersistSyncStride}; }

// Counts the workgroup in (one lane): the last of a group of 16 workgroups counts the group in, on eight words of which every
// workgroup watches one.  (Watchers and arrivals on the same words delay each other: with 128 workgroups that come 3 us after
// the others, a flat form of eight counters takes 2.7 us from the last arrival, this one 1.5; all at once 1.5 either way.)
__device__ __forceinline__ void count_in(const Ctx& c, uint32_t phase) {
  if (!roll_call::count_in(word_of(c.a, kPersistTops + (c.wg & (kPersistGroups - 1))), kGroupOf, phase + 1)) return;
#pragma unroll
  for (int t = 0; t < kPersistTops; ++t) word_of(c.a, t).add(1);
}
__device__ __forceinline__ uint32_t look(Word word) { return __builtin_amdgcn_readfirstlane(word.load()); }
// One wavefront: until every workgroup has been counted `phase` times, or the launch is over (then false).
__device__ __forceinline__ bool wait_grid(const Ctx& c, uint32_t phase) {
  const uint32_t want = phase * kPersistGroups;
  const Word mine = word_of(c.a, c.wg % kPersistTops), ended = word_of(c.a, kPersistEnded);
  const long long t0 = wall_clock64();
  bool ok = true;
  for (int i = 0; look(mine) < want; ++i) {
    const bool late = wall_clock64() - t0 > kWaitTicks;
    if (late || (i % 16 == 15 && look(ended))) {
      if (late && c.lane == 0) {
        ended.store(kPersistLost);
        atomicOr(c.a.err_flag, kErrUnfinished);
      }
      ok = false;
      break;
    }
  }
  asm volatile("" ::: "memory");
  return ok;
}
// One wavefront asks until what load() brings is all there (load() gives the largest word of it), or the launch is over; *stop then.
struct Asker {
  const PersistArgs& a;
  int* stop;
  __device__ __forceinline__ static bool missing(uint32_t top) { return __builtin_amdgcn_ballot_w64(top == kNotThere) != 0; }
  template <class Load>
  __device__ __forceinline__ void operator()(Load load) const {
    long long t0 = 0;
    for (int i = 0; missing(load()); ++i) {
      asm volatile("" ::: "memory");  // the loads are made again
      if (i == 0) t0 = wall_clock64();
      if (i % 64 != 63) continue;
      const Word ended = word_of(a, kPersistEnded);
      const bool late = wall_clock64() - t0 > kWaitTicks;
      if (late || look(ended)) {
        if (late) {
          ended.store(kPersistLost);
          atomicOr(a.err_flag, kErrUnfinished);
        }
        *stop = 1;
        break;
      }
    }
  }
};
// Where nothing has to be asked for: the readers have waited for the counters.
struct Known {
  __device__ __forceinline__ static bool missing(uint32_t) { return false; }
  template <class Load>
  __device__ __forceinline__ void operator()(Load load) const { load(); }
};
// Behind the first phase, which hands nothing on but the rows of qkv, a workgroup that has waited longer than the limit gives the
// launch up for all of them, unless all are there (false).  It is over then for whoever waits now or comes later.
__device__ __forceinline__ bool give_up(const Ctx& c) {
  int closed = 0;
  if (c.lane == 0) {
    if (c.a.told) atomicOr(c.a.err_flag, kErrStalled);
    closed = roll_call::close([&](int g) { return word_of(c.a, kPersistTops + g); }, kPersistGroups, kGroupOf);
    if (closed) {
      Word{c.a.sync + kPersistGaveUp}.store(1);
      __hip_atomic_store(c.a.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      word_of(c.a, kPersistEnded).store(kPersistSkipped);
    }
  }
  return __builtin_amdgcn_readfirstlane(closed);
}

// 1/rms of the current residual and, where the operand was divided by an older one, times that one's rms
__device__ __forceinline__ float scale_of(float cur, float old, bool two, float inv_d, float eps) {
  float sc = 1.0f / sqrtf(cur * inv_d + eps);
  if (two) sc *= sqrtf(old * inv_d + eps);
  return sc;
}

// Where a tile of the residual goes.
struct TileOut {
  Rsrc h;
  h16_t* x;
  float* ss;
  float* ss_out;  // the same for the launches that follow, or NULL
  int* err_flag;
  int d, B;
  // the one-tile form: rows of a piece of x, and how often x and ss are written, each time that many bytes further on
  int x_rows, copies, x_copy, ss_copy;
  // ... the columns of a tile that have no row write the copies, at_once of them at a time: this lane those of `row` from `first` on
  int row, first, at_once;
  __device__ __forceinline__ TileOut(const PersistArgs& a, h16_t* x_, float* ss_, int which, int rows, int copies_, bool last, int lane)
      : h(rsrc_of(nullptr)), x(keep(x_)), ss(keep(ss_)), ss_out(last ? a.ss[which] : nullptr),
        err_flag(keep(a.err_flag)), d(keep(a.d)), B(keep(a.B)), x_rows(keep(rows)), copies(copies_), x_copy(a.at_hand.x_copy),
        ss_copy(a.at_hand.ss_copy), row((lane & 15) % B), first((lane & 15) / B), at_once(16 / B) {}
  __device__ __forceinline__ TileOut(const PersistArgs& a, h16_t* x_, int which, bool last)
      : h(rsrc_of(keep(a.h))), x(keep(x_)), ss(keep(a.ss_in[which])), ss_out(last ? a.ss[which] : nullptr),
        err_flag(keep(a.err_flag)), d(keep(a.d)), B(keep(a.B)), x_rows(0), copies(1), x_copy(0), ss_copy(0), row(0), first(0), at_once(1) {}
};
// Place of row m, column n of an operand whose pieces hold `rows` rows (16: the layout of act_off()).
__device__ __forceinline__ int packed_off(int m, int n, int rows) {
  return (n >> 5) * (rows * 32) + ((n & 31) >> 3) * (rows * 8) + m * 8 + (n & 7);
}
// Where a tile's operand and squares will go in a later block: nothing is written there yet.
__device__ __forceinline__ void not_there(const TileOut& to, int nt, int lane) {
  const int n = nt * 16 + (lane >> 4) * 4;
  const uint2 none = make_uint2(kNotThere, kNotThere);
  for (int c = 0; c < to.copies; c += to.at_once) {
    if (to.first >= min(to.at_once, to.copies - c)) continue;
    st8((char*)(to.x + packed_off(to.row, n, to.x_rows)) + (c + to.first) * to.x_copy, none);
    if (lane < 16) st4((float*)((char*)(to.ss + to.row * kPersistGrid + nt) + (c + to.first) * to.ss_copy), __uint_as_float(kNotThere));
  }
}
// h += sum; x' = fp16(h gain r); the squares' sum of the tile.  Lane: row m, columns n = 16 nt + 4 (lane / 16) ..
// PACKED: x in pieces of to.x_rows rows, and h stays with the caller (returned).
template <int BT, bool PACKED = false>
__device__ __forceinline__ v4f residual_tile(const TileOut& to, int nt, int mt, int lane, v4f sum, v4f h_old, v4f gain, float sc) {
  const int m = mt * 16 + (lane & 15), n = nt * 16 + (lane >> 4) * 4;
  const bool live = m < to.B;
  v4f hv = h_old + sum;
  if (!live) hv = v4f{0.f, 0.f, 0.f, 0.f};
  bool out_of_range = false;
  uint2 pk;
  pk.x = pack_h16x2_track(hv[0] * gain[0] * sc, hv[1] * gain[1] * sc, out_of_range);
  pk.y = pack_h16x2_track(hv[2] * gain[2] * sc, hv[3] * gain[3] * sc, out_of_range);
  if (live && !PACKED) st16(to.h, (m * to.d + n) * 4, 0, __builtin_bit_cast(v4u, hv));
  if constexpr (!PACKED) {
    if (live) st8(to.x + act_off(m, n, 16 * BT), pk);
  } else if (to.copies == 1) {
    if (live) st8(to.x + packed_off(m, n, to.x_rows), pk);
  } else {
    const int from = (lane & 48) + to.row;
    const uint2 mine = make_uint2(__shfl(pk.x, from, 64), __shfl(pk.y, from, 64));
    for (int c = 0; c < to.copies; c += to.at_once)
      if (to.first < min(to.at_once, to.copies - c))
        st8((char*)(to.x + packed_off(to.row, n, to.x_rows)) + (c + to.first) * to.x_copy, mine);
  }
  float ss = fmaf(hv[0], hv[0], hv[1] * hv[1]) + fmaf(hv[2], hv[2], hv[3] * hv[3]);  // rounded as in the separate launches
  ss += __shfl_xor(ss, 16, 64);
  ss += __shfl_xor(ss, 32, 64);
  const float s = __uint_as_float(written(__float_as_uint(ss)));
  if (PACKED && to.copies > 1) {
    const float mine = __shfl(s, to.row, 64);
    for (int c = 0; c < to.copies; c += to.at_once)
      if (lane < 16 && to.first < min(to.at_once, to.copies - c))
        st4((float*)((char*)(to.ss + to.row * kPersistGrid + nt) + (c + to.first) * to.ss_copy), mine);
  }
  if (lane < 16 && live) {
    if (!PACKED || to.copies == 1) st4(to.ss + m * kPersistGrid + nt, s);
    if (to.ss_out) st4(to.ss_out + nt * 16 * BT + m, ss);
  }
  if (live && out_of_range) atomicOr(to.err_flag, kErrFp16Range);
  return hv;
}

// The unit of a workgroup in the attention phase, the same in every block: (sequence, kv head, chunk) and its place in the cache.
// Places that are congruent modulo 8 (one die, one L2) take a run of units, the sequence counting fastest: those that sample
// from one prompt read its pages together.
struct AttnUnit {
  int b, g, chunk;
  AttnDecRange r;
  bool there;   // the workgroup has a unit
  bool active;  // ... and its chunk holds a part of the context
  __device__ __forceinline__ AttnUnit(const PersistArgs& a, int place) {
    const int die = place & 7, slot = place >> 3, run = a.attn_units / 8, more = a.attn_units % 8;
    there = slot < run + (die < more);
    const int u = there ? die * run + min(die, more) + slot : 0;
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

// ---- attention: one unit per workgroup, the same in every block
struct AttnLds {  // rotated queries, this position's key and value, the wavefronts' results
  __attribute__((aligned(16))) h16_t q[16][kHeadDim], k[kHeadDim], v[kHeadDim];
  float o[AW][AGMAX][kHeadDim + 1];
  float m[AW][16], l[AW][16];
};
// What a wavefront holds of its unit for the whole launch: its place, the ids of its first pair of pages, the rotation of the
// position.  table (LDS): the page ids of the chunk.
struct AttnHeld {
  int b, g, chunk, pos, lo, hi, id0, id1;
  bool there, active;
  float rope_c, rope_s;
  // Mpad: rows of the operand that the output goes to; 0: the caller clears the part of a unit that is not active
  __device__ __forceinline__ AttnHeld(const PersistArgs& a, int place, int wave, int lane, int* table, int Mpad) {
    const AttnUnit u(a, place);
    b = u.b; g = u.g; chunk = u.chunk; pos = u.r.pos; lo = u.r.lo; hi = u.r.hi;
    there = u.there;
    active = u.active;
    const int* pages = a.at.pool.page_table + (size_t)b * a.at.pool.max_pages;
    const int tid = wave * 64 + lane, last = a.at.pool.max_pages - 1;
    if (active)
      for (int i = tid; i < hi - lo; i += AW * 64) table[i] = pages[lo + i];
    id0 = __builtin_amdgcn_readfirstlane(pages[min(lo + 2 * wave, last)]);
    id1 = __builtin_amdgcn_readfirstlane(pages[min(lo + 2 * wave + 1, last)]);
    const size_t at = (size_t)max(pos, 0) * (kHeadDim / 2) + lane;
    rope_c = a.at.cos[at];
    rope_s = a.at.sin[at];
    if (there && !active && Mpad) {
      // a chunk beyond the context contributes nothing, which its consumer learns from a zero sum; its part of the operand
      // is cleared so that stale bits never meet a zero weight.  Once: nobody writes it in this launch.
      const int G = a.at.Hq / a.at.Hkv;
      if (tid < G * (kHeadDim / 8)) {
        const int h = tid / (kHeadDim / 8), d0 = (tid % (kHeadDim / 8)) * 8;
        h16_t* o = a.at.o + chunk * a.at.o_chunk_stride + act_off(b, (g * G + h) * kHeadDim + d0, Mpad);
        st8(o, make_uint2(0u, 0u));
        st8(o + 4, make_uint2(0u, 0u));
        if (d0 == 0) st8(a.at.ml + (((size_t)b * a.at.Hq + g * G + h) * a.at.n_chunks + chunk) * 2, make_uint2(0xff800000u, 0u));
      }
    }
  }
};
// How the rows of qkv come to a unit and where its output goes: enter() lets the wavefront into the phase, where the rows of qkv are there
// (false: the launch ends).
template <class Enter>
struct CountedUnit {
  int Mpad;
  Enter enter;
  __device__ __forceinline__ const float* qkv(const PersistArgs& a) const { return keep(a.at.qkv); }
  __device__ __forceinline__ h16_t* out(const PersistArgs& a, int chunk) const { return keep(a.at.o) + chunk * a.at.o_chunk_stride; }
  __device__ __forceinline__ float* ml(const PersistArgs& a) const { return keep(a.at.ml); }
  __device__ __forceinline__ size_t place(int m, int k) const { return act_off(m, k, Mpad); }
  __device__ __forceinline__ void before_stores() const {}
  // load() once the rows are there
  template <class Load>
  __device__ __forceinline__ bool operator()(const PersistArgs&, Load load) const {
    if (!enter()) return false;
    load();
    return true;
  }
};
template <class Enter>
__device__ __forceinline__ CountedUnit<Enter> counted_unit(int Mpad, Enter enter) { return {Mpad, enter}; }

// The active unit in block l, by wavefronts 0 .. AW - 1; two barriers of the workgroup.  The stores are left to be drained.
// TWO_SETS: two sets of registers for keys and values, the next pair of pages on its way while one is multiplied.
template <bool TWO_SETS, class Hand>
__device__ __forceinline__ bool attend(const AttnHeld& u, AttnLds& at, const int* table, int l, int wave, const Hand& hand) {
        const Ctx c = fresh(wave);
        const PersistArgs& a = c.a;
        const int w = c.wave, lane = c.lane, tid = w * 64 + lane, col = lane & 15, lg = lane >> 4;
        const int Hq = a.at.Hq, Hkv = a.at.Hkv, G = Hq / Hkv;
        const KvPool& pool = a.at.pool;
        const h16_t* kbase = dec_page<kHeadDim>(pool, l, 0, 0, u.g);
        const h16_t* vbase = dec_page<kHeadDim>(pool, l, 1, 0, u.g);
        const size_t pstride = (size_t)pool.n_kv_heads * (kPageTokens * kHeadDim);
        const int pg0 = u.lo + 2 * w;
        // the first pair of pages is of earlier steps, but for the current position, which is put in below
        KvFrags<kHeadDim> cur = load_kv<kHeadDim>(kbase + u.id0 * pstride, kbase + u.id1 * pstride, vbase + u.id0 * pstride,
                                                  vbase + u.id1 * pstride, lane);
        const int n_st = pg0 < u.hi ? (u.hi - pg0 + 2 * AW - 1) / (2 * AW) : 0;
        auto page_id = [&](int pg) { return (size_t)table[min(pg, u.hi - 1) - u.lo] * pstride; };
        auto load_stage = [&](int i) {
          const int pg = pg0 + 2 * AW * i;
          const size_t o0 = page_id(pg), o1 = page_id(pg + 1);
          return load_kv<kHeadDim>(kbase + o0, kbase + o1, vbase + o0, vbase + o1, lane);
        };
        KvFrags<kHeadDim> alt;
        if constexpr (TWO_SETS) {
          if (n_st > 1) alt = load_stage(1);
        }
        const float* row = hand.qkv(a) + (size_t)u.b * (Hq + 2 * Hkv) * kHeadDim;
        int* const err_flag = keep(a.err_flag);
        const int n_chunks = keep(a.at.n_chunks);
        h16_t* const out = hand.out(a, u.chunk);
        float* const ml = hand.ml(a);
        const int cur_page = u.pos / kPageTokens, slot = u.pos % kPageTokens;
        const bool owner = cur_page >= u.lo && cur_page < u.hi;
        const bool appends = owner && w == AW - 1;
        auto rot = [&](float x, float y, float s) { return fmaf(x, u.rope_c, y * s); };  // rounded as in k_attn_dec
        {
          const float* qp = row + (size_t)(u.g * G + min(w, G - 1)) * kHeadDim;
          const float* kp = row + (size_t)(Hq + u.g) * kHeadDim;
          const float* vp = kp + (size_t)Hkv * kHeadDim;
          float q0, q1, x0 = 0.f, x1 = 0.f, v0 = 0.f, v1 = 0.f;
          if (!hand(a, [&] {
                q0 = ld4(qp + lane); q1 = ld4(qp + lane + 64);
                if (appends) {
                  x0 = ld4(kp + lane); x1 = ld4(kp + lane + 64);
                  v0 = ld4(vp + lane); v1 = ld4(vp + lane + 64);
                }
                return max(largest(__builtin_bit_cast(v4u, v4f{q0, q1, x0, x1})), max(__float_as_uint(v0), __float_as_uint(v1)));
              }))
            return false;
          if (appends) {
            const h16_t k0 = f32_to_h16_flag(rot(x0, x1, -u.rope_s), err_flag), k1 = f32_to_h16_flag(rot(x1, x0, u.rope_s), err_flag);
            const h16_t y0 = f32_to_h16_flag(v0, err_flag), y1 = f32_to_h16_flag(v1, err_flag);
            at.k[lane] = k0; at.k[lane + 64] = k1;
            at.v[lane] = y0; at.v[lane + 64] = y1;
            const size_t page = (size_t)table[cur_page - u.lo] * pstride;
            h16_t* kd = const_cast<h16_t*>(kbase) + page;
            h16_t* vd = const_cast<h16_t*>(vbase) + page;
            kd[(lane >> 3) * 128 + slot * 8 + (lane & 7)] = k0;
            kd[((lane + 64) >> 3) * 128 + slot * 8 + (lane & 7)] = k1;
            vd[lane * kPageTokens + slot] = y0;
            vd[(lane + 64) * kPageTokens + slot] = y1;
          }
          if (w < G) {
            at.q[w][lane] = f32_to_h16_flag(rot(q0, q1, -u.rope_s), err_flag);
            at.q[w][lane + 64] = f32_to_h16_flag(rot(q1, q0, u.rope_s), err_flag);
          }
        }
        lds_barrier();
        v8h qf[kHeadDim / 32];
  #pragma unroll
        for (int kb = 0; kb < kHeadDim / 32; ++kb) {
          v4u raw = {0u, 0u, 0u, 0u};
          if (col < G) raw = *reinterpret_cast<const v4u*>(&at.q[col][kb * 32 + 8 * lg]);
          qf[kb] = __builtin_bit_cast(v8h, raw);
        }
        const int qpos = (col < G) ? u.pos : -1;
        AttnState<kHeadDim / 16> st;
        attn_init(st);
        const float scale2 = 0.08838834764831845f * 1.4426950408889634f;  // log2(e) / sqrt(head_dim)
        // a stage that another one follows lies wholly before the position
        int j = 0;
        if constexpr (TWO_SETS) {
          auto attend_full = [&](const KvFrags<kHeadDim>& f, int i) {
            attn_step1<kHeadDim, false>(f, (pg0 + 2 * AW * i) * kPageTokens, qf, qpos, scale2, st, lane);
          };
          for (; j + 2 < n_st; j += 2) {  // stages j and j + 1 are on their way
            attend_full(cur, j);
            cur = load_stage(j + 2);
            attend_full(alt, j + 1);
            alt = load_stage(min(j + 3, n_st - 1));
          }
          if (j + 1 < n_st) {
            attend_full(cur, j);
            cur = alt;
            ++j;
          }
        } else {
          // one register set, each half refilled as soon as it is used
          for (; j + 1 < n_st; ++j) {
            const int pg = pg0 + 2 * AW * (j + 1);
            const size_t o0 = page_id(pg), o1 = page_id(pg + 1);
            const v8h pf = attn_weights1<kHeadDim, false>(cur, (pg0 + 2 * AW * j) * kPageTokens, qf, qpos, scale2, st, lane);
            load_keys<kHeadDim>(cur, kbase + o0, kbase + o1, lane);
            attn_values1<kHeadDim>(cur, pf, st);
            load_values<kHeadDim>(cur, vbase + o0, vbase + o1, lane);
          }
        }
        if (j < n_st) {
          const int pg = pg0 + 2 * AW * j, p = cur_page - pg;
          if (owner && (p == 0 || p == 1)) {
            // the current position's key and value, whatever the load saw of the append
            if (col == slot) {
  #pragma unroll
              for (int kb = 0; kb < kHeadDim / 32; ++kb) {
                const v8h k = *reinterpret_cast<const v8h*>(&at.k[kb * 32 + 8 * lg]);
                if (p == 0) cur.k[0][kb] = k;
                else cur.k[1][kb] = k;
              }
            }
            if (lg == slot >> 2) {
              const uint32_t shift = (slot & 1) * 16, mask = 0xffffu << shift;
  #pragma unroll
              for (int cb = 0; cb < kHeadDim / 16; ++cb) {
                const uint32_t v = (uint32_t)at.v[cb * 16 + col] << shift;
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
            for (int r = 0; r < 4; ++r) at.o[w][col][cb * 16 + 4 * lg + r] = st.o[cb][r];
        }
        if (lg == 0) {
          at.m[w][col] = st.m;
          at.l[w][col] = sum_l;
        }
        lds_barrier();
        hand.before_stores();
        // merge the wavefronts: thread t < 16 G owns (head h, 8 consecutive dims)
        if (tid < G * (kHeadDim / 8)) {
          const int h = tid / (kHeadDim / 8), d0 = (tid % (kHeadDim / 8)) * 8;
          float mm = -INFINITY, ll = 0.f, acc[8] = {};
  #pragma unroll
          for (int v = 0; v < AW; ++v) mm = fmaxf(mm, at.m[v][h]);
  #pragma unroll
          for (int v = 0; v < AW; ++v) {
            const float f = __builtin_amdgcn_exp2f(at.m[v][h] - mm);
            ll += f * at.l[v][h];
  #pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += f * at.o[v][h][d0 + e];
          }
          const float inv = 1.0f / ll;  // every page of an active chunk holds at least one visible key
          uint32_t pk[4];
  #pragma unroll
          for (int e = 0; e < 4; ++e) pk[e] = pack_h16x2_flag(acc[2 * e] * inv, acc[2 * e + 1] * inv, err_flag);
          h16_t* o = out + hand.place(u.b, (u.g * G + h) * kHeadDim + d0);
          st8(o, make_uint2(pk[0], pk[1]));
          st8(o + 4, make_uint2(pk[2], pk[3]));
          if (n_chunks > 1 && d0 == 0)
            st8(ml + (((size_t)u.b * Hq + u.g * G + h) * n_chunks + u.chunk) * 2,
                make_uint2(__float_as_uint(mm * 0.6931471805599453f), __float_as_uint(ll)));  // the consumer works in natural units
        }
  return true;
}

// Buffers of block l (see Operand): what its QKV projection reads, and what it leaves for the next one.
__device__ __forceinline__ h16_t* x_of(const PersistArgs& a, int l) { return l == 0 ? a.x : a.xr + (size_t)(l - 1) * a.x_stride; }
__device__ __forceinline__ h16_t* x_behind(const PersistArgs& a, int l) { return l + 1 == a.n_layers ? a.x : a.xr + (size_t)l * a.x_stride; }

// decode_persistent_some.hip: the step by the workgroups that are there, after a launch that was given up
void launch_some(const PersistArgs& a, int bt, hipStream_t st);

// decode_persistent_rows.hip, bt tiles of 16 rows (2 to 4), where persist_rows_fit()
void launch_rows(const PersistArgs& a, int bt, int gu_tiles, hipStream_t st);

}  // namespace persist
}  // namespace bf16
}  // namespace mtmc
