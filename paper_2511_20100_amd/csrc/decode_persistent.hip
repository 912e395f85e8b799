// The residual blocks of a decode step as ONE launch (MTMC_OPT_PERSISTENT_DECODE): one tile of 16 rows here, two to four tiles
// in decode_persistent_rows.hip.
//
// What bounds a step of few rows as six launches per block is not its bytes: a dependent launch costs 4 to 5 us before its
// first weight arrives, and a block's 93 MB (1.5 B shape, 15 us at the rate of a plain read) took 48 us as six launches.  Here
// one workgroup per CU stays for the whole step, and the weights of the next phase are on their way while it waits for what the
// last one gives: they depend on nothing.  A phase gets its operand in one of two ways:
//
//   ASK false  the grid waits on counters in memory: stores drained (0.5 to 1 us), counted (1.5 us from the last arrival), and
//              then the operand is read (1 us), through the caches where many workgroups read the same.  But the rows of qkv and
//              the sums of the splits, which have few readers each, are asked for as below (two of six waits of a block; 23 steps
//              of the 1.5 B shape behind 200 tokens, 16 rows: 27.2 -> 25.6 ms, 8 rows 25.0 -> 22.6).
//   ASK true   (up to kPersistAskRows rows) readers ask for the operand until no word of it says "not written yet", past the
//              caches: 1.5 to 2 us from the store to the product.  Every round of asking moves the operand of all workgroups,
//              so this is for few rows, and what all of them ask for is there in eight copies (one: the asking alone took the
//              first 2 us of the gate / up projection).  23 steps of the 1.5 B shape behind 200 tokens, counters -> asking:
//              one row 21.4 -> 19.7 ms, 2 rows 21.4 -> 20.4, 4 rows 22.48 -> 22.56; 1.3 B blocks with a kv head per query head, 4
//              rows, 8.33 -> 8.57; of four 7 B blocks one row 14.62 -> 14.53: the line is at 2.
//
// With either, the gate / up weights of which registers hold four k tiles have the others in LDS, asked for ahead of the O
// projection: by the time its operand is there all of them are (same steps, all in registers -> this: one row 24.5 -> 23.8 ms,
// 16 rows 28.5 -> 27.1; 16 rows after 1500 tokens 44.2 -> 42.8).
//
// What is left of the 23 us of a block at one row: six phases of 1.5 to 2 us from store to operand, 0.5 to 1 for sums and epilogue,
// attention 3.5, the chunks in the O projection 2.3, and 3 us in which the down weights come, for which there is no room ahead.
//
//   wavefronts 0 .. 7    stream weights and multiply; their sums per range of K go to LDS.  They ask for the next weights only
//                        when the stores of the phase are on their way (ASK) or counted: ahead of them in the CU's queue to
//                        memory they held these up by 2 to 3 us.
//   wavefronts 8 .. 11   add up the ranges in order, run the epilogues, store, and without ASK drain their stores, count the
//                        workgroup in and (one of them) watch the counters.  They hold no weights in flight: loads return in
//                        order, and a look at a counter would come back behind them.
//
// What one workgroup writes and another reads goes past the caches that are not coherent between the dies: device-scope
// (sc1) stores and loads.  Everything else (weights, tables, pages of earlier steps) is read as usual.  Every sum has the ranges
// and the order of the launches of decode_bf16.hip, so the results are theirs bit for bit.
//
// All kPersistGrid workgroups have to be resident at once: one per CU, and no second persistent launch of the process under way
// (PersistentTurn).  What else holds a CU, and for how long, nobody here knows.  So the first wait of a launch is its roll call
// (roll_call.h): the phase before it changes nothing that a step starts from, and where not all workgroups come within the limit, the
// launch ends there and decode_persistent_some.hip does the step.
#include <type_traits>

#include "decode_persistent.h"
#include "kernels.h"

namespace mtmc {
namespace bf16 {
namespace persist {
namespace {

constexpr int kComputeWaves = AW, kControlWaves = 4, kThreads = (kComputeWaves + kControlWaves) * 64;
constexpr int kItems = 48;  // sums of 16 x 16 values that a phase hands over at once
constexpr int kTail = 12;   // weight tiles of the gate / up projection that a wavefront keeps in LDS: with the rest 155 of 160 KB

struct Shared {
  union {
    v4f red[kItems][64];  // sums per range of K, as the accumulators lie in the lanes
    AttnLds at;
    struct {
      v4f sums[16][64];                      // red of the O projection
      float ml[kComputeWaves][2][8][16];     // per wavefront, head in hand, chunk and row: the chunk's rescaled sum
      float share[kComputeWaves][2][8][16];  // ... and its share
    } o;
  };
  v4u tail[kComputeWaves][kTail][64];
  int table[ATAB];                       // page ids of the attention unit
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

// Where what block l hands on lies.  ASK: in the block's piece of memory (persist_hand(), which also says when its places are
// marked as not written); else in buffers of 16 rows, one per block for what is read through the caches.  What comes in and goes
// out has 16 rows.
template <bool ASK>
struct Place {
  const PersistArgs& a;
  int l, wg;
  using Asking = std::conditional_t<ASK, Asker, Known>;
  using Rows = Operand<1, ASK ? kDeviceScope : 0>;  // through the caches where the counters have been waited for
  __device__ __forceinline__ static Asking asker(const PersistArgs& a, int* stop) {
    if constexpr (ASK) return Asker{a, stop};
    else return Known{};
  }
  __device__ __forceinline__ char* hand(int block) const { return a.hand + (size_t)(block % kPersistPieces) * a.at_hand.bytes; }
  __device__ __forceinline__ int rows() const { return ASK ? a.B : 16; }
  // of the copies that are written, the one of this workgroup (0: where to write the first)
  __device__ __forceinline__ h16_t* x(int block, int mine) const {
    if constexpr (ASK) return block == 0 || block == a.n_layers ? a.x : (h16_t*)(hand(block) + a.at_hand.x + mine * a.at_hand.x_copy);
    else return block == 0 || block == a.n_layers ? a.x : a.xr + (size_t)(block - 1) * a.x_stride;
  }
  __device__ __forceinline__ h16_t* xo(int mine) const {
    if constexpr (ASK) return (h16_t*)(hand(l) + a.at_hand.xo + mine * a.at_hand.x_copy);
    else return a.xo + (size_t)l * a.x_stride;
  }
  // sums of squares: of what goes into a block, and behind the O projection
  __device__ __forceinline__ float* ss0(int block, int mine) const {
    if constexpr (ASK) {
      if (block != 0 && block != a.n_layers) return (float*)(hand(block) + a.at_hand.ss0 + mine * a.at_hand.ss_copy);
    }
    return a.ss_in[0];
  }
  __device__ __forceinline__ float* ss1(int block, int mine) const {
    if constexpr (ASK) return (float*)(hand(block) + a.at_hand.ss1 + mine * a.at_hand.ss_copy);
    else return a.ss_in[1];
  }
  __device__ __forceinline__ int mine() const { return ASK ? wg % kPersistCopies : 0; }
  __device__ __forceinline__ int x_rows(int block) const { return block == 0 || block == a.n_layers ? 16 : rows(); }
  __device__ __forceinline__ int copies(int block) const { return !ASK || block == a.n_layers ? 1 : kPersistCopies; }
  __device__ __forceinline__ h16_t* act() const {
    if constexpr (ASK) return (h16_t*)(hand(l) + a.at_hand.act);
    else return a.act + (size_t)l * a.act_stride;
  }
  __device__ __forceinline__ float* qkv() const {
    if constexpr (ASK) return (float*)(hand(l) + a.at_hand.qkv);
    else return (float*)(a.hand + (l & 1) * a.at_hand.qkv_copy);  // persist_hand_rows()
  }
  __device__ __forceinline__ float* part() const {
    if constexpr (ASK) return (float*)(hand(l) + a.at_hand.part);
    else return (float*)(a.hand + a.at_hand.part);
  }
  __device__ __forceinline__ int o_chunk() const { return ASK ? a.at_hand.o_chunk : (int)(a.at.o_chunk_stride * sizeof(h16_t)); }
  __device__ __forceinline__ h16_t* o(int chunk) const {
    char* first;
    if constexpr (ASK) first = hand(l) + a.at_hand.o;
    else first = (char*)a.at.o;
    return (h16_t*)(first + chunk * o_chunk());
  }
  __device__ __forceinline__ float* ml() const {
    if constexpr (ASK) return (float*)(hand(l) + a.at_hand.ml);
    else return a.at.ml;
  }
};

// The attention unit's side of it; enter() as in CountedUnit.
template <bool ASK, class Enter>
struct OneTileUnit {
  int l;
  int* stop;
  int rows;
  Enter enter;
  __device__ __forceinline__ const float* qkv(const PersistArgs& a) const { return keep(Place<ASK>{a, l, 0}.qkv()); }
  __device__ __forceinline__ h16_t* out(const PersistArgs& a, int chunk) const { return keep(Place<ASK>{a, l, 0}.o(chunk)); }
  __device__ __forceinline__ float* ml(const PersistArgs& a) const { return keep(Place<ASK>{a, l, 0}.ml()); }
  __device__ __forceinline__ size_t place(int m, int k) const { return packed_off(m, k, rows); }
  __device__ __forceinline__ void before_stores() const {
    if constexpr (ASK) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the marks of write()
  }
  // The part of the output that thread tid stores (if there is one), as `words`; the statistics with it as `stat`.
  __device__ __forceinline__ void write(const PersistArgs& a, const AttnHeld& u, int tid, uint2 words, uint2 stat) const {
    const int Hq = a.at.Hq, G = Hq / a.at.Hkv;
    if (tid >= G * (kHeadDim / 8)) return;
    const int h = u.g * G + tid / (kHeadDim / 8), d0 = (tid % (kHeadDim / 8)) * 8;
    h16_t* o = out(a, u.chunk) + place(u.b, h * kHeadDim + d0);
    st8(o, words);
    st8(o + 4, words);
    if (a.at.n_chunks > 1 && d0 == 0) st8(ml(a) + (((size_t)u.b * Hq + h) * a.at.n_chunks + u.chunk) * 2, stat);
  }
  template <class Load>
  __device__ __forceinline__ bool operator()(const PersistArgs& a, Load load) const {
    if (!enter()) return false;
    Asker{a, stop}(load);
    return true;
  }
};

// The row scales of a phase.  The sums of squares of a row's tiles lie side by side (kPersistGrid floats per row).  P partial sums
// of them (part p: tiles p, p + P, ...), then those in order: the order of a launch of 16 P threads.  The four control
// wavefronts take four rows each, 16 lanes to a row, all loads in one go; what they leave in sh.scale is read behind a barrier.
// The older sums are long there: what comes of them is out of the way when the new ones come.
template <int P, bool TWO, class Asking>
__device__ __forceinline__ void row_scales(Shared& sh, const Ctx& c, const Asking& asker, const float* cur, const float* old) {
  const PersistArgs& a = c.a;
  const int cw = c.wave - kComputeWaves, m = cw * 4 + (c.lane >> 4), q = c.lane & 15;
  if (cw * 4 >= a.B) return;
  // lane q: parts q, q + G, ... (PP of them), part p's tiles p + P k (K of them)
  constexpr int G = P == 20 ? 10 : 16, PP = P / G, K = P == 20 ? 5 : (kPersistGrid + P - 1) / P;
  const int row = min(m, a.B - 1) * kPersistGrid;
  auto load = [&](const float* ss, float (&v)[PP][K]) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < PP; ++i) v[i][k] = ld4(ss + row + min(q + G * i + P * k, a.nt_d - 1));
    uint32_t top = 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < PP; ++i) top = max(top, __float_as_uint(v[i][k]));
    return top;
  };
  auto add = [&](const float (&v)[PP][K], float (&part)[16][68]) {
    if (P != 20 || q < G) {
#pragma unroll
      for (int i = 0; i < PP; ++i) {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) sum += q + G * i + P * k < a.nt_d ? v[i][k] : 0.f;
        part[m][q + G * i] = sum;
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the rows are the wavefront's own
    float total = 0.f;
    if (q == 0) {
      v4f p4[P / 4];
#pragma unroll
      for (int p = 0; p < P / 4; ++p) p4[p] = *reinterpret_cast<const v4f*>(&part[m][4 * p]);
#pragma unroll
      for (int p = 0; p < P; ++p) total += p4[p / 4][p % 4];
    }
    return total;
  };
  float before = 1.f, va[PP][K];
  if constexpr (TWO) {
    float vb[PP][K];
    if constexpr (std::is_same_v<Asking, Known>) load(cur, va);
    asker([&] { return load(old, vb); });
    before = sqrtf(add(vb, sh.part[1]) * a.inv_d + a.eps);
  }
  if constexpr (!TWO || !std::is_same_v<Asking, Known>) asker([&] { return load(cur, va); });
  const float now = add(va, sh.part[0]);
  if (q == 0) sh.scale[m] = 1.0f / sqrtf(now * a.inv_d + a.eps) * before;  // scale_of()
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

// Behind the second barrier of a phase the control wavefronts have its stores on their way (ASK) or counted (else): only then the
// compute wavefronts ask for the next weights, which would be ahead of those stores in the CU's queue to memory, and write over
// what the phase had in LDS.  A launch that ends early does so behind a barrier; wavefronts that have left are not waited for.
template <int GU_TILES, int DN_RANGES, bool ASK>
__device__ __forceinline__ void control(Shared& sh, int wave) {
  const int cw = wave - kComputeWaves;
  const bool lead = cw == 0;
  constexpr int kGuRanges = GU_TILES == 6 ? 8 : 4;
  uint32_t phase = 0;
  auto running = [&] {
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(sh.stop) == 0;
  };
  // lets the compute wavefronts into the phase; false: the launch ends here
  auto enter = [&](const Ctx& c) {
    if constexpr (ASK) return true;
    if (lead && phase > 0 && !wait_grid(c, phase)) sh.stop = 1;
    return running();
  };
  auto done = [&](const Ctx& c) {  // stores of all control wavefronts
    if constexpr (ASK) return running();
    arrive(c, &sh.arrived, phase++);
    lds_barrier();
    return true;
  };
  auto done_lead = [&](const Ctx& c) {  // stores of the lead's own, or drained before a barrier
    if constexpr (ASK) return running();
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (lead && c.lane == 0) count_in(c, phase);
    ++phase;
    lds_barrier();
    return true;
  };
  // behind the barrier: what was loaded before is there, so that no store has to be waited for on its behalf; and (ASK) the marks
  // of the block behind this one (persist_hand())
  auto loads_done = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  auto marked = [] {
    if constexpr (ASK) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  const v4u none = v4u{kNotThere, kNotThere, kNotThere, kNotThere};
  const int n_layers = fresh(wave).a.n_layers;
  bool attends, attn_active;
  v4f h = v4f{0.f, 0.f, 0.f, 0.f};  // the lead's tile of the residual
  {
    const Ctx c = fresh(wave);
    const AttnUnit u(c.a, attn_place(c.a, c.wg));
    attends = u.there;
    attn_active = u.active;
    const int m = c.lane & 15, rq = (c.lane >> 4) * 4;
    if (lead && c.wg < c.a.nt_d) h = ld16f(rsrc_of(c.a.h), (min(m, c.a.B - 1) * c.a.d + c.wg * 16 + rq) * 4, 0);
  }
  float down_scale = 0.f;
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const int place = qkv_place(wg);
      const Rsrc out = rsrc_of(keep(at.qkv()));
      const int nt_qkv = keep(a.nt_qkv), B = keep(a.B);
      if (!enter(c)) return;
      auto each_tile = [&](auto f) {  // f(u, offset of this lane) for the wavefront's tiles
        for (int u = cw; place + u * kPersistGrid < nt_qkv; u += kControlWaves) f(u, ((m * nt_qkv + place + u * kPersistGrid) * 16 + rq) * 4);
      };
      if (ASK && l + 1 < n_layers && m < B) {
        const Rsrc behind = rsrc_of(Place<ASK>{a, l + 1, wg}.qkv());
        each_tile([&](int, int off) { st16(behind, off, 0, none); });
      }
      if (l == 0) {
        if (lane < 4) sh.scale[cw * 4 + lane] = 1.f;
      } else if (place < nt_qkv) {
        row_scales<64, true>(sh, c, at.asker(a, &sh.stop), at.ss0(l, at.mine()), at.ss1(l - 1, at.mine()));
      }
      for (int u = 0; place + u * kPersistGrid < nt_qkv; ++u) {
        lds_barrier();
        if ((u & 3) == cw) {
          const int nt = place + u * kPersistGrid;
          marked();
          const v4f sum = sum_ranges<16>(sh, (u & 1) * 16, lane);
          const int off = ((m * nt_qkv + nt) * 16 + rq) * 4;
          if (m < B) st16(out, off, 0, written(sum * sh.scale[m]));
          if (!ASK && m < B) st16(rsrc_of(Place<ASK>{a, l + 1, wg}.qkv()), off, 0, none);  // the units of the block before have read it
        }
      }
      if (!(l == 0 ? done(c) : running())) return;
    }
    // ---- attention
    {
      const Ctx c = fresh(wave);
      if (lead && l == 0) {
        if (ASK && c.lane == 0) count_in(c, 0);
        if (!answer_roll(c)) sh.stop = 1;
      }
      if (l == 0 && !running()) return;
      if (attends) {
        if (attn_active) {
          lds_barrier();
          lds_barrier();
        }
        if (!ASK) lds_barrier();
      }
      if (!done_lead(c)) return;
    }
    // ---- O projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const bool has_tile = wg < a.nt_d;
      const TileOut to(a, at.xo(0), at.ss1(l, 0), 1, at.rows(), ASK ? kPersistCopies : 1, l + 1 == n_layers, lane);
      const int ranges = keep(a.o_ranges);
      v4f gain = v4f{0.f, 0.f, 0.f, 0.f};
      if (lead && has_tile)
        gain = *reinterpret_cast<const v4f*>((const float*)((const char*)a.ffn_norm + l * a.layer_stride) + wg * 16 + rq);
      if (!enter(c)) return;
      if (has_tile) {
        if (ASK && lead && l + 1 < n_layers) {
          const Place<ASK> behind{a, l + 1, wg};
          not_there(TileOut(a, behind.xo(0), behind.ss1(l + 1, 0), 1, behind.rows(), kPersistCopies, false, lane), wg, lane);
        }
        const auto asker = at.asker(a, &sh.stop);
        const float* const ss = at.ss0(l, at.mine());
        if (ranges == 16) row_scales<64, false>(sh, c, asker, ss, ss);
        else if (ranges == 12) row_scales<48, false>(sh, c, asker, ss, ss);
        else row_scales<32, false>(sh, c, asker, ss, ss);
        lds_barrier();
        if (lead) {
          loads_done();
          const v4f sum = ranges == 16 ? sum_ranges<16>(sh, 0, lane) : ranges == 12 ? sum_ranges<12>(sh, 0, lane) : sum_ranges<8>(sh, 0, lane);
          h = residual_tile<1, true>(to, wg, 0, lane, sum, h, gain, sh.scale[m]);
        }
      }
      if (!done_lead(c)) return;
    }
    // ---- gate / up projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      h16_t* const act = keep(at.act());
      const int nt_gu = keep(a.nt_gu), B = keep(a.B);
      int* const err_flag = keep(a.err_flag);
      if (!enter(c)) return;
      const GuShare<GU_TILES> share(a, wg);
      if (share.first < nt_gu) {
        if (ASK && l + 1 < n_layers && m < B) {
          h16_t* const behind = Place<ASK>{a, l + 1, wg}.act();
          for (int p = cw; p < share.tiles / 2 && share.first + 2 * p < nt_gu; p += kControlWaves)
            st8(behind + packed_off(m, ((share.first >> 1) + p) * 16 + rq, B), make_uint2(kNotThere, kNotThere));
        }
        row_scales<4 * kGuRanges, true>(sh, c, at.asker(a, &sh.stop), at.ss1(l, at.mine()), at.ss0(l, at.mine()));
        lds_barrier();
        marked();
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
            st8(act + packed_off(m, (j >> 1) * 16 + rq, at.rows()), pk);
            out_of_range |= far;
          }
        }
        if (out_of_range) atomicOr(err_flag, kErrFp16Range);
      }
      if (!done(c)) return;
    }
    // ---- down projection: sums per split of K
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const Rsrc out = rsrc_of(keep(at.part()));
      const int d = keep(a.d), nt_d = keep(a.nt_d), B = keep(a.B), ks = keep(a.ks_down);
      if (!enter(c)) return;
      constexpr int kTiles = DN_RANGES == 5 ? 3 : DN_RANGES == 8 ? 2 : 4;
      const int split = DN_RANGES == 5 ? wg & 7 : wg % ks;
      const int tile = DN_RANGES == 5 ? (wg >> 3) + kPersistGrid / 8 * cw : wg / ks * kTiles + cw;
      const bool has = cw < kTiles && tile < nt_d;
      const int off = ((split * at.rows() + m) * d + tile * 16 + rq) * 4;
      if (ASK && has && l + 1 < n_layers && m < B) st16(rsrc_of(Place<ASK>{a, l + 1, wg}.part()), off, 0, none);
      const float* const ss = at.ss1(l, at.mine());
      if (wg < nt_d) row_scales<4 * DN_RANGES, false>(sh, c, at.asker(a, &sh.stop), ss, ss);
      lds_barrier();
      down_scale = sh.scale[m];
      if (has) {
        marked();
        const v4f sum = sum_ranges<DN_RANGES>(sh, cw * DN_RANGES, lane);
        if (m < B) st16(out, off, 0, written(sum));
      }
      if (!running()) return;
    }
    // ---- sum of the splits, residual, operand of the next block: the lead alone
    if (lead) {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int wg = c.wg, lane = c.lane, m = lane & 15, rq = (lane >> 4) * 4;
      const bool last = l + 1 == n_layers, has_tile = wg < a.nt_d;
      const TileOut to(a, at.x(l + 1, 0), at.ss0(l + 1, 0), 0, at.x_rows(l + 1), at.copies(l + 1), last, lane);
      const Rsrc part = rsrc_of(keep(at.part()));
      const int ks = keep(a.ks_down), from = (min(m, to.B - 1) * to.d + wg * 16 + rq) * 4, step = at.rows() * to.d * 4;
      const float* gp = last ? a.final_norm : (const float*)((const char*)a.attn_norm + (l + 1) * a.layer_stride);
      v4f gain = v4f{0.f, 0.f, 0.f, 0.f};
      if (has_tile) gain = *reinterpret_cast<const v4f*>(gp + wg * 16 + rq);
      if (ASK && has_tile && l + 2 < n_layers) {
        const Place<ASK> behind{a, l + 1, wg};
        not_there(TileOut(a, behind.x(l + 2, 0), behind.ss0(l + 2, 0), 0, a.B, kPersistCopies, false, lane), wg, lane);
      }
      if (has_tile) {
        const Asker asker{a, &sh.stop};
        v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < ks; s0 += 8) {
          v4f v[8];
          asker([&] {
            uint32_t top = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = ld16f(part, from, min(s0 + u, ks - 1) * step);
#pragma unroll
            for (int u = 0; u < 8; ++u) top = max(top, largest(__builtin_bit_cast(v4u, v[u])));
            return top;
          });
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (s0 + u < ks) sum = sum + v[u];
        }
        loads_done();
        h = residual_tile<1, true>(to, wg, 0, lane, sum, h, gain, down_scale);
      }
      if (!ASK) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        if (c.lane == 0) count_in(c, phase);
        if (has_tile && m < to.B)  // read
          for (int s = 0; s < ks; ++s) st16(part, from, s * step, none);
      }
    }
    ++phase;
  }
}

// ======================================================================================
// compute wavefronts
// ======================================================================================
// The gate / up stream of one wavefront, n k tiles from k0 on.  The weights of the first T wait in LDS, where ahead() has them
// brought; those of the next PF are ahead in registers (start()).
template <int NB, int PF>
struct GateUp {
  static constexpr int T = kTail / NB;
  Stream<NB, 1, PF, PF> st;
  int k0, n, last;
  v4u (*tail)[64];
  __device__ __forceinline__ GateUp(int k0_, int n_, int last_, v4u (*tail_)[64]) : k0(k0_), n(n_), last(last_), tail(tail_) {}
  __device__ __forceinline__ void ahead(Rsrc w, const int (&rows)[NB], int lane) const {
    constexpr int kNonTemporal = 2;  // as load_weight() has it
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w, (__attribute__((address_space(3))) void*)tail[t * NB + nb], 16,
                                                 t < n ? lane * 16 : kReach, rows[nb] + min(k0 + t, last) * 1024, 0, kNonTemporal);
  }
  __device__ __forceinline__ void start(Rsrc w, const int (&rows)[NB], int lane) {
    st.start(w, rows, k0 + T, n - T, 0, 0, last, lane);
  }
  template <class Rows, class Asking>
  __device__ __forceinline__ void run(const Rows& x, const Asking& asker, v4f (&acc)[NB][1]) {
    v8h xt[T];
    asker([&] {
      uint32_t top = 0;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        Rows y = x;
        y.off[0] = t < n ? x.off[0] : kReach;
        xt[t] = y.tile(0, min(k0 + t, last));
      }
      st.operands(x);
#pragma unroll
      for (int t = 0; t < T; ++t) top = max(top, largest(__builtin_bit_cast(v4u, xt[t])));
      return max(top, st.largest_ahead());
    });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the tiles in LDS are there: they were asked for before the operand
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (t < n) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[nb][0] = mfma16(__builtin_bit_cast(v8h, tail[t * NB + nb][st.lane]), xt[t], acc[nb][0]);
      }
    }
    st.run_asking(x, asker, acc, PF);
  }
};
// two streams side by side
template <class S, class Rows, class Asking>
__device__ __forceinline__ void run_both(S& s0, S& s1, const Rows& x, const Asking& asker, v4f (&a0)[1][1], v4f (&a1)[1][1]) {
  asker([&] {
    s0.operands(x);
    s1.operands(x);
    return max(s0.largest_ahead(), s1.largest_ahead());
  });
  s0.run_asking(x, asker, a0, S::kOperandsAhead);
  s1.run_asking(x, asker, a1, S::kOperandsAhead);
}

template <int GU_TILES, int DN_RANGES, bool ASK>
__device__ __forceinline__ void compute(Shared& sh, int wave) {
  auto running = [&] {
    lds_barrier();
    return __builtin_amdgcn_readfirstlane(sh.stop) == 0;
  };
  auto enter = [&] {
    if constexpr (ASK) return true;
    return running();
  };
  auto done = [&] {
    if constexpr (ASK) return running();
    lds_barrier();
    return true;
  };
  const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
  const int n_layers = fresh(wave).a.n_layers;
  const Ctx first = fresh(wave);
  const AttnHeld unit(first.a, attn_place(first.a, first.wg), wave, first.lane, sh.table, ASK ? 0 : 16);
  // f(gate / up stream, weights, row tiles) of this wavefront in block l: 8 ranges of K over all the tiles, or 4 over half of them
  auto gate_up = [&](const Ctx& c, int l, auto f) {
    const PersistArgs& a = c.a;
    constexpr int kRanges = GU_TILES == 6 ? 8 : 4;
    const GuShare<GU_TILES> share(a, c.wg);
    const int w = c.wave, kt_d = keep(a.kt_d), nt_gu = keep(a.nt_gu), first_tile = keep(share.first);
    const int per = (kt_d + kRanges - 1) / kRanges, s = w % kRanges;
    const Rsrc W = rsrc_of(a.wgu + (size_t)l * a.layer_stride / sizeof(h16_t));
    auto with = [&](auto tiles_per_wave, auto depth) {
      constexpr int kTiles = decltype(tiles_per_wave)::value, PF = decltype(depth)::value;
      const int j0 = (w / kRanges) * kTiles;
      int rows[kTiles];
#pragma unroll
      for (int i = 0; i < kTiles; ++i) rows[i] = min(first_tile + j0 + i, nt_gu - 1) * kt_d * 1024;
      GateUp<kTiles, PF> g(s * per, min(per, kt_d - s * per), kt_d - 1, sh.tail[w]);
      f(g, W, rows, j0 * kRanges + s, std::integral_constant<int, kRanges>{});
    };
    constexpr int kFull = GU_TILES * kRanges / 8, kPair = 2 * kRanges / 8;
    if (first_tile >= nt_gu) return;
    if (share.tiles == GU_TILES) with(std::integral_constant<int, kFull>{}, std::integral_constant<int, kFull >= 5 ? 4 : 6>{});
    else with(std::integral_constant<int, kPair>{}, std::integral_constant<int, 6>{});
  };
  for (int l = 0; l < n_layers; ++l) {
    // ---- QKV projection: one row tile at a time, 16 ranges of K, two per wavefront
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int w = c.wave, wg = c.wg, lane = c.lane;
      const h16_t* const W = a.wqkv + (size_t)l * a.layer_stride / sizeof(h16_t);
      const h16_t* const x = keep(at.x(l, at.mine()));
      const int kt_d = keep(a.kt_d), nt_qkv = keep(a.nt_qkv), B = keep(a.B), per = (kt_d + 15) / 16;
      const auto xr = Place<ASK>::Rows::packed(x, at.x_rows(l), lane, B);
      const auto asker = at.asker(a, &sh.stop);
      Stream<1, 1, 4, 4> s0, s1;
      auto start = [&](int nt) {
        int rows[1] = {nt * kt_d * 1024};
        s0.start(rsrc_of(W), rows, w * per, min(per, kt_d - w * per), 0, 0, kt_d - 1, lane);
        s1.start(rsrc_of(W), rows, (w + 8) * per, min(per, kt_d - (w + 8) * per), 0, 0, kt_d - 1, lane);
      };
      int nt = qkv_place(wg);
      if (nt < nt_qkv) {
        start(nt);
        if (!enter()) return;
        for (int u = 0;; ++u) {
          v4f a0[1][1] = {{zero}}, a1[1][1] = {{zero}};
          run_both(s0, s1, xr, asker, a0, a1);
          sh.red[(u & 1) * 16 + w][lane] = a0[0][0];
          sh.red[(u & 1) * 16 + w + 8][lane] = a1[0][0];
          lds_barrier();
          nt += kPersistGrid;
          if (nt >= nt_qkv) break;
          start(nt);
        }
      } else if (!enter()) {
        return;
      }
    }
    if (!done()) return;
    // ---- attention
    {
      const Ctx c = fresh(wave);
      auto enter_attention = [&] { return l == 0 ? running() : true; };  // the first time the roll call
      const auto hand = OneTileUnit<ASK, decltype(enter_attention)>{l, &sh.stop, Place<ASK>{c.a, l, c.wg}.rows(), enter_attention};
      const int tid = c.wave * 64 + c.lane;
      if (ASK && unit.there && l + 1 < n_layers) {
        const uint2 none = make_uint2(kNotThere, kNotThere);
        OneTileUnit<ASK, decltype(enter_attention)>{l + 1, &sh.stop, hand.rows, enter_attention}.write(c.a, unit, tid, none, none);
      }
      if (unit.active) {
        if (!attend<false>(unit, sh.at, sh.table, l, wave, hand)) return;
      } else {
        if (!enter_attention()) return;
        const int G = c.a.at.Hq / c.a.at.Hkv;
        if (ASK && unit.there && persist_empty_unit_asks(c.wave, G)) {
          // a chunk beyond the context contributes nothing, which its consumer learns from a zero sum; who stores that waits for the rows
          // of qkv as the others do, or a workgroup with nothing else to do would be blocks ahead (persist_hand())
          const float* const row = hand.qkv(c.a) + (size_t)unit.b * c.a.nt_qkv * 16 + unit.g * G * kHeadDim;
          Asker{c.a, &sh.stop}([&] { return __float_as_uint(ld4(row + c.lane)); });
          hand.before_stores();
          hand.write(c.a, unit, tid, make_uint2(0u, 0u), make_uint2(0xff800000u, 0u));
        }
      }
      if (!ASK && unit.there) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
      }
    }
    if (!done()) return;
    // ---- O projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int w = c.wave, wg = c.wg, lane = c.lane, kt_nq = keep(a.kt_nq), B = keep(a.B);
      const h16_t* const W = a.wo + (size_t)l * a.layer_stride / sizeof(h16_t) + (size_t)wg * kt_nq * 512;
      const int R = keep(a.o_ranges), NC = keep(a.at.n_chunks);
      const auto asker = at.asker(a, &sh.stop);
      const auto xr = Operand<1, kDeviceScope>::packed(keep(at.o(0)), at.rows(), lane, B);
      auto gate_up_ahead = [&] {
        gate_up(c, l, [&](auto& g, Rsrc w_gu, const auto& rows, int, auto) { g.ahead(w_gu, rows, lane); });
      };
      if (wg >= a.nt_d) {
        gate_up_ahead();
        if (!enter()) return;
      } else if (NC == 1) {
        const int per = (kt_nq + R - 1) / R;
        int rows[1] = {0};
        Stream<1, 1, 4, 4> s0, s1;
        s0.start(rsrc_of(W), rows, w * per, min(per, kt_nq - w * per), 0, 0, kt_nq - 1, lane);
        s1.start(rsrc_of(W), rows, (w + 8) * per, min(per, kt_nq - (w + 8) * per), 0, 0, kt_nq - 1, lane);  // empty with 8 ranges
        gate_up_ahead();
        if (!enter()) return;
        v4f a0[1][1] = {{zero}}, a1[1][1] = {{zero}};
        run_both(s0, s1, xr, asker, a0, a1);
        sh.red[w][lane] = a0[0][0];
        sh.red[w + 8][lane] = a1[0][0];
        lds_barrier();
      } else {
        // The chunks of the context are combined here, head by head: out += sum_chunk share * (W_head . o_chunk), share =
        // l exp(m - max m) / sum l exp(m - max m).  Range v takes heads v, v + R, ...; this wavefront ranges w and (12
        // ranges) w + 8: its list of heads, two in hand at a time, up to six (head, chunk) operands on their way at once.
        constexpr int kItemsAhead = 5;
        const int n_heads = keep(a.at.Hq), col = lane & 15, lg = lane >> 4;
        const float* const ml = keep(at.ml());
        const int chunk_bytes = at.o_chunk();
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
        gate_up_ahead();
        if (!enter()) return;
        v4f acc = zero;
        for (int e0 = 0; e0 < n_e; e0 += 2) {
          if (e0) load_heads(e0);
          // chunk statistics of the two heads: lane (row, lg) has chunks lg and lg + 4
          uint2 st[2][2];
          const int n_items = min(2, n_e - e0) * NC;
          v8h xf[kItemsAhead][4];
          auto load_items = [&](int i0) {
#pragma unroll
            for (int q = 0; q < kItemsAhead; ++q) {
              const int i = min(i0 + q, n_items - 1), h = i >= NC ? 1 : 0;
              const int off = (i - h * NC) * chunk_bytes + head_of(e0 + h) * 4 * xr.step;
#pragma unroll
              for (int t = 0; t < 4; ++t) xf[q][t] = xr.load(0, off + t * xr.step);
            }
          };
          auto largest_item = [&] {
            uint32_t top = 0;
#pragma unroll
            for (int q = 0; q < kItemsAhead; ++q)
#pragma unroll
              for (int t = 0; t < 4; ++t) top = max(top, largest(__builtin_bit_cast(v4u, xf[q][t])));
            return top;
          };
          asker([&] {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int k = 0; k < 2; ++k)
                st[i][k] = ld8(ml + (((size_t)min(col, B - 1) * n_heads + head_of(e0 + i)) * NC + min(lg + 4 * k, NC - 1)) * 2);
            load_items(0);
            uint32_t top = ASK ? largest_item() : 0u;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int k = 0; k < 2; ++k) top = max(top, max(st[i][k].x, st[i][k].y));
            return top;
          });
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
            sh.o.ml[w][i][lg][col] = cl[i][0];
            sh.o.ml[w][i][lg + 4][col] = cl[i][1];
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            float den = 0.f;  // in chunk order
#pragma unroll
            for (int k = 0; k < 8; ++k) den += sh.o.ml[w][i][k][col];
            sh.o.share[w][i][lg][col] = den > 0.f ? cl[i][0] / den : 0.f;
            sh.o.share[w][i][lg + 4][col] = den > 0.f ? cl[i][1] / den : 0.f;
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          for (int i0 = 0; i0 < n_items; i0 += kItemsAhead) {
            if (i0) asker([&] {
              load_items(i0);
              return ASK ? largest_item() : 0u;
            });
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
                acc = acc + part * sh.o.share[w][h][k][col];
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
    if (!done()) return;
    // ---- gate / up projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int lane = c.lane;
      const auto xr = Place<ASK>::Rows::packed(keep(at.xo(at.mine())), at.rows(), lane, keep(a.B));
      const auto asker = at.asker(a, &sh.stop);
      bool has = false, on = true;
      gate_up(c, l, [&](auto& g, Rsrc w_gu, const auto& rows, int red0, auto ranges) {
        constexpr int kTiles = std::extent_v<std::remove_reference_t<decltype(rows)>>, kRanges = decltype(ranges)::value;
        g.start(w_gu, rows, lane);
        has = true;
        if (!(on = enter())) return;
        v4f acc[kTiles][1];
        clear(acc);
        g.run(xr, asker, acc);
#pragma unroll
        for (int i = 0; i < kTiles; ++i) sh.red[red0 + i * kRanges][lane] = acc[i][0];
        lds_barrier();
      });
      if (!has) on = enter();
      if (!on) return;
    }
    if (!done()) return;
    // ---- down projection
    {
      const Ctx c = fresh(wave);
      const PersistArgs& a = c.a;
      const Place<ASK> at{a, l, c.wg};
      const int w = c.wave, wg = c.wg, lane = c.lane;
      const h16_t* const W = a.wdown + (size_t)l * a.layer_stride / sizeof(h16_t);
      const h16_t* const x = keep(at.act());
      const int kt_F = keep(a.kt_F), nt_d = keep(a.nt_d), ks = keep(a.ks_down), B = keep(a.B);
      const int per_split = (kt_F + ks - 1) / ks, split = DN_RANGES == 5 ? wg & 7 : wg % ks;
      const int kbeg = split * per_split, kend = min(kt_F, kbeg + per_split);
      const int per = (max(kend - kbeg, 0) + DN_RANGES - 1) / DN_RANGES;
      const auto xr = Place<ASK>::Rows::packed(x, at.rows(), lane, B);
      const auto asker = at.asker(a, &sh.stop);
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
        if (!enter()) return;
        v4f a0[1][1] = {{zero}}, a1[1][1] = {{zero}};
        run_both(s0, s1, xr, asker, a0, a1);
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
        if (!enter()) return;
        v4f acc[2][1];
        clear(acc);
        st.ask(xr, asker);
        st.run_asking(xr, asker, acc, PF);
#pragma unroll
        for (int i = 0; i < 2; ++i) sh.red[(j0 + i) * DN_RANGES + s][lane] = acc[i][0];
        lds_barrier();
      }
    }
    if (!done()) return;
  }
}

template <int GU_TILES, int DN_RANGES, bool ASK>
__global__ __launch_bounds__(kThreads, 3) void k_decode_layers(PersistArgs) {  // read through the kernel argument segment: fresh()
  __shared__ Shared sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) {
    sh.arrived = 0;
    sh.stop = 0;
  }
  __syncthreads();
  if (wave < kComputeWaves) compute<GU_TILES, DN_RANGES, ASK>(sh, wave);
  else control<GU_TILES, DN_RANGES, ASK>(sh, wave);
}

template <int GU_TILES, bool ASK>
void launch_gu(const PersistArgs& a, int dn, hipStream_t st) {
  switch (dn) {
    case 5: k_decode_layers<GU_TILES, 5, ASK><<<kPersistGrid, kThreads, 0, st>>>(a); break;
    case 8: k_decode_layers<GU_TILES, 8, ASK><<<kPersistGrid, kThreads, 0, st>>>(a); break;
    default: k_decode_layers<GU_TILES, 4, ASK><<<kPersistGrid, kThreads, 0, st>>>(a); break;
  }
}
template <bool ASK>
void launch_ask(const PersistArgs& a, int gu_tiles, int dn, hipStream_t st) {
  if (gu_tiles == 4) launch_gu<4, ASK>(a, dn, st);
  else if (gu_tiles == 6) launch_gu<6, ASK>(a, dn, st);
  else launch_gu<10, ASK>(a, dn, st);
}

}  // namespace

void launch_one_tile(const PersistArgs& a, int gu_tiles, int dn_ranges, hipStream_t st) {
  if (a.B > kPersistAskRows) {
    launch_fill_u32(reinterpret_cast<uint32_t*>(a.hand), kNotThere, (size_t)a.at_hand.bytes / 4, st);
    return launch_ask<false>(a, gu_tiles, dn_ranges, st);
  }
  launch_fill_u32(reinterpret_cast<uint32_t*>(a.hand), kNotThere, (size_t)a.at_hand.bytes / 2, st);  // two pieces
  launch_ask<true>(a, gu_tiles, dn_ranges, st);
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
