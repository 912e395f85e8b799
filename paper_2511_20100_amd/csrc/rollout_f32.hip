// The decode steps of a generation of the fp32 path as ONE launch.
//
// What bounds such a step is no work: eight rows of a two-block model (d 256, vocabulary 4096) are twelve dependent products of
// a few KB, and as launches of their own each takes 4 to 9 us, most of it start, cold loads and end (68 us a step; 59 with the
// folds and the attention of f32_device.h; 42 here, where 1.2 to 1.9 us lie between two phases, 1.4 are a product's sums, 3.2 the
// attention and 6 the sampler).
// Here every workgroup stays for all steps and knows its tiles of every product.  It asks for their weights, waits for the
// operand, adds up and stores; nobody counts or watches anybody else.  That is done by the data themselves: a buffer
// holds kAbsent (a NaN that no result has) until its value is there, and a reader asks again until it sees no such word.  One trip
// of a store and one of a load from product to product, where counters take stores drained, an arrival, and a look at it besides.
//
// A step's values lie in one of three sets, in turn.  The set of the step before is filled with kAbsent again by the workgroups
// of the LM head, before they store a logit.  Whoever read from it has led to the residual that the LM head has seen; and
// whoever comes to it again, two steps on, has waited for the step between, which began with the tokens of this one and so
// with every one of its logits.  (With two sets a workgroup that has no tile of the LM head could come back before it is
// cleared.)  All of that holds for each block of eight rows by itself: blocks never wait for each other.
//
// The workgroups that find a place on the device in time share out the tiles, 256 as a rule, however few there are (roll_call.h);
// they all stay, so that every wait ends.
#include <algorithm>

#include "device_scope.h"
#include "f32_device.h"
#include "frag.h"
#include "kernels.h"
#include "roll_call.h"

namespace mtmc {
namespace f32 {
namespace {

using namespace device_scope;

constexpr int kThreads = 256, kRows = 8, kSets = kRolloutSets;
constexpr uint32_t kAbsent = 0xffffffffu;
constexpr int kMaxK = 2040;  // eight rows of the operand in LDS
constexpr long long kWaitTicks = 60 * 100000000ll;  // what is waited for always comes

__device__ __forceinline__ bool absent(float x) { return __float_as_uint(x) == kAbsent; }
__device__ __forceinline__ bool absent(v4f x) { return absent(x[0]) || absent(x[1]) || absent(x[2]) || absent(x[3]); }
__device__ __forceinline__ float present(float x) { return absent(x) ? __uint_as_float(0x7fc00000u) : x; }

template <int HD>
struct Shared {
  union {
    float a[kRows * (kMaxK + 4)];
    AttnDecLds<HD> attn;
    SampleLds sample;
  };
  float raw[(kDecHeads + 2) * HD];  // the position's projections: queries, key, value
  roll_call::Roster who;
  int stop;
};

// Where this launch waits.
struct Patience {
  uint32_t* lost;  // somebody has given up
  int* err_flag;
  // asks again until done(): the values are there; false: given up, here or elsewhere
  template <class Ask, class Done>
  __device__ __forceinline__ bool until(Ask ask, Done done) const {
    const long long t0 = wall_clock64();
    for (int i = 0;; ++i) {
      ask();
      if (!__any(!done())) return true;
      if (wall_clock64() - t0 > kWaitTicks || (i % 16 == 15 && __hip_atomic_load(lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
        __hip_atomic_store(lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicOr(err_flag, kErrUnfinished);
        return false;
      }
    }
  }
};

// Rows m0 .. of a block of eight, K values each, into sh.a (row stride K + 4): values of row m at off + m stride (bytes).
// Absent words are waited for, at first by each wavefront for one of them: many that ask for all of it hold up the stores they
// wait for.  false: the launch ends (the same for all threads; a barrier either way).
template <int N, int HD>  // 32 threads a row, N loads of 16 bytes at once
__device__ __forceinline__ bool take_quads(Shared<HD>& sh, const Patience& wait, Rsrc src, int off, int stride, int m0, int B, int K,
                                           int tid) {
  static_assert(kThreads == 32 * kRows, "");
  const int quads = K / 4, from = off + min(m0 + (tid >> 5), B - 1) * stride, to = (tid >> 5) * (K + 4);
  bool ok = true;
  for (int q0 = tid & 31; q0 - (tid & 31) < quads; q0 += 32 * N) {
    v4f v[N];
    bool there;
    auto ask = [&] {
      there = true;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        v[j] = ld16f(src, from + min(q0 + 32 * j, quads - 1) * 16, 0);
        there = there && !absent(v[j]);
      }
    };
    ok = ok && wait.until(ask, [&] { return there; });
#pragma unroll
    for (int j = 0; j < N; ++j) *reinterpret_cast<v4f*>(&sh.a[to + min(q0 + 32 * j, quads - 1) * 4]) = v[j];
  }
  return ok;
}
template <int HD>
__device__ __forceinline__ bool take_rows(Shared<HD>& sh, const Patience& wait, Rsrc src, int off, int stride, int m0, int B, int K,
                                          int tid) {
  v4f x;
  const int pick = blockIdx.x * (kThreads / 64) + (tid >> 6);  // not all the same one
  const int at = off + min(m0 + pick % kRows, B - 1) * stride + (pick / kRows * 8) % (K / 4) * 16;
  bool ok = wait.until([&] { x = ld16f(src, at, 0); }, [&] { return !absent(x); });
  ok = ok && (kRows * K / 4 <= 2 * kThreads ? take_quads<2>(sh, wait, src, off, stride, m0, B, K, tid)
                                            : take_quads<6>(sh, wait, src, off, stride, m0, B, K, tid));
  if (!ok) sh.stop = 1;
  __syncthreads();
  return sh.stop == 0;
}

// Where a product's values lie: byte offsets in `base` of row 0, and the bytes from row to row.
struct Place {
  Rsrc r;
  float* base;
  int off, stride;  // bytes
};

// The tiles of a phase go round the n workgroups that are there, from workgroup `first` (0 .. n - 1) on.
struct Share {
  int id, n, first;
  // The first tile of this workgroup; its next ones are n apart.  first moves on by the phase's tiles, so that the next one finds
  // workgroups that have its weights.
  __device__ __forceinline__ int first_tile(int total) {
    const int at = id < first ? id + n - first : id - first;
    first = n == kRolloutGrid ? (first + total) % kRolloutGrid : (first + total) % n;
    return at;
  }
};

// C[m, n] = product of the rows at A with W [N, K]: of the norm (gain: not NULL) or of the rows themselves plus the value at R.
// behind(m0, nb, n_nb, columns): what else a tile does between operand and result.
template <int NC_, int HD, class Behind>
__device__ __forceinline__ bool product_of(Shared<HD>& sh, const Patience& wait, Share& work, const Place& A, const Place& C, const Place& R,
                                        const float* W, const float* gain, bool swiglu, int B, int N, int K, float eps,
                                        Behind behind) {
  using Tile = RowsTile<ROWS_ANY, NC_>;
  constexpr int MR = Tile::MR, NC = Tile::NC, kAhead = 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, columns = swiglu ? NC / 2 : NC;
  const int n_nb = (N + 4 * columns - 1) / (4 * columns), total = n_nb * ((B + kRows - 1) / kRows);
  int held = -1;
  for (int u = work.first_tile(total); u < total; u += work.n) {
    Tile t;
    t.any_norm = gain != nullptr;
    t.any_swiglu = swiglu;
    const int nb = u % n_nb, mb = u / n_nb, m0 = mb * MR, n0 = (nb * 4 + wave) * columns;
    const float* wp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wp[c] = W + (size_t)t.weight_row(min(n0, N - 1), c, N) * K;
    float4 w[kAhead][NC], g[kAhead];
    auto load = [&](int k0) {
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        const int k = min(k0 + j * 256 + lane * 4, K - 4);
#pragma unroll
        for (int c = 0; c < NC; ++c) w[j][c] = *(const float4*)(wp[c] + k);
        g[j] = gain ? *(const float4*)(gain + k) : make_float4(1.f, 1.f, 1.f, 1.f);
      }
    };
    load(0);
    const int m = m0 + Tile::row(lane), n = n0 + Tile::column(lane);
    const bool mine = t.owns(lane) && m < B && n < N;
    if (held != mb) {
      if (held >= 0) __syncthreads();  // the block before has been multiplied
      held = mb;
      if (!take_rows(sh, wait, A.r, A.off, A.stride, m0, B, K, tid)) return false;
    }
    float old = 0.f;
    if (!gain) old = ld4(R.base + (size_t)(R.off + min(m, B - 1) * R.stride) / 4 + min(n, N - 1));  // older than A: it is there
    behind(m0, nb, n_nb, columns);
    for (int k0 = 0; k0 < K; k0 += kAhead * 256) {
      if (k0) load(k0);
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        const int k = k0 + j * 256 + lane * 4;
        if (k < K) {
          float4 a[MR];
#pragma unroll
          for (int i = 0; i < MR; ++i) a[i] = *(const float4*)&sh.a[i * (K + 4) + k];
          t.add(a, w[j], g[j]);
        }
      }
    }
    float sum = t.finish(lane, K, eps);
    if (!gain) sum = old + sum;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // of behind(): its stores come first
    if (mine) st4(C.base + (size_t)(C.off + m * C.stride) / 4 + n, present(sum));
  }
  if (held >= 0) __syncthreads();  // sh.a makes room
  return true;
}
// Two weight rows per wavefront while that is one round: what a wavefront multiplies and folds is half of a phase (8 rows, d 256:
// 47.6 us a step with four, 44.6 with two).
template <int HD, class Behind>
__device__ __forceinline__ bool product(Shared<HD>& sh, const Patience& wait, Share& work, const Place& A, const Place& C, const Place& R,
                                        const float* W, const float* gain, bool swiglu, int B, int N, int K, float eps,
                                        Behind behind) {
  const int per = swiglu ? 4 : 8;
  return (N + per - 1) / per * ((B + kRows - 1) / kRows) <= kRolloutGrid
             ? product_of<2>(sh, wait, work, A, C, R, W, gain, swiglu, B, N, K, eps, behind)
             : product_of<4>(sh, wait, work, A, C, R, W, gain, swiglu, B, N, K, eps, behind);
}

template <int HD>
__device__ __forceinline__ bool attention_step(Shared<HD>& sh, const Patience& wait, Share& work, const RolloutArgs& a,
                                               const Place& qkv, const Place& o, int layer, int step) {
  const int tid = threadIdx.x, Hq = a.Hq, Hkv = a.pool.n_kv_heads, G = Hq / Hkv, total = a.B * Hkv;
  for (int u = work.first_tile(total); u < total; u += work.n) {
    const int t = u / Hkv, g = u % Hkv, pos = (a.row_pos ? a.row_pos[t] : a.pos_base) + step;
    const int* table = a.pool.page_table + (size_t)t * a.pool.max_pages;
    const AttnDecHeld<HD> held = attention_dec_hold<HD>(tid, pos, table, a.cos, a.sin, a.pool, layer, g);
    const float* row = qkv.base + (size_t)(qkv.off + t * qkv.stride) / 4;
    const int n = (G + 2) * HD;  // queries, key, value of the kv head
    constexpr int N = ((kDecHeads + 2) * HD + kThreads - 1) / kThreads;
    float x[N];
    auto from = [&](int e) {
      if (e < G * HD) return g * G * HD + e;
      return (e < (G + 1) * HD ? Hq + g - G : Hq + Hkv + g - (G + 1)) * HD + e;
    };
    bool all;
    auto ask = [&] {
      all = true;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        x[j] = ld4(row + from(min(tid + j * kThreads, n - 1)));
        all = all && !absent(x[j]);
      }
    };
    if (!wait.until(ask, [&] { return all; })) sh.stop = 1;
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (tid + j * kThreads < n) sh.raw[tid + j * kThreads] = x[j];
    __syncthreads();
    if (sh.stop) return false;
    float* out = o.base + (size_t)(o.off + t * o.stride) / 4 + g * G * HD;
    attention_dec_unit<HD>(sh.attn, tid, G, true, pos, table, a.pool, layer, g, held,
                           [&](int h, int i) { return sh.raw[h * HD + i]; }, [&](int i) { return sh.raw[G * HD + i]; },
                           [&](int i) { return sh.raw[(G + 1) * HD + i]; },
                           [&](int h, int c, float v) { st4(out + h * HD + c, present(v)); });
    __syncthreads();
  }
  return true;
}

template <int HD>
__device__ __forceinline__ bool sample_step(Shared<HD>& sh, const Patience& wait, Share& work, const RolloutArgs& a, const bf16::SampleCtl& ctl,
                                            const Place& logits, const Place& next, int step) {
  constexpr int kShare = kSampleWaves * 64 / kThreads;  // wavefronts of k_sample per wavefront here
  const int tid = threadIdx.x, V = a.V;
  for (int b = work.first_tile(a.B); b < a.B; b += work.n) {
    SampleState st[kShare];
    bool ok = true;
    const int row = logits.off + b * logits.stride;
    for (int v0 = tid; (v0 - tid) * 4 < V; v0 += kShare * kThreads) {
      v4f z[kShare];
      float4 noise[kShare];  // before the logits are there
#pragma unroll
      for (int j = 0; j < kShare; ++j) noise[j] = sample_noise(v0 + j * kThreads, ctl, step, b);
      bool all;
      auto ask = [&] {
        all = true;
#pragma unroll
        for (int j = 0; j < kShare; ++j) {
          const int v4 = v0 + j * kThreads;
          z[j] = ld16f(logits.r, row + min(v4 * 4, (V - 1) / 4 * 4) * 4, 0);
#pragma unroll
          for (int k = 0; k < 4; ++k) all = all && (v4 * 4 + k >= V || !absent(z[j][k]));
        }
      };
      ok = ok && wait.until(ask, [&] { return all; });
#pragma unroll
      for (int j = 0; j < kShare; ++j) {
        const int v4 = v0 + j * kThreads;
        const float zs[4] = {z[j][0], z[j][1], z[j][2], z[j][3]};
        if (v4 * 4 < V) st[j].push(zs, noise[j], v4, V, ctl);
      }
    }
    if (!ok) sh.stop = 1;
#pragma unroll
    for (int j = 0; j < kShare; ++j) st[j].publish(sh.sample, j * (kThreads / 64) + (tid >> 6), tid & 63);
    __syncthreads();
    if (sh.stop) return false;
    if (tid < 64) {
      const int tok = sample_row(sh.sample, ctl, b, step, V, tid, a.cur_ids, a.err_flag,
                                 [&](int v) { return ld4(logits.base + (size_t)row / 4 + v); });
      if (tid == 0) sh.sample.tok = tok;
    }
    __syncthreads();
    if (step + 1 < a.last_step) {
      const float* e = a.embed + (size_t)sh.sample.tok * a.d;
      float* h = next.base + (size_t)(next.off + b * next.stride) / 4;
      for (int c = tid; c < a.d; c += kThreads) st4(h + c, present(e[c]));
    }
    __syncthreads();
  }
  return true;
}

// One instance of each kind of phase: the code of a step has to stay in the instruction cache (64 KB for two CUs; a copy per
// phase was 129 KB).
template <int HD>
__global__ __launch_bounds__(kThreads) void k_rollout(RolloutArgs a) {
  __shared__ Shared<HD> sh;
  const int tid = threadIdx.x;
  if (tid == 0) {
    sh.stop = 0;
    const long long t0 = wall_clock64();
    auto expired = [&] { return wall_clock64() - t0 > a.roll_ticks; };
    sh.who = roll_call::join(Word{a.sync}, Word{a.sync + 64}, kRolloutGrid, expired);
    if (sh.who.n == kRolloutGrid) sh.who.id = blockIdx.x;  // neighbouring tiles on different dies
    else if (sh.who.id == 0) __hip_atomic_store(a.gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (a.told && expired()) atomicOr(a.err_flag, kErrStalled);
  }
  __syncthreads();
  Share work{__builtin_amdgcn_readfirstlane(sh.who.id), __builtin_amdgcn_readfirstlane(sh.who.n), 0};
  if (work.id < 0) return;
  const bf16::SampleCtl ctl = *a.ctl;
  const Patience wait{a.sync + 128, a.err_flag};
  const int nq = a.Hq * HD, nqkv = nq + 2 * a.pool.n_kv_heads * HD, per_layer = nqkv + nq + 2 * a.d + a.F;
  const int stride = a.row_floats * 4;
  const Rsrc all = rsrc_of(a.sets);
  for (int b = work.id; b < a.B; b += work.n)  // what the sampler before this launch has left
    for (int c = tid; c < a.d; c += kThreads)
      st4(a.sets + ((size_t)(a.first_step % kSets) * a.B + b) * a.row_floats + c, present(a.h0[(size_t)b * a.d + c]));
  for (int step = a.first_step; step < a.last_step; ++step) {
    const int set = step % kSets * a.B * stride, next = (step + 1) % kSets * a.B * stride, last = (step + 2) % kSets * a.B * stride;
    auto place = [&](int off) { return Place{all, a.sets, set + off * 4, stride}; };
    Place h = place(0);
    const Place logits = place(a.d + a.n_layers * per_layer);
    work.first = 0;
    for (int l = 0, phase = 0;; phase = (phase + 1) & 3, l += phase == 0) {
      const bool head = l == a.n_layers;
      const int at = a.d + l * per_layer;
      const size_t w = (size_t)l * a.layer_stride;
      auto of = [&](const float* p) { return (const float*)((const char*)p + w); };
      const Place qkv = place(at), o = place(at + nqkv), h1 = place(at + nqkv + nq), act = place(at + nqkv + nq + a.d),
                  h2 = place(at + nqkv + nq + a.d + a.F);
      // QKV projection or LM head; O projection; gate / up; down
      Place A = h, C = head ? logits : qkv;
      const float *W = head ? a.lm_head : of(a.wqkv), *gain = head ? a.final_norm : of(a.attn_norm);
      int N = head ? a.V : nqkv, K = a.d;
      if (phase == 1) {
        A = o; C = h1; W = of(a.wo); gain = nullptr; N = a.d; K = nq;
      } else if (phase == 2) {
        A = h1; C = act; W = of(a.wgu); gain = of(a.ffn_norm); N = a.F;
      } else if (phase == 3) {
        A = act; C = h2; W = of(a.wdown); gain = nullptr; N = a.d; K = a.F;
      }
      // behind the LM head's operand: a tile's share of its rows in the last set, by the wavefronts that have logits to store
      auto clear = [&](int m0, int nb, int n_nb, int per) {
        if (!head) return;
        const int quads = min(kRows, a.B - m0) * (a.row_floats / 4), share = (quads + n_nb - 1) / n_nb;
        const int threads = min(kThreads, (a.V - nb * 4 * per + per - 1) / per * 64);
        for (int e = nb * share + tid; tid < threads && e < min(quads, (nb + 1) * share); e += threads)
          st16(all, last + m0 * stride + e * 16, 0, v4u{kAbsent, kAbsent, kAbsent, kAbsent});
      };
      if (!product(sh, wait, work, A, C, phase == 3 ? h1 : h, W, gain, phase == 2, a.B, N, K, a.eps, clear)) return;
      if (head) break;
      if (phase == 0 && !attention_step<HD>(sh, wait, work, a, qkv, o, l, step)) return;
      if (phase == 3) h = h2;
    }
    if (!sample_step(sh, wait, work, a, ctl, logits, Place{all, a.sets, next, stride}, step)) return;
  }
}

}  // namespace

size_t rollout_row_floats(int n_layers, int d, int Hq, int Hkv, int hd, int F, int V) {
  const size_t nq = (size_t)Hq * hd;
  return (d + n_layers * (2 * nq + 2 * (size_t)Hkv * hd + 2 * (size_t)d + F) + V + 3) / 4 * 4;
}
bool rollout_fits(const RolloutArgs& a) {
  const int hd = a.pool.head_dim, nq = a.Hq * hd, nqkv = nq + 2 * a.pool.n_kv_heads * hd;
  // The products' form for few rows, operands in LDS, values four at a time, one workgroup per kv head's queries, all sets within a
  // descriptor's reach; and few tiles: every product of a block in one round, the LM head in two.  Steps as launches of their own / here: d 256, 4096 ids,
  // 8 rows 59 / 43 us, 16 rows 60 / 47, 32 rows (four rounds) 82 / 92; d 960, F 1920, 8 rows 97 / 86, 16 rows (two rounds) 124 / 156;
  // d 1280, 8000 ids, 8 rows 100 / 97, 12 rows (four rounds) 109 / 124.  And few keys: a workgroup here takes its units one after the
  // other with nobody else on its CU; d 256, 8 rows, 400 keys 100 / 100, 700 keys 136 / 154, 1400 keys 242 / 284
  const int blocks = (a.B + kRows - 1) / kRows;
  if (std::max({(nqkv + 15) / 16, (a.d + 15) / 16, (a.F + 7) / 8}) * blocks > kRolloutGrid ||
      (a.V + 15) / 16 * blocks > 2 * kRolloutGrid || a.pool.max_pages * kPageTokens > 384)
    return false;
  return (hd == 64 || hd == 128) && a.Hq % a.pool.n_kv_heads == 0 && a.Hq / a.pool.n_kv_heads <= kDecHeads && a.d % 4 == 0 &&
         a.F % 4 == 0 && std::max({a.d, a.F, nq}) <= kMaxK && few_rows(a.B, std::max({nqkv, a.d, 2 * a.F, a.V})) &&
         kSets * (size_t)a.B * a.row_floats * 4 < (size_t)kReach;
}
void rollout(const RolloutArgs& a, hipStream_t st) {
  launch_fill_u32((uint32_t*)a.sets, kAbsent, kSets * (size_t)a.B * a.row_floats, st);
  launch_fill_u32(a.sync, 0u, kRolloutSyncWords, st);
  if (a.pool.head_dim == 64) k_rollout<64><<<kRolloutGrid, kThreads, 0, st>>>(a);
  else k_rollout<128><<<kRolloutGrid, kThreads, 0, st>>>(a);
}

}  // namespace f32
}  // namespace mtmc
