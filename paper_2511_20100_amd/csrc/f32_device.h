// What a step of the fp32 path computes, for the launches of its own (kernels_f32.hip) and for the form that stays on the
// device for a whole generation (rollout_f32.hip): the same sums in the same order.
#pragma once

#include <type_traits>

#include "bf16_kernels.h"
#include "device_utils.h"

namespace mtmc {
namespace f32 {

// ---- sums over the lanes of a wavefront, without the LDS: between halves and rows of 16 lanes by the swap instructions, inside
// a row by its rotations and mirrors (a shuffle through the LDS is 100 cycles and more, the folds of a product were 1.6 of
// its launch's 4.8 us)
template <int OFF>
__device__ __forceinline__ float from_lane(float x) {  // a lane whose bit OFF differs, in the same row of 16
  static_assert(OFF == 8 || OFF == 4 || OFF == 2 || OFF == 1, "");
  constexpr int kCtrl = OFF == 8 ? 0x128 /* row_ror:8 */ : OFF == 4 ? 0x141 /* row_half_mirror */
                      : OFF == 2 ? 0x4e /* quad_perm 2 3 0 1 */ : 0xb1 /* quad_perm 1 0 3 2 */;
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), kCtrl, 0xf, 0xf, false));
}
// a of the lanes without bit OFF (16 or 32) beside b of these, and the same of the lanes that have it
template <int OFF>
__device__ __forceinline__ float2 swap_lanes(float a, float b) {
  if constexpr (OFF == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
  } else {
    static_assert(OFF == 16, "");
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
}
// f over the two lanes that bit OFF tells apart
template <int OFF, class F>
__device__ __forceinline__ float over_lanes(float x, F f) {
  if constexpr (OFF >= 16) {
    const float2 s = swap_lanes<OFF>(x, x);
    return f(s.x, s.y);
  } else {
    return f(x, from_lane<OFF>(x));
  }
}
template <class F>
__device__ __forceinline__ float over_wave(float x, F f) {
  x = over_lanes<32>(x, f);
  x = over_lanes<16>(x, f);
  x = over_lanes<8>(x, f);
  x = over_lanes<4>(x, f);
  x = over_lanes<2>(x, f);
  return over_lanes<1>(x, f);
}
__device__ __forceinline__ float lanes_sum(float x) {
  return over_wave(x, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float lanes_max(float x) {
  return over_wave(x, [](float a, float b) { return fmaxf(a, b); });
}
// 2 HALF values per lane: lanes OFF apart exchange halves and add, then OFF / 2 apart, ... down to one value per lane,
// the one whose index the lane's bits from OFF downwards spell
template <int HALF, int OFF, int N>
__device__ __forceinline__ void fold_lanes(float (&v)[N], int lane) {
  const bool hi = lane & OFF;
#pragma unroll
  for (int i = 0; i < HALF; ++i) {
    if constexpr (OFF >= 16) {
      const float2 s = swap_lanes<OFF>(v[i], v[i + HALF]);
      v[i] = s.x + s.y;
    } else {
      const float send = hi ? v[i] : v[i + HALF];
      v[i] = (hi ? v[i + HALF] : v[i]) + from_lane<OFF>(send);
    }
  }
  if constexpr (HALF > 1) fold_lanes<HALF / 2, OFF / 2>(v, lane);
}

// ---- products of few rows: 8 rows x 4 (or 2) weight rows per wavefront, its 64 lanes along K.  Every value is the same sum of
// lanes 32, 16, 8, 4, 2 and 1 apart, however many a wavefront has.
//   ROWS_NORM    A is the residual: row m is scaled by gain[k] and, after the sum, by 1 / rms of the row
//   ROWS_SWIGLU  weight rows n and N + n are gate and up of output column n: C = silu(gate) * up
//   ROWS_ANY     norm and swiglu are known at run time
enum { ROWS_ADD = 1, ROWS_NORM = 2, ROWS_SWIGLU = 4, ROWS_ANY = 8 };
__device__ __forceinline__ float dot4(float4 a, float4 b) {  // rounded alike wherever it is inlined
  return fmaf(a.x, b.x, a.y * b.y) + fmaf(a.z, b.z, a.w * b.w);
}
template <int MODE, int NC_ = 4>
struct RowsTile {
  static constexpr int MR = 8, NC = NC_, kLanes = 64 / (MR * NC);  // lanes a value ends up in
  static_assert(NC == 2 || NC == 4, "");
  float v[NC * MR] = {}, ss[MR] = {};
  bool any_norm = false, any_swiglu = false;  // ROWS_ANY

  __device__ __forceinline__ bool norm() const { return MODE == ROWS_ANY ? any_norm : (MODE & ROWS_NORM) != 0; }
  __device__ __forceinline__ bool swiglu() const { return MODE == ROWS_ANY ? any_swiglu : (MODE & ROWS_SWIGLU) != 0; }
  __device__ __forceinline__ int columns() const { return swiglu() ? NC / 2 : NC; }  // output columns per wavefront
  // row of W that is the tile's weight row c (n0: its first output column)
  __device__ __forceinline__ int weight_row(int n0, int c, int N) const {
    return c >= columns() ? min(n0 + c - NC / 2, N - 1) + N : min(n0 + c, N - 1);
  }
  // four values of k per lane
  __device__ __forceinline__ void add(float4 (&a)[MR], const float4 (&w)[NC], float4 gain) {
    if (MODE & (ROWS_NORM | ROWS_ANY)) {  // without a norm the gain is 1
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        ss[i] += dot4(a[i], a[i]);
        a[i].x *= gain.x; a[i].y *= gain.y; a[i].z *= gain.z; a[i].w *= gain.w;
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = 0; i < MR; ++i) v[c * MR + i] += dot4(a[i], w[c]);
  }
  // the value of row i, column c, which the lane ends up with; owns(lane): whether it is the one to store it
  __device__ __forceinline__ static int column(int lane) { return lane / kLanes / MR; }
  __device__ __forceinline__ static int row(int lane) { return lane / kLanes % MR; }
  __device__ __forceinline__ bool owns(int lane) const { return lane % kLanes == 0 && (!swiglu() || lane < 32); }
  __device__ __forceinline__ float finish(int lane, int K, float eps) {
    fold_lanes<MR * NC / 2, 32>(v, lane);  // the first exchange decides the highest bit of the value's index
    auto add = [](float a, float b) { return a + b; };
    float sum = v[0];
    if constexpr (kLanes > 2) sum = over_lanes<2>(sum, add);
    sum = over_lanes<1>(sum, add);
    if (norm()) {
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        ss[i] = over_lanes<32>(ss[i], add);
        if constexpr (NC == 4) ss[i] = over_lanes<16>(ss[i], add);
      }
      fold_lanes<4, 4 * kLanes>(ss, lane);  // by the bits that spell the lane's row
      float t = ss[0];
      if constexpr (kLanes > 2) t = over_lanes<2>(t, add);
      t = over_lanes<1>(t, add);
      sum *= 1.0f / sqrtf(t / (float)K + eps);
    }
    if (swiglu()) {
      const float up = swap_lanes<32>(sum, sum).y;  // the upper lanes have the up rows
      sum = sum / (1.0f + expf(-sum)) * up;
    }
    return sum;
  }
};

__device__ __forceinline__ float* page_ptr(const KvPool& pool, int layer, int which, int page, int g) {
  return (float*)pool.base +
         ((((size_t)layer * 2 + which) * pool.n_pages + page) * pool.n_kv_heads + g) *
             (size_t)(kPageTokens * pool.head_dim);
}

// ---- decode attention (one token per sequence): rotary embedding, append and attention.  A workgroup of 256 threads per
// (sequence, kv head, up to kDecHeads of its query heads): the new key and value are used from LDS (the first workgroup
// of a kv head also writes them to their page).  Keys are taken 256 at a time: every thread scores one for all heads, then
// wavefront h does the online softmax of head h and adds up its values (lane = dims 4 c .. + 3 and a part of the keys):
// two barriers per 256 keys.  The first keys and values are older than the position: held() asks for them before the
// projections are there.
constexpr int kDecHeads = 4;
template <int HD>
struct AttnDecLds {
  static constexpr int PARTS = 64 / (HD / 4);  // 4 parts at 64 dims, 2 at 128
  __attribute__((aligned(16))) float q[kDecHeads][HD];
  __attribute__((aligned(16))) float kn[HD], vn[HD];
  float p[kDecHeads][256];
  __attribute__((aligned(16))) float part[PARTS][kDecHeads][HD];
  float l[kDecHeads];
};
template <int HD>
struct AttnDecHeld {
  static constexpr int C4 = HD / 4, PARTS = AttnDecLds<HD>::PARTS, NV = 16;
  int page;        // of the position
  float cos, sin;  // of the position, dimension tid % (HD / 2)
  float4 k[C4];    // key tid
  float4 v[NV];    // values apart + PARTS j
};
template <int HD>
__device__ __forceinline__ AttnDecHeld<HD> attention_dec_hold(int tid, int pos, const int* table, const float* cos, const float* sin,
                                                              const KvPool& pool, int layer, int g) {
  using Held = AttnDecHeld<HD>;
  Held held;
  const int lane = tid & 63, ac = lane / Held::PARTS, apart = lane % Held::PARTS, last = max(pos - 1, 0);
  const int key = min(tid, last), kpage = table[key / kPageTokens];
  int vpage[Held::NV];
#pragma unroll
  for (int j = 0; j < Held::NV; ++j) vpage[j] = table[min(apart + Held::PARTS * j, last) / kPageTokens];
  held.page = table[pos / kPageTokens];
  held.cos = cos[(size_t)pos * (HD / 2) + tid % (HD / 2)];
  held.sin = sin[(size_t)pos * (HD / 2) + tid % (HD / 2)];
  const float* kp = page_ptr(pool, layer, 0, kpage, g) + (size_t)(key % kPageTokens) * HD;
#pragma unroll
  for (int c = 0; c < Held::C4; ++c) held.k[c] = *(const float4*)(kp + 4 * c);
#pragma unroll
  for (int j = 0; j < Held::NV; ++j) {
    const int at = min(apart + Held::PARTS * j, last);
    held.v[j] = *(const float4*)(page_ptr(pool, layer, 1, vpage[j], g) + (size_t)(at % kPageTokens) * HD + 4 * ac);
  }
  return held;
}
// query(h, i), key(i), value(i): the position's projections; out(h, c, x) takes the result.  nh heads, appends: writes the page.
template <int HD, class Query, class Key, class Value, class Out>
__device__ __forceinline__ void attention_dec_unit(AttnDecLds<HD>& sm, int tid, int nh, bool appends, int pos, const int* table,
                                                   const KvPool& pool, int layer, int g,
                                                   const AttnDecHeld<HD>& held, Query query, Key key_of, Value value_of, Out out) {
  constexpr int HALF = HD / 2, C4 = HD / 4, PARTS = AttnDecLds<HD>::PARTS;
  auto& q = sm.q;
  auto& kn = sm.kn;
  auto& vn = sm.vn;
  auto& p = sm.p;
  auto& part = sm.part;
  auto turned = [](float x, float c, float y, float s) { return fmaf(x, c, y * s); };
  for (int e = tid; e < kDecHeads * HALF; e += 256) {
    const int h = e / HALF, i = e % HALF;
    float lo = 0.f, hi = 0.f;
    if (h < nh) {
      lo = query(h, i);
      hi = query(h, i + HALF);
    }
    q[h][i] = turned(lo, held.cos, hi, -held.sin);  // i is tid % HALF
    q[h][i + HALF] = turned(hi, held.cos, lo, held.sin);
  }
  const int page = held.page, slot = pos % kPageTokens;
  if (tid < HALF) {
    const float lo = key_of(tid), hi = key_of(tid + HALF);
    const float ra = turned(lo, held.cos, hi, -held.sin), rb = turned(hi, held.cos, lo, held.sin);
    kn[tid] = ra;
    kn[tid + HALF] = rb;
    if (appends) {
      float* kp = page_ptr(pool, layer, 0, page, g) + (size_t)slot * HD;
      kp[tid] = ra;
      kp[tid + HALF] = rb;
    }
  } else if (tid >= 64 && tid < 64 + HALF) {
    for (int i = tid - 64; i < HD; i += HALF) {
      const float x = value_of(i);
      vn[i] = x;
      if (appends) page_ptr(pool, layer, 1, page, g)[(size_t)slot * HD + i] = x;
    }
  }
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)HD);
  const int lane = tid & 63, ah = tid >> 6, ac = lane / PARTS, apart = lane % PARTS;
  float m = -INFINITY, l = 0.f;  // of head ah
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  const int n_ctx = pos + 1;
  for (int c0 = 0; c0 < n_ctx; c0 += 256) {
    const int key = c0 + tid;
    if (key < n_ctx) {
      float d[kDecHeads] = {};
      auto score = [&](auto heads, int c, float4 kv) {
#pragma unroll
        for (int h = 0; h < decltype(heads)::value; ++h) d[h] += dot4(*(const float4*)(&q[h][4 * c]), kv);
      };
      // the position's own key comes from LDS, by a selection: through one pointer for both these would be flat loads, four of
      // them in a row, 4 us
      auto own = [&](int c, float4 kv) { return key == pos ? *(const float4*)(kn + 4 * c) : kv; };
      using Two = std::integral_constant<int, 2>;
      using All = std::integral_constant<int, kDecHeads>;
      if (c0 == 0 && nh <= 2) {
#pragma unroll
        for (int c = 0; c < C4; ++c) score(Two{}, c, own(c, held.k[c]));
      } else if (c0 == 0) {
#pragma unroll
        for (int c = 0; c < C4; ++c) score(All{}, c, own(c, held.k[c]));
      } else {
        const int at = min(key, pos - 1);
        const float* kp = page_ptr(pool, layer, 0, table[at / kPageTokens], g) + (size_t)(at % kPageTokens) * HD;
#pragma unroll 4
        for (int c = 0; c < C4; ++c) score(All{}, c, own(c, *(const float4*)(kp + 4 * c)));
      }
#pragma unroll
      for (int h = 0; h < kDecHeads; ++h) p[h][tid] = d[h] * scale;
    } else {
#pragma unroll
      for (int h = 0; h < kDecHeads; ++h) p[h][tid] = -INFINITY;
    }
    __syncthreads();
    float s[4], mx = m;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = p[ah][lane + 64 * i];
      mx = fmaxf(mx, s[i]);
    }
    mx = lanes_max(mx);
    const float corr = expf(m - mx);  // exp(-inf) = 0 on the first chunk
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = c0 + lane + 64 * i < n_ctx ? expf(s[i] - mx) : 0.f;
      p[ah][lane + 64 * i] = e;  // read back by this wavefront only
      sum += e;
    }
    l = fmaf(l, corr, lanes_sum(sum));
    m = mx;
    acc.x *= corr; acc.y *= corr; acc.z *= corr; acc.w *= corr;
    __builtin_amdgcn_wave_barrier();
    const int n_here = min(256, n_ctx - c0);
    auto weigh = [&](float w, float4 vv) {
      acc.x = fmaf(w, vv.x, acc.x); acc.y = fmaf(w, vv.y, acc.y); acc.z = fmaf(w, vv.z, acc.z); acc.w = fmaf(w, vv.w, acc.w);
    };
    const float4 new_v = *(const float4*)(vn + 4 * ac);
    int i = apart;
    if (c0 == 0) {
#pragma unroll
      for (int j = 0; j < AttnDecHeld<HD>::NV; ++j) {
        const int kk = apart + PARTS * j;
        float4 vv = kk == pos ? new_v : held.v[j];
        if (kk >= n_here) vv = make_float4(0.f, 0.f, 0.f, 0.f);
        weigh(p[ah][kk], vv);  // no key, no weight
      }
      i += PARTS * AttnDecHeld<HD>::NV;
    }
#pragma unroll 4
    for (; i < n_here; i += PARTS) {
      const int kk = c0 + i;
      const int at = min(kk, pos - 1);
      const float4 vv = *(const float4*)(page_ptr(pool, layer, 1, table[at / kPageTokens], g) + (size_t)(at % kPageTokens) * HD + 4 * ac);
      weigh(p[ah][i], kk == pos ? new_v : vv);
    }
    __syncthreads();  // the scores make room for the next keys'
  }
  if (lane == 0) sm.l[ah] = l;
  *(float4*)(&part[apart][ah][4 * ac]) = acc;
  __syncthreads();
  for (int e = tid; e < nh * HD; e += 256) {
    const int h = e / HD, c = e % HD;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < PARTS; ++w) sum += part[w][h][c];
    out(h, c, sum / sm.l[h]);
  }
}

// ---- sampling from the logits of a row by kSampleWaves wavefronts, or by fewer that each do the work of several
constexpr int kSampleWaves = 16;
struct SampleLds {
  Lse lse[kSampleWaves];
  Best best[kSampleWaves];
  int tok;
};
// the larger logit, the lower index of equal ones; over the lanes that bit OFF tells apart
template <int OFF>
__device__ __forceinline__ Best best_over_lanes(Best b) {
  if constexpr (OFF >= 16) {
    const float2 y = swap_lanes<OFF>(b.y, b.y), i = swap_lanes<OFF>(__int_as_float(b.idx), __int_as_float(b.idx));
    return best_merge(Best{y.x, __float_as_int(i.x)}, Best{y.y, __float_as_int(i.y)});
  } else {
    return best_merge(b, Best{from_lane<OFF>(b.y), __float_as_int(from_lane<OFF>(__int_as_float(b.idx)))});
  }
}
// what is added to the logits 4 v4 .. of row b
__device__ __forceinline__ float4 sample_noise(int v4, const bf16::SampleCtl& ctl, int step, int b) {
  if (ctl.greedy) return make_float4(0.f, 0.f, 0.f, 0.f);
  const uint4 r = philox4x32_10(make_uint4((uint32_t)v4, (uint32_t)step, ctl.seq_offset + b, 0u), ctl.key0, ctl.key1);
  return make_float4(gumbel_from_bits(r.x), gumbel_from_bits(r.y), gumbel_from_bits(r.z), gumbel_from_bits(r.w));
}
struct SampleState {
  Lse lse = lse_empty();
  Best best = best_empty();
  // logits 4 v4 .. of the row
  __device__ __forceinline__ void push(const float (&z)[4], float4 noise, int v4, int V, const bf16::SampleCtl& ctl) {
    const float add[4] = {noise.x, noise.y, noise.z, noise.w};
    float zt[4], m = lse.m;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = v4 * 4 + k;
      zt[k] = v < V ? (ctl.greedy ? z[k] : z[k] * ctl.inv_temp) : -INFINITY;
      m = zt[k] > m ? zt[k] : m;
      if (v < V) best = best_merge(best, Best{zt[k] + add[k], v});
    }
    if (m == -INFINITY) {  // nothing yet (a NaN counts)
#pragma unroll
      for (int k = 0; k < 4; ++k) lse.s += zt[k] == -INFINITY ? 0.f : zt[k];
      return;
    }
    float s = lse.s * expf(lse.m - m);
#pragma unroll
    for (int k = 0; k < 4; ++k) s += expf(zt[k] - m);
    lse = Lse{m, s};
  }
  __device__ __forceinline__ Lse lse_over_lanes() const {
    const float m = lanes_max(lse.m);
    return Lse{m, lanes_sum(m == -INFINITY ? lse.s : lse.s * expf(lse.m - m))};
  }
  __device__ __forceinline__ Best best_over_wave() const {
    Best b = best_over_lanes<32>(best);
    b = best_over_lanes<16>(b);
    b = best_over_lanes<8>(b);
    b = best_over_lanes<4>(b);
    b = best_over_lanes<2>(b);
    return best_over_lanes<1>(b);
  }
  // of the wavefront, which is number w of kSampleWaves
  __device__ __forceinline__ void publish(SampleLds& sm, int w, int lane) const {
    const Lse l = lse_over_lanes();
    const Best b = best_over_wave();
    if (lane == 0) {
      sm.lse[w] = l;
      sm.best[w] = b;
    }
  }
};
// One wavefront, behind a barrier: writes the token's id and log-probability; returns the id whose embedding comes next.
// logit(v): the row's logit.
template <class Logit>
__device__ __forceinline__ int sample_row(const SampleLds& sm, const bf16::SampleCtl& ctl, int b, int step, int V, int lane,
                                          int* cur_ids, int* err_flag, Logit logit) {
  SampleState st;
  if (lane < kSampleWaves) {
    st.lse = sm.lse[lane];
    st.best = sm.best[lane];
  }
  const Lse lse = st.lse_over_lanes();
  const Best best = st.best_over_wave();
  if (lane) return 0;
  // no logit compared greater than -inf: the token is out of range, which its embedding reports
  const float zb = best.idx < V ? logit(best.idx) : NAN;
  const float zt = ctl.greedy ? zb : zb * ctl.inv_temp;
  int tok = best.idx;
  float lp = zt - (lse.m + logf(lse.s));
  if (ctl.done) {
    if (__hip_atomic_load(ctl.done + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
      tok = ctl.stop_id;
      lp = 0.f;
    } else if (tok == ctl.stop_id) {
      __hip_atomic_store(ctl.done + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ctl.out_lens[b] = step + 1;
    }
  }
  cur_ids[b] = tok;
  ctl.out_ids[(size_t)b * ctl.max_new + step] = tok;
  ctl.out_logprobs[(size_t)b * ctl.max_new + step] = lp;
  if (tok < 0 || tok >= V) {
    atomicOr(err_flag, 1);
    tok = tok < 0 ? 0 : V - 1;
  }
  return tok;
}

}  // namespace f32
}  // namespace mtmc
