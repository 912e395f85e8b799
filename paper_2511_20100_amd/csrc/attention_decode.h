// Pieces of the decode attention: what its own launch (decode_bf16.hip) and the persistent decode step
// (decode_persistent.hip) both work with.
#pragma once

#include "attention_core.h"
#include "bf16_kernels.h"
#include "device_utils.h"
#include "frag.h"

namespace mtmc {
namespace bf16 {

template <int HD>
__device__ __forceinline__ h16_t* dec_page(const KvPool& pool, int layer, int which, int page, int g) {
  return (h16_t*)pool.base +
         ((((size_t)layer * 2 + which) * pool.n_pages + page) * pool.n_kv_heads + g) * (size_t)(kPageTokens * HD);
}

constexpr int AW = 8;        // wavefronts per workgroup
constexpr int AGMAX = 8;     // query heads per kv head at most
constexpr int ATAB = 512;    // page-table entries of one chunk kept in LDS

template <int HD>
struct KvFrags {
  v8h k[2][HD / 32];
  v4u v[HD / 16];
};
template <int HD>
__device__ __forceinline__ void load_keys(KvFrags<HD>& f, const h16_t* K0, const h16_t* K1, int lane) {
#pragma unroll
  for (int kb = 0; kb < HD / 32; ++kb) {
    f.k[0][kb] = load_frag(K0 + kb * 512, lane);
    f.k[1][kb] = load_frag(K1 + kb * 512, lane);
  }
}
template <int HD>
__device__ __forceinline__ void load_values(KvFrags<HD>& f, const h16_t* V0, const h16_t* V1, int lane) {
  const int voff = (lane & 15) * kPageTokens + 4 * (lane >> 4);
#pragma unroll
  for (int cb = 0; cb < HD / 16; ++cb) {
    const uint2 x = *reinterpret_cast<const uint2*>(V0 + cb * 256 + voff);
    const uint2 y = *reinterpret_cast<const uint2*>(V1 + cb * 256 + voff);
    f.v[cb] = v4u{x.x, x.y, y.x, y.y};
  }
}
template <int HD>
__device__ __forceinline__ KvFrags<HD> load_kv(const h16_t* K0, const h16_t* K1, const h16_t* V0, const h16_t* V1,
                                               int lane) {
  KvFrags<HD> f;
  load_keys<HD>(f, K0, K1, lane);
  load_values<HD>(f, V0, V1, lane);
  return f;
}

// One step (two pages, 32 tokens from tok0) of a single block of query columns on loaded fragments.
// The softmax state is kept in base-2 units: scale2 = log2(e) / sqrt(head_dim), st.m = running maximum of
// scale2 * score, weights = 2^(scale2 * score - m) (one v_exp_f32 each).  MASK = false: every token of the step
// is visible to the query (tok0 + 31 <= position), so nothing is compared; the unused columns (zero queries)
// then carry finite garbage that nobody reads.
// In two halves (scores and weights of the keys, then the values), so that a caller can refill what a half has consumed.
template <int HD, bool MASK>
__device__ __forceinline__ v8h attn_weights1(const KvFrags<HD>& f, int tok0, const v8h (&qf)[HD / 32], int qpos,
                                             float scale2, AttnState<HD / 16>& st, int lane) {
  const int lg = lane >> 4;
  v4f s0 = v4f{0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int kb = 0; kb < HD / 32; ++kb) {
    s0 = mfma16(f.k[0][kb], qf[kb], s0);
    s1 = mfma16(f.k[1][kb], qf[kb], s1);
  }
  float sv[8];
  float tmax = -INFINITY;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int t0 = tok0 + 4 * lg + r, t1 = t0 + 16;
    sv[r] = (!MASK || t0 <= qpos) ? s0[r] * scale2 : -INFINITY;
    sv[4 + r] = (!MASK || t1 <= qpos) ? s1[r] * scale2 : -INFINITY;
    tmax = fmaxf(tmax, fmaxf(sv[r], sv[4 + r]));
  }
  tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
  tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
  const float m_new = fmaxf(st.m, tmax);
  const float m_safe = (MASK && m_new == -INFINITY) ? 0.f : m_new;
  const float corr = __builtin_amdgcn_exp2f(st.m - m_safe);
  float p[8], psum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    p[e] = __builtin_amdgcn_exp2f(sv[e] - m_safe);
    psum += p[e];
  }
  st.l = st.l * corr + psum;
  st.m = m_new;
  v4u pk;
  pk[0] = pack_h16x2_inrange(p[0], p[1]);  // weights lie in [0, 1]
  pk[1] = pack_h16x2_inrange(p[2], p[3]);
  pk[2] = pack_h16x2_inrange(p[4], p[5]);
  pk[3] = pack_h16x2_inrange(p[6], p[7]);
  if (__any(corr != 1.0f)) {  // the running maximum of some column moved: rescale what has been summed
#pragma unroll
    for (int cb = 0; cb < HD / 16; ++cb) st.o[cb] = st.o[cb] * corr;
  }
  return __builtin_bit_cast(v8h, pk);
}
template <int HD>
__device__ __forceinline__ void attn_values1(const KvFrags<HD>& f, v8h weights, AttnState<HD / 16>& st) {
#pragma unroll
  for (int cb = 0; cb < HD / 16; ++cb) st.o[cb] = mfma16(__builtin_bit_cast(v8h, f.v[cb]), weights, st.o[cb]);
}
template <int HD, bool MASK>
__device__ __forceinline__ void attn_step1(const KvFrags<HD>& f, int tok0, const v8h (&qf)[HD / 32], int qpos,
                                           float scale2, AttnState<HD / 16>& st, int lane) {
  attn_values1<HD>(f, attn_weights1<HD, MASK>(f, tok0, qf, qpos, scale2, st, lane), st);
}

// Pages [lo, end) of sequence b are the chunk's, [lo, hi) those of its context so far (as k_attn_dec has them).
struct AttnDecRange {
  int pos0, lo, end, pos, hi;
};
__device__ __forceinline__ AttnDecRange attn_dec_pages(const AttnDecArgs& a, int b, int chunk) {
  AttnDecRange r;
  r.pos0 = a.row_pos ? a.row_pos[b] : a.pos_base;
  r.lo = chunk * a.chunk_pages;
  r.end = r.lo + a.chunk_pages;
  if (a.split_at_prompt) {
    const int nb = ((r.pos0 + 1) / kPageTokens) & ~1;  // even: the steps take pages in pairs
    r.lo = chunk ? nb : 0;
    r.end = chunk ? a.pool.max_pages : nb;
  }
  return r;
}
// ... once the step counter is known.  A negative position base marks a slot that holds no sequence (rows packed into fewer
// slots): nothing to attend.
__device__ __forceinline__ void attn_dec_position(const AttnDecArgs& a, int b, int step, AttnDecRange& r) {
  r.pos = r.pos0 + (a.row_step0 ? min(step - a.row_step0[b], a.max_step) : step);
  r.hi = r.pos0 < 0 ? r.lo : min(r.pos / kPageTokens + 1, r.end);
}

}  // namespace bf16
}  // namespace mtmc
