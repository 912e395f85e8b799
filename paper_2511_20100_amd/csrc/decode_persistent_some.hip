// The residual blocks of a decode step by whatever workgroups are there: what does the step when the persistent launch before
// it (decode_persistent.hip, decode_persistent_rows.hip) was given up because something else held a part of the device.  Behind one that
// was not, which is the rule, its workgroups look at a word and leave.  With the roll call that costs up to 4 us a step (63 steps of
// one row 62.64 -> 62.66 ms, 127 of 64 rows 219.5 -> 220.0), by as many workgroups as there are CUs or by 16.
//
// The workgroups that come within 20 us share all units of each phase out among themselves, one after the other, and wait for each
// other alone (roll_call.h), so it ends however few they are.  Every sum has the ranges and the order of the launches it
// stands in for, a wavefront adds them up for a tile by itself, and everything handed on goes past the caches: the same bits, in
// 2.4 (16 rows) to 2.9 (one row) times their time with the device to itself (63 steps of the 1.5 B shape: 91 -> 218 ms, 89 -> 260).
#include "decode_persistent.h"

namespace mtmc {
namespace bf16 {
namespace persist {
namespace {

constexpr int kWaves = AW, kThreads = kWaves * 64;
constexpr long long kRosterTicks = 2000;

template <int BT>
struct Shared {
  AttnLds at;
  int table[ATAB];
  float part[16 * BT][64];  // partial sums of a row's squares
  float total[2][16 * BT];  // sums of the rows' squares: now, and of the older residual
  roll_call::Roster who;
  int lost;
};

// The sums of the rows' squares in P partial sums each (part p: tiles p, p + P, ...), all threads.
template <int BT>
__device__ __forceinline__ void row_totals(Shared<BT>& sh, int which, const float* ss, int nt_d, int P) {
  const int parts = min(P, nt_d);
  for (int e = threadIdx.x; e < 16 * BT * parts; e += kThreads) {
    const int row = e / parts, p = e - row * parts;
    float sum = 0.f;
    for (int t = p; t < nt_d; t += P) sum += ld4(ss + row * kPersistGrid + t);
    sh.part[row][p] = sum;
  }
  __syncthreads();
  if (threadIdx.x < 16 * BT) {
    float sum = 0.f;
    for (int p = 0; p < parts; ++p) sum += sh.part[threadIdx.x][p];
    sh.total[which][threadIdx.x] = sum;
  }
  __syncthreads();
}

using Rows = Operand<1, kDeviceScope>;

// Row tile at `row` (bytes into w) times the rows of x over k tiles k0 .. k0 + n - 1 of both.
__device__ __forceinline__ v4f range_of(Rsrc w, int row, const Rows& x, int k0, int n, int lane) {
  constexpr int kAhead = 4;
  v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < n; i0 += kAhead) {
    v8h wf[kAhead], xf[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int k = k0 + min(i0 + j, n - 1);
      wf[j] = load_weight(w, lane * 16, row + k * 1024);
      xf[j] = x.tile(0, k);
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
      if (i0 + j < n) acc = mfma16(wf[j], xf[j], acc);
  }
  return acc;
}
// ... over k tiles kbeg .. kend - 1 in `ranges` ranges, added up in order
__device__ __forceinline__ v4f ranges_of(Rsrc w, int row, const Rows& x, int kbeg, int kend, int ranges, int lane) {
  const int per = (max(kend - kbeg, 0) + ranges - 1) / ranges;
  v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < ranges; ++s) sum = sum + range_of(w, row, x, kbeg + s * per, min(per, kend - (kbeg + s * per)), lane);
  return sum;
}

// The O projection behind a split context: heads v, v + R, ... are range v; a head's chunks are combined by their share.
__device__ __forceinline__ v4f heads_of(const PersistArgs& a, Rsrc w, int row, const Rows& x, int mt, int lane) {
  const int NC = a.at.n_chunks, Hq = a.at.Hq, R = a.o_ranges, m = mt * 16 + (lane & 15);
  const int chunk_bytes = (int)(a.at.o_chunk_stride * sizeof(h16_t));
  v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
  for (int v = 0; v < R; ++v) {
    v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
    for (int head = v; head < Hq; head += R) {
      float ck[8], lk[8], mx = -INFINITY, den = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool live = k < NC && m < a.B;
        const uint2 st = ld8(a.at.ml + (((size_t)min(m, a.B - 1) * Hq + head) * NC + min(k, NC - 1)) * 2);
        ck[k] = live ? __uint_as_float(st.x) : -INFINITY;
        lk[k] = live ? __uint_as_float(st.y) : 0.f;
        mx = fmaxf(mx, ck[k]);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        ck[k] = lk[k] > 0.f ? lk[k] * expf(ck[k] - mx) : 0.f;
        den += ck[k];
      }
      v8h wf[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) wf[t] = load_weight(w, lane * 16, row + (head * 4 + t) * 1024);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (k >= NC) break;
        const float share = den > 0.f ? ck[k] / den : 0.f;
        v4f part = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) part = mfma16(wf[t], x.load(0, k * chunk_bytes + (head * 4 + t) * x.step), part);
        acc = acc + part * share;
      }
    }
    sum = sum + acc;
  }
  return sum;
}

template <int BT>
__global__ __launch_bounds__(kThreads, 2) void k_decode_layers_some(PersistArgs a) {
  __shared__ Shared<BT> sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid == 0) {
    sh.who = roll_call::Roster{-1, 0};
    sh.lost = 0;
    if (word_of(a, kPersistEnded).load() == kPersistSkipped) {
      const long long t0 = wall_clock64();
      sh.who = roll_call::join(word_of(a, kPersistSeats), word_of(a, kPersistList), gridDim.x,
                               [&] { return wall_clock64() - t0 > kRosterTicks; });
    }
  }
  __syncthreads();
  const int id = __builtin_amdgcn_readfirstlane(sh.who.id), n = __builtin_amdgcn_readfirstlane(sh.who.n);
  if (id < 0) return;

  uint32_t met = 0;
  // Until all that are on the list have come here; what they have stored is where others see it.
  auto meet = [&] {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    ++met;
    if (tid == 0) {
      const Word word = word_of(a, kPersistMet);
      const long long t0 = wall_clock64();
      word.add(1);
      while (word.load() < met * n) {
        if (wall_clock64() - t0 <= kWaitTicks && word_of(a, kPersistEnded).load() == kPersistSkipped) continue;
        atomicOr(a.err_flag, kErrUnfinished);
        word_of(a, kPersistEnded).store(kPersistLost);
        sh.lost = 1;
        break;
      }
    }
    __syncthreads();
    return sh.lost == 0;
  };
  const int first = id * kWaves + wave, stride = n * kWaves, col = lane & 15, rq = (lane >> 4) * 4;
  // f(tile, mt) for this wavefront's share of tiles x BT
  auto share = [&](int tiles, auto f) {
    for (int i = first; i < tiles * BT; i += stride) f(i / BT, i % BT);
  };
  const int B = a.B, nt_d = a.nt_d;
  const Rsrc qkv = rsrc_of(a.qkv), part = rsrc_of(a.part);
  for (int l = 0; l < a.n_layers; ++l) {
    auto weights = [&](const h16_t* w) { return rsrc_of(w + (size_t)l * a.layer_stride / sizeof(h16_t)); };
    auto gains = [&](const float* p, int layer) { return (const float*)((const char*)p + layer * a.layer_stride); };
    // h += sum, the operand behind it and its squares
    auto residual = [&](const TileOut& to, int nt, int mt, v4f sum, const float* gain) {
      const int m = mt * 16 + col;
      const v4f h_old = ld16f(to.h, (min(m, B - 1) * to.d + nt * 16 + rq) * 4, 0);
      residual_tile<BT>(to, nt, mt, lane, sum, h_old, *reinterpret_cast<const v4f*>(gain + nt * 16 + rq),
                        scale_of(sh.total[0][m], 0.f, false, a.inv_d, a.eps));
    };
    // ---- QKV projection
    if (l > 0) {
      row_totals<BT>(sh, 0, a.ss_in[0], nt_d, 4 * a.qkv_ranges / BT);
      row_totals<BT>(sh, 1, a.ss_in[1], nt_d, 4 * a.qkv_ranges / BT);
    }
    share(a.nt_qkv, [&](int nt, int mt) {
      const int m = mt * 16 + col;
      const v4f sum = ranges_of(weights(a.wqkv), nt * a.kt_d * 1024, Rows::tiled(x_of(a, l), BT, mt, lane, B), 0, a.kt_d, a.qkv_ranges, lane);
      const float sc = l > 0 ? scale_of(sh.total[0][m], sh.total[1][m], true, a.inv_d, a.eps) : 1.f;
      if (m < B) st16(qkv, ((m * a.nt_qkv + nt) * 16 + rq) * 4, 0, __builtin_bit_cast(v4u, sum * sc));
    });
    if (!meet()) return;
    // ---- attention
    for (int place = id; place < kPersistGrid; place += n) {
      const AttnHeld unit(a, place, wave, lane, sh.table, 16 * BT);
      __syncthreads();
      if (unit.active) attend<false>(unit, sh.at, sh.table, l, wave, counted_unit(16 * BT, [] { return true; }));
      __syncthreads();
    }
    if (!meet()) return;
    // ---- O projection
    row_totals<BT>(sh, 0, a.ss_in[0], nt_d, 4 * a.o_ranges / BT);
    {
      const TileOut to(a, a.xo + (size_t)l * a.x_stride, 1, l + 1 == a.n_layers);
      share(nt_d, [&](int nt, int mt) {
        const Rows x = Rows::tiled(a.at.o, BT, mt, lane, B);
        const int row = nt * a.kt_nq * 1024;
        const v4f sum = a.at.n_chunks == 1 ? ranges_of(weights(a.wo), row, x, 0, a.kt_nq, a.o_ranges, lane)
                                           : heads_of(a, weights(a.wo), row, x, mt, lane);
        residual(to, nt, mt, sum, gains(a.ffn_norm, l));
      });
    }
    if (!meet()) return;
    // ---- gate / up projection
    row_totals<BT>(sh, 0, a.ss_in[1], nt_d, 4 * a.gu_ranges / BT);
    row_totals<BT>(sh, 1, a.ss_in[0], nt_d, 4 * a.gu_ranges / BT);
    share(a.nt_gu / 2, [&](int pair, int mt) {
      const int m = mt * 16 + col, row = 2 * pair * a.kt_d * 1024;
      const Rows x = Rows::tiled(a.xo + (size_t)l * a.x_stride, BT, mt, lane, B);
      v4f gs = ranges_of(weights(a.wgu), row, x, 0, a.kt_d, a.gu_ranges, lane);
      v4f us = ranges_of(weights(a.wgu), row + a.kt_d * 1024, x, 0, a.kt_d, a.gu_ranges, lane);
      const float sc = scale_of(sh.total[0][m], sh.total[1][m], true, a.inv_d, a.eps);
      gs = gs * sc;
      us = us * sc;
      uint2 pk;
      bool far = false;
      pk.x = pack_h16x2_track(silu_p(gs[0]) * us[0], silu_p(gs[1]) * us[1], far);
      pk.y = pack_h16x2_track(silu_p(gs[2]) * us[2], silu_p(gs[3]) * us[3], far);
      if (m < B) {
        st8(a.act + (size_t)l * a.act_stride + act_off(m, pair * 16 + rq, 16 * BT), pk);
        if (far) atomicOr(a.err_flag, kErrFp16Range);
      }
    });
    if (!meet()) return;
    // ---- down projection: sums per split of K
    const int ks = a.ks_down, per_split = (a.kt_F + ks - 1) / ks;
    share(nt_d * ks, [&](int i, int mt) {
      const int nt = i / ks, split = i - nt * ks, m = mt * 16 + col, kbeg = split * per_split;
      const v4f sum = ranges_of(weights(a.wdown), nt * a.kt_F * 1024, Rows::tiled(a.act + (size_t)l * a.act_stride, BT, mt, lane, B), kbeg,
                                min(a.kt_F, kbeg + per_split), a.dn_ranges, lane);
      if (m < B) st16(part, ((split * 16 * BT + m) * a.d + nt * 16 + rq) * 4, 0, __builtin_bit_cast(v4u, sum));
    });
    if (!meet()) return;
    // ---- sum of the splits, residual, operand of the next block
    row_totals<BT>(sh, 0, a.ss_in[1], nt_d, 4 * a.dn_ranges / BT);
    {
      const bool last = l + 1 == a.n_layers;
      const TileOut to(a, x_behind(a, l), 0, last);
      share(nt_d, [&](int nt, int mt) {
        const int at = (min(mt * 16 + col, B - 1) * a.d + nt * 16 + rq) * 4;
        v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < ks; ++s) sum = sum + ld16f(part, at, s * 64 * BT * a.d);
        residual(to, nt, mt, sum, last ? a.final_norm : gains(a.attn_norm, l + 1));
      });
    }
    if (!meet()) return;
  }
}

}  // namespace

void launch_some(const PersistArgs& a, int bt, hipStream_t st) {
  if (bt == 1) k_decode_layers_some<1><<<kPersistGrid, kThreads, 0, st>>>(a);
  else if (bt == 2) k_decode_layers_some<2><<<kPersistGrid, kThreads, 0, st>>>(a);
  else if (bt == 3) k_decode_layers_some<3><<<kPersistGrid, kThreads, 0, st>>>(a);
  else k_decode_layers_some<4><<<kPersistGrid, kThreads, 0, st>>>(a);
}

}  // namespace persist
}  // namespace bf16
}  // namespace mtmc
