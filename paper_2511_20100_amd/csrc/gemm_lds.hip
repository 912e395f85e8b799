// Large-batch GEMM of the prefill / scoring pass, staged through LDS.
//
// Workgroup tile: 32 NB output features x 32 MB tokens, full K.  Four wavefronts (one per SIMD and workgroup) in a
// 2 x 2 arrangement own NB x MB accumulator blocks of v_mfma_f32_16x16x32_f16 each.  The 16x16x32 shape and not
// 32x32x16: both are limited by power here, not by issue slots (a register-only loop on pseudo-random operands, the library's
// matrix probe, attains 1.68 PFLOP/s with 16x16x32 on the card where it read 1.56 with 32x32x16), because the smaller shape
// moves half as many accumulator bytes per product: on that card the gate/up GEMM of the 1.5 B scoring pass ran at 1.70 GHz
// with the matrix pipes occupied 0.69 of the cycles, and runs at 1.85 GHz and 0.68 now.  The sums are the same bit for bit.
//
// Both operands already sit in memory as 1 KiB MFMA operand blocks (frag.h), so staging is a plain copy: every k-step
// (32 columns of K) needs 2 NB weight blocks and 2 MB activation blocks, which the wavefronts fetch with LDS-direct
// 16-byte buffer loads (no registers involved; the block's address is scalar arithmetic alone) into a ring of ST
// buffers, ST - 1 steps ahead of the one being multiplied.  One workgroup barrier per step: it makes the step's
// blocks visible to every wavefront and at the same time guarantees that the buffer refilled next (read in the previous
// step) is no longer in use.
//
// What bounds it (256 x 256 tiles, 98 304 tokens, this file alone in a harness): without the copies the loop runs at 1.57
// PFLOP/s, with them at 1.38, and with the epilogue's HBM traffic at 1.25 (down projection).  In the scoring pass, profiled in
// turn on one card with the form of 32x32x16 and flat addresses before it: gate/up 4.65 -> 4.28 ms, O + down 2.70 -> 2.59,
// LM head 26.1 -> 24.2.  The fragment reads of a step are issued in its first half: spread over the whole step, their latency
// stood before the next step's first product (1.19 -> 1.28 PFLOP/s at 4096^2 x 8192).
#include <algorithm>

#include "bf16_kernels.h"
#include "device_utils.h"
#include "frag.h"

namespace mtmc {
namespace bf16 {

namespace {

constexpr int kCus = 256;   // CUs of the device; a multiple of the 8 XCDs
constexpr int kXcds = 8;

// A workgroup tile: 2 x 2 wavefronts of NB x MB blocks of 16 x 16, a ring of ST stages, PC workgroups per CU.
template <int NB_, int MB_, int ST_, int PC_>
struct Tile {
  static constexpr int NB = NB_, MB = MB_, ST = ST_, PC = PC_;
  static constexpr int TN = 2 * NB, TM = 2 * MB;               // 16-row tiles per workgroup tile side
  static constexpr int kStage = (TN + TM) * 1024;              // weight blocks, then activation blocks
  static constexpr int kLds = ST * kStage;
  static constexpr int LW = NB / 2, LX = MB / 2, NL = LW + LX; // blocks a wavefront copies per step
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// One 1 KiB operand block global -> LDS: lane l moves the 16 bytes at base + soff + voff (voff = 16 l) to dst + 16 l.
// The descriptor spans the address space: every offset is clamped to the operand by its caller.
__device__ __forceinline__ void copy_block_to_lds(const uint8_t* base, uint32_t voff, uint32_t soff, uint8_t* dst) {
#if defined(__HIP_DEVICE_COMPILE__)
  auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, -1, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)dst, 16, voff, soff, 0, 0);
#endif
}

// s_waitcnt on the vector-memory counter alone (the other counters left at their maxima).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// acc += A B with the accumulator pinned to the AGPR half of the register file (left to itself the register allocator
// spreads the accumulators over both halves and spills).  An accumulator is used again NB MB products later, far
// beyond the dependent-issue distance of the instruction.
__device__ __forceinline__ void mfma16_acc(v4f& acc, v8h a, v8h b) {
  asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b) : "memory");
}

// silu with the hardware exp2 / reciprocal (about 1e-6 relative error; the result is rounded to fp16 anyway):
// the evaluations would otherwise take a tenth of a block's time
__device__ __forceinline__ float silu_l(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
}

// Output blocks in bands of kBand token blocks x all feature blocks, features slow: workgroups that run together on
// an XCD share panels in its L2.  Every XCD owns one contiguous run of that order, equal to one block (with whole token
// blocks per XCD, 21 token blocks gave five XCDs three and three two), and its workgroups walk the run in turn.
constexpr int kBand = 4;
struct Block { int nb, mb; };
__device__ __forceinline__ Block block_at(int t, int nb_n, int nb_m) {
  const int band = t / (kBand * nb_n), r = t - band * (kBand * nb_n);
  const int height = min(kBand, nb_m - band * kBand);
  const int nb = r / height;
  return Block{nb, band * kBand + (r - nb * height)};
}
// first block of an XCD's run of `total`
__device__ __forceinline__ int run_of_xcd(int xcd, int total) { return (int)((long long)total * xcd / kXcds); }

enum { LEPI_STORE = 0, LEPI_ADD = 1, LEPI_SWIGLU = 2, LEPI_ROPE64 = 3, LEPI_ROPE128 = 4 };
struct RopeArgs : LargeArgs {
  RopeOut rope;
};

// Where this wavefront's share of a block's copies comes from: one base per operand (k-step 0), advanced by k-steps,
// and a 32-bit offset per piece (tile indices past the end are clamped: such blocks are multiplied but never stored).
template <class T>
struct TileSrc {
  const uint8_t* w;
  const uint8_t* x;
  uint32_t wo[T::LW], xo[T::LX];
};
template <class T>
__device__ __forceinline__ TileSrc<T> tile_src(const uint8_t* Wt, const uint8_t* Xt, int n_tiles, int m_tiles, int K,
                                               int nt_base, int mt_base, int uwave, int k0) {
  TileSrc<T> s;
  s.w = Wt + ((size_t)nt_base * K + k0) * 1024;
  s.x = Xt + ((size_t)k0 * m_tiles + mt_base) * 1024;
#pragma unroll
  for (int j = 0; j < T::LW; ++j)
    s.wo[j] = (uint32_t)(min(nt_base + T::LW * uwave + j, n_tiles - 1) - nt_base) * (uint32_t)K * 1024u;
#pragma unroll
  for (int j = 0; j < T::LX; ++j) s.xo[j] = (uint32_t)(min(mt_base + T::LX * uwave + j, m_tiles - 1) - mt_base) * 1024u;
  return s;
}

// The matrix pipeline of a workgroup over a SEQUENCE of output blocks.  `tile_at(nt_base, mt_base, k0)` names the
// next block and the k-step it starts at (false: no more), `epilogue(acc, nt_base, mt_base, k0)` consumes a finished one:
// acc = the NB x MB accumulator blocks of this wavefront (wn, wm).  The k-steps of consecutive blocks form one stream
// through the ring of ST LDS buffers: while the last steps of a block are multiplied the first steps of the next one are
// already being fetched, and its first fragments are read, so that a new block starts without refilling the pipeline
// and its copies run under the epilogue of the previous one.  A block is Ks k-steps of operands whose rows are
// K steps long; Ks >= ST and even.
template <class T, typename TileAt, typename Epilogue>
__device__ __forceinline__ void lds_gemm_stream(const uint8_t* Wt, const uint8_t* Xt, int n_tiles, int m_tiles, int K, int Ks,
                                                uint8_t* lds, int lane, int uwave, TileAt tile_at, Epilogue epilogue) {
  constexpr int NB = T::NB, MB = T::MB, ST = T::ST, NL = T::NL, SB = T::kStage;
  const int wn = uwave & 1, wm = uwave >> 1;
  int nt_base = 0, mt_base = 0, k0 = 0;
  if (!tile_at(nt_base, mt_base, k0)) return;  // whole workgroup
  const size_t xstep = (size_t)m_tiles * 1024;
  const uint32_t l16 = lane * 16;
  struct Frags { v8h w[NB], x[MB]; };
  auto read_frag = [&](Frags& f, const uint8_t* sb, int i) {
    if (i < MB) f.x[i] = *reinterpret_cast<const v8h*>(sb + (T::TN + MB * wm + i) * 1024);
    else f.w[i - MB] = *reinterpret_cast<const v8h*>(sb + (NB * wn + i - MB) * 1024);
  };
  auto issue_one = [&](const TileSrc<T>& s, int kk, uint8_t* sb, int j) {
    if (j < T::LW) copy_block_to_lds(s.w + (size_t)kk * 1024, l16, s.wo[j], sb + (T::LW * uwave + j) * 1024);
    else copy_block_to_lds(s.x + (size_t)kk * xstep, l16, s.xo[j - T::LW], sb + (T::TN + T::LX * uwave + j - T::LW) * 1024);
  };
  TileSrc<T> cur = tile_src<T>(Wt, Xt, n_tiles, m_tiles, K, nt_base, mt_base, uwave, k0);
  // ---- fill the ring with the first ST steps of the first block, read its first fragments
#pragma unroll
  for (int s = 0; s < ST; ++s)
#pragma unroll
    for (int j = 0; j < NL; ++j) issue_one(cur, s, lds + s * SB, j);
  Frags fa, fb;
  wait_vmcnt<(ST - 1) * NL>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < NB + MB; ++i) read_frag(fa, lds + l16, i);

  int off = 0;  // LDS offset of the buffer that the step being multiplied was read from
  for (;;) {
    int nt_next = 0, mt_next = 0, k0_next = 0;
    const bool has_next = tile_at(nt_next, mt_next, k0_next);
    const TileSrc<T> nxt = has_next ? tile_src<T>(Wt, Xt, n_tiles, m_tiles, K, nt_next, mt_next, uwave, k0_next) : cur;
    v4f acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = v4f{0.f, 0.f, 0.f, 0.f};
    asm volatile("s_nop 7" ::: "memory");  // accumulator writes settle before the first (inline-asm) MFMA reads them
    // Step kt multiplies the fragments already in registers; between its products go the LDS reads of the fragments
    // of the next step (first half) and the block fetches of step kt + ST into the buffer step kt was read from.
    auto step = [&](const Frags& fc, Frags& fn, int kt) {
      constexpr int VM = (ST - 2) * NL;
      // own LDS reads done (they all feed `fc`); blocks of the next step landed, those of later ones may fly
      __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4) | (0 << 8));
      __builtin_amdgcn_s_barrier();
      uint8_t* fbuf = lds + off;
      off = off + SB == ST * SB ? 0 : off + SB;
      const uint8_t* rb = lds + off + l16;
      // step kt + ST: of this block, else of the next one, else (nothing follows) a clamped copy nobody reads
      const int ka = kt + ST;
      const bool own = ka < Ks;
      const TileSrc<T>& src = own ? cur : nxt;
      const int kk = own ? ka : (has_next ? ka - Ks : Ks - 1);
      constexpr int NM = NB * MB, NR = NB + MB;
      int ir = 0, ic = 0;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        mfma16_acc(acc[i / MB][i % MB], fc.w[i / MB], fc.x[i % MB]);
        if (ir < NR && 2 * i * NR >= ir * NM) { read_frag(fn, rb, ir); ++ir; }
        if (ic < NL && i >= NM / 16 + ic * NM * 15 / 16 / NL) { issue_one(src, kk, fbuf, ic); ++ic; }
      }
    };
    for (int kt = 0; kt < Ks; kt += 2) {
      step(fa, fb, kt);
      step(fb, fa, kt + 1);
    }
    // the last MFMAs were issued from inline assembly: give them time to retire before their accumulators are read
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    epilogue(acc, nt_base, mt_base, k0);
    if (!has_next) break;
    // the epilogue's stores (and loads) share the counter with the copies: drain it so that the waits of the
    // next block count copies only (they have been flying under the epilogue)
    wait_vmcnt<0>();
    nt_base = nt_next;
    mt_base = mt_next;
    k0 = k0_next;
    cur = nxt;
  }
  wait_vmcnt<0>();  // the clamped copies past the last step still target this workgroup's LDS
}

// acc[nb][mb] of lane l holds token 16 mb + l % 16 and features 16 nb + 4 (l / 16) + 0..3 of the wavefront's part of
// the block.  fp32 forms: out[token][feature] = (ADD: +=) acc; the old values of the next 16 tokens are requested while
// the current ones are stored (where the CU hosts a second workgroup, that one's products fill the wait instead).
template <class T, bool ADD>
__device__ __forceinline__ void store_f32(v4f (&acc)[T::NB][T::MB], float* out, int ld, int M, int N, int nt0, int mt0, int lane) {
  constexpr int NB = T::NB, MB = T::MB;
  const int m0 = mt0 * 16 + (lane & 15), n0 = nt0 * 16 + (lane >> 4) * 4;
  const bool full = (mt0 + MB) * 16 <= M && (nt0 + NB) * 16 <= N;  // wavefront-uniform
  constexpr int PF = T::PC == 1 ? 2 : 1;
  v4f old[PF][NB];
  auto fetch = [&](int mb) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int m = m0 + mb * 16, n = n0 + nb * 16;
      old[mb % PF][nb] = v4f{0.f, 0.f, 0.f, 0.f};
      if (full || (m < M && n < N)) old[mb % PF][nb] = *reinterpret_cast<const v4f*>(out + (size_t)m * ld + n);
    }
  };
  if (ADD && PF == 2) fetch(0);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    if (ADD && mb + PF - 1 < MB) fetch(mb + PF - 1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      // one accumulator block at a time: it is taken from its registers here, not earlier (volatile statements keep
      // their order), which keeps the accumulators out of the VGPR half until they are needed
      asm volatile("" : "+a"(acc[nb][mb])::"memory");
      const int m = m0 + mb * 16, n = n0 + nb * 16;
      v4f v = acc[nb][mb];
      if (ADD) v = v + old[mb % PF][nb];
      if (full || (m < M && n < N)) *reinterpret_cast<v4f*>(out + (size_t)m * ld + n) = v;
    }
  }
}

// silu(gate) * up -> tiled fp16 operand; weight row tiles alternate gate / up.  The values are packed without a clamp and
// the packed pairs are tested with three integer instructions per pair for a magnitude of 0x7bff or more: an infinity, a NaN,
// or 65504, which magnitudes up to 65520 round to.  Only if one is found the block is packed again with the clamp, and the
// values themselves decide on the flag.
template <class T>
__device__ __forceinline__ void store_swiglu(v4f (&acc)[T::NB][T::MB], const LargeArgs& a, int nt0, int mt0, int lane) {
  constexpr int NB = T::NB, MB = T::MB;
  const int m0 = mt0 * 16 + (lane & 15), rq = (lane >> 4) * 4, Mpad = a.m_tiles * 16;
  uint32_t bad = 0;
  auto put = [&](int nb, int mb, bool clamp) {
    const int m = m0 + mb * 16, nt = nt0 + nb;
    if (m >= a.M || nt >= a.n_tiles) return;
    const v4f g = acc[nb][mb], u = acc[nb + 1][mb];
    float v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = silu_l(g[r]) * u[r];
    uint2 pk;
    if (clamp) {
      bool out_of_range = false;
      pk.x = pack_h16x2_track(v[0], v[1], out_of_range);
      pk.y = pack_h16x2_track(v[2], v[3], out_of_range);
      if (out_of_range) atomicOr(a.err_flag, kErrFp16Range);
    } else {
      pk.x = pack_h16x2_inrange(v[0], v[1]);
      pk.y = pack_h16x2_inrange(v[2], v[3]);
      bad |= (((pk.x & 0x7fff7fffu) + 0x04010401u) | ((pk.y & 0x7fff7fffu) + 0x04010401u)) & 0x80008000u;
    }
    *reinterpret_cast<uint2*>(a.out_bf16 + act_off(m, (nt >> 1) * 16 + rq, Mpad)) = pk;
  };
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; nb += 2) {
      asm volatile("" : "+a"(acc[nb][mb]), "+a"(acc[nb + 1][mb])::"memory");
      put(nb, mb, false);
    }
  if (__builtin_expect(__any(bad != 0), 0)) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; nb += 2) put(nb, mb, true);
  }
}

// Rotary form: the wavefront's 8 feature tiles are one head of 128 dims or two of 64, and a lane holds dims i .. i + 3 and
// i + hd / 2 .. of one token, so it rotates what it holds.  q goes to rows, k and v to the pages (layouts: attention_core.h).
// The fp32 projection is never written and read back: 16 of the 20 KiB that a token of the 1.5 B shape moved, and a launch.
// Projection and rotary kernel, before and now: 874 -> 645 us (98 304 tokens x 2048 features), 102 -> 89 (5439 x 3072, 64-dim
// heads), 46.6 -> 36.0 (4096 x 2048, in a pass without room for a split reduction: with it the projection of so few blocks is
// split, and keeps the separate kernels).
template <class T, int HD>
__device__ __forceinline__ void store_rope(v4f (&acc)[T::NB][T::MB], const RopeArgs& a, int nt0, int mt0, int lane) {
  constexpr int MB = T::MB, BPH = HD / 16, HB = BPH / 2;
  static_assert(T::NB == 8, "a wavefront holds whole heads");
  const RopeOut& r = a.rope;
  const int col = lane & 15, rq = (lane >> 4) * 4;
  h16_t* const kv = (h16_t*)r.pool.base;
  bool out_of_range = false;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int t = (mt0 + mb) * 16 + col;
    const bool live = t < a.M;
    const int seq = min(t, a.M - 1) / r.S, pos = r.pos_base + min(t, a.M - 1) - seq * r.S;
    const float* cs = r.cos + (size_t)pos * (HD / 2) + rq;
    const float* sn = r.sin + (size_t)pos * (HD / 2) + rq;
#pragma unroll
    for (int hs = 0; hs < 8 / BPH; ++hs) {
      const int head = nt0 / BPH + hs;  // wavefront-uniform
#pragma unroll
      for (int nb = 0; nb < BPH; ++nb) asm volatile("" : "+a"(acc[hs * BPH + nb][mb])::"memory");
      if (!live || head >= r.Hq + 2 * r.Hkv) continue;
      if (head < r.Hq + r.Hkv) {
        h16_t *lo, *hi;  // where dims rq .. + 3 of the two halves go; + 16 nb dims: step elements
        int step;
        if (head < r.Hq) {
          lo = r.q + ((size_t)t * r.Hq + head) * HD + rq;
          hi = lo + HD / 2;
          step = 16;
        } else {
          const int page = r.pool.page_table[(size_t)seq * r.row_stride * r.pool.max_pages + pos / kPageTokens];
          lo = kv + ((((size_t)r.layer * 2) * r.pool.n_pages + page) * r.Hkv + head - r.Hq) * (kPageTokens * HD) +
               (rq >> 3) * 128 + (pos % kPageTokens) * 8 + (rq & 7);
          hi = lo + HD / 16 * 128;
          step = 256;
        }
#pragma unroll
        for (int nb = 0; nb < HB; ++nb) {
          const v4f x = acc[hs * BPH + nb][mb], y = acc[hs * BPH + nb + HB][mb];
          const v4f c = *reinterpret_cast<const v4f*>(cs + 16 * nb), s = *reinterpret_cast<const v4f*>(sn + 16 * nb);
          const v4f rx = x * c - y * s, ry = y * c + x * s;
          uint2 p, q;
          p.x = pack_h16x2_track(rx[0], rx[1], out_of_range); p.y = pack_h16x2_track(rx[2], rx[3], out_of_range);
          q.x = pack_h16x2_track(ry[0], ry[1], out_of_range); q.y = pack_h16x2_track(ry[2], ry[3], out_of_range);
          *reinterpret_cast<uint2*>(lo + nb * step) = p;
          *reinterpret_cast<uint2*>(hi + nb * step) = q;
        }
      } else {
        const int g = head - r.Hq - r.Hkv;
        const int page = r.pool.page_table[(size_t)seq * r.row_stride * r.pool.max_pages + pos / kPageTokens];
        h16_t* vp = kv + ((((size_t)r.layer * 2 + 1) * r.pool.n_pages + page) * r.Hkv + g) * (kPageTokens * HD) +
                    rq * kPageTokens + pos % kPageTokens;
#pragma unroll
        for (int nb = 0; nb < BPH; ++nb) {
          const v4f v = acc[hs * BPH + nb][mb];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            out_of_range |= !fits_h16(v[e]);
            vp[(16 * nb + e) * kPageTokens] = f32_to_h16(v[e]);
          }
        }
      }
    }
  }
  if (out_of_range) atomicOr(a.err_flag, kErrFp16Range);
}

// Blocks that hold tokens: rows packed on the device (d_rows) fill only part of the capacity the launch is sized for.
// Whatever the block's height, all rows up to the next multiple of 256 are computed (from cleared inputs): a launch with
// taller blocks reads them next.
template <class T>
__device__ __forceinline__ int row_blocks(int m_tiles, const int* d_rows) {
  const int nb_m = (m_tiles + T::TM - 1) / T::TM;
  return d_rows ? min(nb_m, (((*d_rows + 255) & ~255) + T::TM * 16 - 1) / (T::TM * 16)) : nb_m;
}

template <class T, int EPI, class Args>
__global__ __launch_bounds__(256, T::PC) void k_gemm_lds(Args a) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int lane = threadIdx.x & 63, uwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb_n = (a.n_tiles + T::TN - 1) / T::TN, nb_m = row_blocks<T>(a.m_tiles, a.d_rows);
  // persistent workgroup: gridDim.x is a multiple of 8, so this workgroup and the gridDim.x / 8 - 1 others of its
  // XCD share out the XCD's run of blocks
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3, end = run_of_xcd(xcd + 1, nb_n * nb_m);
  int t = run_of_xcd(xcd, nb_n * nb_m) + (int)(blockIdx.x >> 3) - stride;
  auto tile_at = [&](int& nt_base, int& mt_base, int&) {
    t += stride;
    if (t >= end) return false;
    const Block blk = block_at(t, nb_n, nb_m);
    nt_base = blk.nb * T::TN;
    mt_base = blk.mb * T::TM;
    return true;
  };
  auto epilogue = [&](v4f (&acc)[T::NB][T::MB], int nt_base, int mt_base, int) {
    const int nt0 = nt_base + T::NB * (uwave & 1), mt0 = mt_base + T::MB * (uwave >> 1);
    if constexpr (EPI == LEPI_ROPE64) store_rope<T, 64>(acc, a, nt0, mt0, lane);
    else if constexpr (EPI == LEPI_ROPE128) store_rope<T, 128>(acc, a, nt0, mt0, lane);
    else if constexpr (EPI == LEPI_SWIGLU) store_swiglu<T>(acc, a, nt0, mt0, lane);
    else store_f32<T, EPI == LEPI_ADD>(acc, a.out_f32, a.ld_out, a.M, a.N, nt0, mt0, lane);
  };
  lds_gemm_stream<T>(reinterpret_cast<const uint8_t*>(a.Wt), reinterpret_cast<const uint8_t*>(a.Xt), a.n_tiles, a.m_tiles,
                     a.k_tiles, a.k_tiles, lds, lane, uwave, tile_at, epilogue);
}

// Split-K form for outputs of few blocks and a long reduction (the O and down projections, and the QKV projection,
// of a prompt or a few): a work item is one output block over one of a.k_split equal ranges of k-steps, the items of a
// block are neighbours in an XCD's walk, and every item stores its sum as fp32 into its own slice of a.part
// ([k_split][M][N]); k_splitk_reduce, or the consumer of the output, then adds the slices in order, so the result does
// not depend on which workgroup ran when.
template <class T>
__global__ __launch_bounds__(256, T::PC) void k_gemm_lds_split(LargeArgs a) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  const int lane = threadIdx.x & 63, uwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb_n = (a.n_tiles + T::TN - 1) / T::TN, nb_m = row_blocks<T>(a.m_tiles, a.d_rows);
  const int S = a.k_split, Ks = a.k_tiles / S;
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3, end = run_of_xcd(xcd + 1, nb_n * nb_m * S);
  int t = run_of_xcd(xcd, nb_n * nb_m * S) + (int)(blockIdx.x >> 3) - stride;
  auto tile_at = [&](int& nt_base, int& mt_base, int& k0) {
    t += stride;
    if (t >= end) return false;
    const Block blk = block_at(t / S, nb_n, nb_m);
    nt_base = blk.nb * T::TN;
    mt_base = blk.mb * T::TM;
    k0 = (t % S) * Ks;
    return true;
  };
  auto epilogue = [&](v4f (&acc)[T::NB][T::MB], int nt_base, int mt_base, int k0) {
    store_f32<T, false>(acc, a.part + (size_t)(k0 / Ks) * a.M * a.N, a.N, a.M, a.N, nt_base + T::NB * (uwave & 1),
                        mt_base + T::MB * (uwave >> 1), lane);
  };
  lds_gemm_stream<T>(reinterpret_cast<const uint8_t*>(a.Wt), reinterpret_cast<const uint8_t*>(a.Xt), a.n_tiles, a.m_tiles,
                     a.k_tiles, Ks, lds, lane, uwave, tile_at, epilogue);
}

// out (+)= part[0] + part[1] + ... in that order; four features per thread
__global__ __launch_bounds__(256) void k_splitk_reduce(float* out, int ld_out, const float* part, int S, int M, int N,
                                                       int accumulate, const int* d_rows) {
  const int n4 = N >> 2;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)M * n4) return;
  const int m = (int)(i / n4), n = (int)(i - (size_t)m * n4) * 4;
  if (d_rows && m >= *d_rows) return;
  float* o = out + (size_t)m * ld_out + n;
  const v4f acc = accumulate ? *reinterpret_cast<const v4f*>(o) : v4f{0.f, 0.f, 0.f, 0.f};
  const float* p = part + (size_t)m * N + n;
  *reinterpret_cast<v4f*>(o) = add_slices(acc, S, [&](int s) { return *reinterpret_cast<const v4f*>(p + (size_t)s * M * N); });
}

// Scoring LM head on the same engine: a work item is one block of rows and one slice of the vocabulary (`bps` blocks of
// 256 entries); the logits are computed block by block and folded into running per-row results (log-sum-exp, two
// largest logits, logit of the target token), never stored.  Persistent: the items' blocks form one stream.
// A block's 128 entries of a wavefront are reduced over the four lanes that share a row before they meet the running
// result, so a row's state sits in ONE lane (row 16 mb + l % 16: the lanes l / 16 = mb % 4) and takes registers the
// matrix loop does not need.
template <class T, bool TOP>
__global__ __launch_bounds__(256, T::PC) void k_lmhead_lds(ScoreHeadArgs a, int bps) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  constexpr int NB = T::NB, MB = T::MB, H = MB / 4;
  const int lane = threadIdx.x & 63, uwave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = uwave & 1, wm = uwave >> 1, col = lane & 15, lg = lane >> 4;
  const int nb_n = (a.n_tiles + T::TN - 1) / T::TN, nb_m = row_blocks<T>(a.m_tiles, a.d_rows);
  const int slices = (nb_n + bps - 1) / bps;
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3, end = run_of_xcd(xcd + 1, slices * nb_m);
  int t = run_of_xcd(xcd, slices * nb_m) + (int)(blockIdx.x >> 3) - stride;
  int b_next = 0, b_end = 0, mt_item = 0;  // blocks of the item that tile_at is in
  auto tile_at = [&](int& nt_base, int& mt_base, int&) {
    if (b_next == b_end) {
      t += stride;
      if (t >= end) return false;
      const Block blk = block_at(t, slices, nb_m);
      b_next = blk.nb * bps;
      b_end = min(b_next + bps, nb_n);
      mt_item = blk.mb * T::TM;
    }
    nt_base = b_next++ * T::TN;
    mt_base = mt_item;
    return true;
  };
  Lse lse[H];
  Top2 top[H];
  float zt[H];
  int target[H];
  auto epilogue = [&](v4f (&acc)[NB][MB], int nt_base, int mt_base, int) {
    const int blk = nt_base / T::TN, slice = blk / bps;
    const int nt0 = nt_base + NB * wn, mt0 = mt_base + MB * wm;
    if (blk == slice * bps) {  // a new item
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int m = (mt0 + 4 * h + lg) * 16 + col;
        lse[h] = lse_empty();
        top[h] = top2_empty();
        zt[h] = -INFINITY;
        target[h] = m < a.M ? a.targets[m] : -1;
      }
    }
    const bool full = nt0 + NB <= a.n_tiles;  // all 128 entries exist (wavefront-uniform)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int h = mb >> 2, owner = (mb & 3) * 16 + col;
      float z[NB * 4];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        asm volatile("" : "+a"(acc[nb][mb])::"memory");
#pragma unroll
        for (int r = 0; r < 4; ++r) z[4 * nb + r] = (full || nt0 + nb < a.n_tiles) ? acc[nb][mb][r] : -INFINITY;
      }
      float bm = z[0];
#pragma unroll
      for (int j = 1; j < NB * 4; ++j) bm = fmaxf(bm, z[j]);
      bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
      bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
      // no entry exists (or none compares): nothing to add.  The terms are exp2(z log2(e) - mk) with mk = bm log2(e) rounded;
      // lo is what that rounding lost, a common factor 2^lo of the sum (left in, it stood in the log-probability)
      const float ref = bm > -INFINITY ? bm : 0.f, mk = ref * kLog2e, lo = fmaf(ref, kLog2e, -mk);
      float sum = 0.f;
#pragma unroll
      for (int j = 0; j < NB * 4; ++j) sum += __builtin_amdgcn_exp2f(fmaf(z[j], kLog2e, -mk));
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      sum *= __builtin_amdgcn_exp2f(-lo);
      const int d = __shfl(target[h], owner, 64) - nt0 * 16;  // the target's index among the wavefront's entries
      float hit = -INFINITY;
      const bool here = d >= 0 && d < NB * 16 && ((d >> 2) & 3) == lg;
      if (__any(here)) {
        const int idx = (d >> 4) * 4 + (d & 3);
#pragma unroll
        for (int j = 0; j < NB * 4; ++j)
          if (here && j == idx) hit = z[j];
        hit = fmaxf(hit, __shfl_xor(hit, 16, 64));
        hit = fmaxf(hit, __shfl_xor(hit, 32, 64));
      }
      const bool own = lg == (mb & 3);
      Top2 t2 = top2_empty();
      if (TOP) {
        // two largest of the block and the lowest index of the largest: three instructions per entry, then the indices
        float v1 = -INFINITY, v2 = -INFINITY;
#pragma unroll
        for (int j = 0; j < NB * 4; ++j) {
          v2 = fmaxf(v2, fminf(v1, z[j]));
          v1 = fmaxf(v1, z[j]);
        }
        int i1 = 0x7fffffff;
#pragma unroll
        for (int j = NB * 4 - 1; j >= 0; --j)
          if (z[j] == v1) i1 = (nt0 + (j >> 2)) * 16 + 4 * lg + (j & 3);
        t2 = Top2{v1, i1, v2};
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1)
          t2 = top2_merge(t2, Top2{__shfl_xor(t2.v1, o, 64), __shfl_xor(t2.i1, o, 64), __shfl_xor(t2.v2, o, 64)});
      }
      if (own) {
        const float m_new = fmaxf(lse[h].m, bm);
        if (m_new > -INFINITY) {
          lse[h].s = lse[h].s * __builtin_amdgcn_exp2f((lse[h].m - m_new) * kLog2e) +
                     (bm > -INFINITY ? sum * __builtin_amdgcn_exp2f((bm - m_new) * kLog2e) : 0.f);
          lse[h].m = m_new;
        }
        zt[h] = fmaxf(zt[h], hit);
        if (TOP) top[h] = top2_merge(top[h], t2);
      }
    }
    if (blk + 1 == min(slice * bps + bps, nb_n)) {  // the item's last block
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int m = (mt0 + 4 * h + lg) * 16 + col;
        if (m < a.M) {
          ScorePartial* p = reinterpret_cast<ScorePartial*>(a.part) + ((size_t)(slice * 2 + wn)) * a.M + m;
          p->m = lse[h].m; p->s = lse[h].s; p->v1 = top[h].v1; p->i1 = top[h].i1; p->v2 = top[h].v2; p->zt = zt[h];
        }
      }
    }
  };
  lds_gemm_stream<T>(reinterpret_cast<const uint8_t*>(a.Wt), reinterpret_cast<const uint8_t*>(a.Xt), a.n_tiles, a.m_tiles,
                     a.k_tiles, a.k_tiles, lds, lane, uwave, tile_at, epilogue);
}

// Sampling LM head of 65 .. 128 rows on the same engine: the workgroups of the launch walk the vocabulary in blocks of 128
// entries, and every lane folds its entries of 4 rows into a running (log-sum-exp, Gumbel arg-max) that leaves the kernel once,
// as two partial results per row and workgroup.  The logits are those of k_gemm_rows128 (one accumulator over K in ascending
// order) bit for bit.  That form starts a workgroup, with the row scales (100 KiB of sums of squares) and an empty pipeline, for
// every 128 entries: 128 rows x 151 936 entries x 1536 139 us there and 105 here (76 at the rate of a large read), 152 064 x 3584
// 245 and 222 (176).
using SampleTile = Tile<4, 4, 4, 2>;
__global__ __launch_bounds__(256, SampleTile::PC) void k_lmhead_sample_lds(DecGemmArgs a) {
  using T = SampleTile;
  constexpr int NB = T::NB, MB = T::MB, NT = 256, ROWS = T::TM * 16;
  static_assert(ROWS == 128, "the rows of a launch are one block of tokens");
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  __shared__ float s_scale[ROWS];
  __shared__ int s_row[ROWS], s_step[ROWS];
  __shared__ float s_part[2][NT];
  const int tid = threadIdx.x, lane = tid & 63, uwave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = uwave & 1, wm = uwave >> 1, col = lane & 15, rq = (lane >> 4) * 4;
  const int Mpad = a.m_tiles * 16;  // 80 .. 128
  const SampleCtl ctl = *a.ctl;

  // ---- row scales r_new / r_old: thread t sums the tiles part, part + P, ... of row t % Mpad, the P sums are added in index
  // order (the operations and their order are those of the other forms: the same bits)
  {
    const int P = NT / Mpad, m = tid % Mpad, part = tid / Mpad;
    const bool two = a.ss_cur && a.ss_old != a.ss_cur;
    float sa = 0.f, sb = 0.f;
    if (two && part < P) {
      constexpr int BT = 16;
      for (int t0 = part; t0 < a.ss_tiles; t0 += BT * P) {  // batches of independent loads
        float fa[BT], fb[BT];
#pragma unroll
        for (int u = 0; u < BT; ++u) {
          const int t = t0 + u * P;
          fa[u] = t < a.ss_tiles ? a.ss_cur[(size_t)t * Mpad + m] : 0.f;
          fb[u] = t < a.ss_tiles ? a.ss_old[(size_t)t * Mpad + m] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < BT; ++u) {
          sa += fa[u];
          sb += fb[u];
        }
      }
    }
    s_part[0][tid] = sa;
    s_part[1][tid] = sb;
    __syncthreads();
    if (tid < ROWS) {
      float sc = 1.f;
      if (tid < Mpad && two) {
        float ta = 0.f, tb = 0.f;
        for (int q = 0; q < P; ++q) {
          ta += s_part[0][q * Mpad + tid];
          tb += s_part[1][q * Mpad + tid];
        }
        sc = 1.0f / sqrtf(ta * a.inv_d + a.eps);
        sc *= sqrtf(tb * a.inv_d + a.eps);
      }
      s_scale[tid] = sc;
      // the random numbers of a row follow the row and its own step (an empty slot draws row 0's: unused)
      s_row[tid] = (ctl.slot_row && tid < a.M) ? max(ctl.slot_row[tid], 0) : tid;
      s_step[tid] = *a.d_step - ((ctl.row_step0 && tid < a.M) ? ctl.row_step0[tid] : 0);
    }
    __syncthreads();
  }

  const int nb_n = (a.n_tiles + T::TN - 1) / T::TN;
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3, end = run_of_xcd(xcd + 1, nb_n);
  int t = run_of_xcd(xcd, nb_n) + (int)(blockIdx.x >> 3) - stride;
  auto tile_at = [&](int& nt_base, int& mt_base, int&) {
    t += stride;
    if (t >= end) return false;
    nt_base = t * T::TN;
    mt_base = 0;
    return true;
  };
  Lse2 lse2[MB];
  float by[MB], bz[MB];
  int bi[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    lse2[mb] = lse2_empty();
    by[mb] = -INFINITY;
    bz[mb] = 0.f;
    bi[mb] = 0x7fffffff;
  }
  auto epilogue = [&](v4f (&acc)[NB][MB], int nt_base, int, int) {
    const int nt0 = nt_base + NB * wn;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int m = (MB * wm + mb) * 16 + col;
      const float sc = s_scale[m];
      const uint32_t row = (uint32_t)s_row[m], step = (uint32_t)s_step[m];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        asm volatile("" : "+a"(acc[nb][mb])::"memory");
        if (nt0 + nb >= a.n_tiles) continue;
        const int v0 = (nt0 + nb) * 16 + rq;  // multiple of 4: one generator block per 4 entries
        uint4 rb = make_uint4(0, 0, 0, 0);
        if (!ctl.greedy) rb = philox4x32_10(make_uint4((uint32_t)(v0 >> 2), step, ctl.seq_offset + row, 0u), ctl.key0, ctl.key1);
        const uint32_t rr[4] = {rb.x, rb.y, rb.z, rb.w};
        float zt[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float z = acc[nb][mb][r] * sc;
          zt[r] = ctl.greedy ? z : z * ctl.inv_temp;
        }
        lse2_push4(lse2[mb], zt[0], zt[1], zt[2], zt[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float y = ctl.greedy ? zt[r] : zt[r] + gumbel_from_bits(rr[r]);
          if (y > by[mb]) { by[mb] = y; bi[mb] = v0 + r; bz[mb] = zt[r]; }  // ascending index: the first maximum wins
        }
      }
    }
  };
  lds_gemm_stream<T>(reinterpret_cast<const uint8_t*>(a.Wt), reinterpret_cast<const uint8_t*>(a.Xt), a.n_tiles, a.m_tiles,
                     a.k_tiles, a.k_tiles, lds, lane, uwave, tile_at, epilogue);
  // ---- a row's four column groups (lane / 16); a workgroup without a block leaves empty results
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = (MB * wm + mb) * 16 + col;
    Lse lse = lse_of(lse2[mb]);
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const Lse ol = {__shfl_xor(lse.m, o, 64), __shfl_xor(lse.s, o, 64)};
      const float oy = __shfl_xor(by[mb], o, 64), oz = __shfl_xor(bz[mb], o, 64);
      const int oi = __shfl_xor(bi[mb], o, 64);
      lse = lse_merge(lse, ol);
      if (oy > by[mb] || (oy == by[mb] && oi < bi[mb])) { by[mb] = oy; bi[mb] = oi; bz[mb] = oz; }
    }
    if (lane < 16 && m < a.M) {
      DecSamplePartial* p = reinterpret_cast<DecSamplePartial*>(a.out_f32) + (size_t)m * (2 * gridDim.x) + 2 * blockIdx.x + wn;
      p->m = lse.m; p->s = lse.s; p->y = by[mb]; p->idx = bi[mb]; p->zt = bz[mb];
    }
  }
}

// The runtime's limit on dynamic LDS is raised once per kernel.
template <class T, typename Kernel>
void allow_lds(Kernel* k) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, T::kLds);
}
// workgroups of a launch of `items` work items: one round of the CUs at most, a multiple of the XCDs
template <class T>
int grid_of(size_t items) { return (int)std::min<size_t>((items + kXcds - 1) / kXcds * kXcds, (size_t)kCus * T::PC); }
template <class T>
size_t blocks_of(const LargeArgs& a) {
  return (size_t)((a.n_tiles + T::TN - 1) / T::TN) * ((a.m_tiles + T::TM - 1) / T::TM);
}

template <class T, int EPI, class Args>
void launch_tile(const Args& a, hipStream_t st) {
  static const bool configured = (allow_lds<T>(&k_gemm_lds<T, EPI, Args>), true);
  (void)configured;
  k_gemm_lds<T, EPI, Args><<<grid_of<T>(blocks_of<T>(a)), 256, T::kLds, st>>>(a);
}
template <class T>
void launch_split(const LargeArgs& a, hipStream_t st) {
  static const bool configured = (allow_lds<T>(&k_gemm_lds_split<T>), true);
  (void)configured;
  k_gemm_lds_split<T><<<grid_of<T>(blocks_of<T>(a) * a.k_split), 256, T::kLds, st>>>(a);
}
template <class T>
void launch(const LargeArgs& a, int epi, hipStream_t st) {
  if (a.k_split > 1) launch_split<T>(a, st);
  else if (epi == LEPI_STORE) launch_tile<T, LEPI_STORE>(a, st);
  else if (epi == LEPI_ADD) launch_tile<T, LEPI_ADD>(a, st);
  else launch_tile<T, LEPI_SWIGLU>(a, st);
}

// The tiles, features x tokens per workgroup, and what they were measured to take: microseconds per k-step for a
// workgroup that has its CU to itself, for the two of a CU that hosts two, and per block outside the k-steps (SwiGLU
// form; the fp32 forms move four times the bytes and take 1.7 times as long).  Sums do not depend on the tile.
struct TileCost {
  int features, tokens, per_cu;
  double alone, pair, block;
  void (*run)(const LargeArgs&, int, hipStream_t);
};
const TileCost kTiles[] = {
    {256, 256, 1, 0.74, 0.0, 9.0, &launch<Tile<8, 8, 4, 1>>},   // fewest bytes per product: the large passes
    {192, 256, 1, 0.60, 0.0, 7.0, &launch<Tile<6, 8, 4, 1>>},
    {256, 128, 2, 0.42, 0.76, 5.0, &launch<Tile<8, 4, 3, 2>>},
    {192, 128, 2, 0.37, 0.62, 4.0, &launch<Tile<6, 4, 4, 2>>},
    {128, 128, 2, 0.25, 0.44, 3.0, &launch<Tile<4, 4, 4, 2>>},
    {128, 64, 2, 0.16, 0.30, 1.5, &launch<Tile<4, 2, 4, 2>>},   // a few dozen rows
};

// What a launch takes, by its busiest CU.  Measured against it (this file alone in a harness): 4096 x 1536 x 8960 (features and tokens swapped) 183 us
// in 96 blocks of 256 x 256, 104 us in 256 of 192 x 128; 512 tokens x 17 920 features 38.6 and 32.1 us; 800 tokens 73.6 and
// 44.0 us; 98 304 tokens 4.46 ms in 256 x 256, 4.55-5.2 ms in the others.
double cost_of(const TileCost& t, int features, int tokens, int k_steps, int splits, bool fp32) {
  const long long items = (long long)((features + t.features - 1) / t.features) * ((tokens + t.tokens - 1) / t.tokens) * splits;
  const long long per_cu = (items + kCus - 1) / kCus;
  const double steps = (double)k_steps / splits, out = t.block * (fp32 ? 1.7 : 1.0);
  if (t.per_cu == 1) return per_cu * (steps * t.alone + out);
  return (per_cu / 2) * (steps * t.pair + 2 * out) + (per_cu % 2) * (steps * t.alone + out);
}
const TileCost& best_tile(int features, int tokens, int k_steps, int splits, bool fp32, double* cost) {
  const TileCost* best = nullptr;
  for (const TileCost& t : kTiles) {
    const double c = cost_of(t, features, tokens, k_steps, splits, fp32);
    if (!best || c < *cost) {
      best = &t;
      *cost = c;
    }
  }
  return *best;
}

// rows a launch is expected to hold: where they are packed on the device the launch knows its capacity alone (candidate
// actions of 1 .. A tokens fill about half of it)
int expected_rows(const LargeArgs& a) { return a.d_rows ? (a.M + 1) / 2 : a.M; }

}  // namespace

// Vocabulary blocks per slice of the scoring LM head for R rows: slices as long as they can be while a launch still
// has several items per CU to even out (3332 rows x 128 256 entries: 882 items of 8 blocks on 256 CUs are four rounds where
// 3.4 would do; 127 rows: 75 workgroups in all).
int lmhead_lds_slice(int R) { return R <= 1024 ? 1 : R <= 4096 ? 2 : R <= 16384 ? 4 : 8; }
int lmhead_lds_parts(int n_tiles, int R) {
  const int blocks = (n_tiles + 15) / 16, bps = lmhead_lds_slice(R);
  return 2 * ((blocks + bps - 1) / bps);
}

template <class T, bool TOP>
static void launch_lmhead(const ScoreHeadArgs& a, hipStream_t st) {
  static const bool configured = (allow_lds<T>(&k_lmhead_lds<T, TOP>), true);
  (void)configured;
  const int bps = lmhead_lds_slice(a.M);
  const size_t items = (size_t)(((a.n_tiles + T::TN - 1) / T::TN + bps - 1) / bps) * ((a.m_tiles + T::TM - 1) / T::TM);
  k_lmhead_lds<T, TOP><<<grid_of<T>(items), 256, T::kLds, st>>>(a, bps);
}
void lmhead_score_lds(const ScoreHeadArgs& a, hipStream_t st) {
  // blocks of 128 rows where blocks of 256 would be padding for more than the 8 % that the smaller block costs
  const bool narrow = 1.08 * ((a.m_tiles + 7) / 8) < 2 * ((a.m_tiles + 15) / 16);
  if (narrow) a.want_top ? launch_lmhead<Tile<8, 4, 3, 2>, true>(a, st) : launch_lmhead<Tile<8, 4, 3, 2>, false>(a, st);
  else a.want_top ? launch_lmhead<Tile<8, 8, 4, 1>, true>(a, st) : launch_lmhead<Tile<8, 8, 4, 1>, false>(a, st);
}

// The most splits, up to kMaxSlices and to one round of blocks of 256 x 256, that leave every range even and at least 8 k-steps
// long.  Not by the tile that the launch chooses: the order of the sums then follows from the sizes alone.
int gemm_lds_splits(const LargeArgs& a, size_t part_floats) {
  const int blocks = (a.n_tiles + 15) / 16 * ((a.m_tiles + 15) / 16);  // of 256 x 256
  if (blocks > kCus / 2 || a.N % 4 != 0) return 0;
  for (int s = std::min(kMaxSlices, kCus / blocks); s >= 2; --s)
    if (a.k_tiles % s == 0 && (a.k_tiles / s) % 2 == 0 && a.k_tiles / s >= 8 && (size_t)s * a.M * a.N <= part_floats) return s;
  return 0;
}
int gemm_lds_split(const LargeArgs& a0, bool accumulate, float* part, size_t part_floats, bool leave_parts, hipStream_t st) {
  const int S = part ? gemm_lds_splits(a0, part_floats) : 0;
  if (!S) return 0;
  LargeArgs a = a0;
  a.k_split = S;
  a.part = part;
  double cost = 0.0;
  best_tile(a.N, expected_rows(a), a.k_tiles, S, true, &cost).run(a, LEPI_STORE, st);
  if (leave_parts) return S;
  const size_t quads = (size_t)a.M * (a.N / 4);
  k_splitk_reduce<<<(unsigned)((quads + 255) / 256), 256, 0, st>>>(a.out_f32, a.ld_out, part, S, a.M, a.N,
                                                                  accumulate ? 1 : 0, a.d_rows);
  return S;
}

// A wavefront has to hold whole heads: the blocks of 256 features, of which the measured costs choose.  From 1024 tokens (the
// caller); below, the separate rotary kernel adds up the slices of a split reduction, and a launch has too few such blocks.
// Not where another block is so much better that the separate kernel (7 us, and 6 bytes per value at 4.8 TB/s) costs less than
// the difference: 4608 features x 2048 tokens x 3584 take one round of 98 us in blocks of 256 x 256 and one of 79
// in blocks of 192 x 256 (a layer of a scoring pass: 7 us longer with the epilogue, 12 us shorter at 3072 tokens).
bool gemm_lds_rope(const LargeArgs& a0, const RopeOut& r, hipStream_t st) {
  const RopeArgs a{a0, r};
  const int features = a.n_tiles * 16;
  const double c256 = cost_of(kTiles[0], features, a.M, a.k_tiles, 1, true), c128 = cost_of(kTiles[2], features, a.M, a.k_tiles, 1, true);
  double best = 0.0;
  best_tile(features, a.M, a.k_tiles, 1, true, &best);
  if (std::min(c256, c128) > best + 7.0 + 6.0 * features * a.M / 4.8e6) return false;
  const bool wide = c256 <= c128;
  if (a.rope.pool.head_dim == 64) {
    if (wide) launch_tile<Tile<8, 8, 4, 1>, LEPI_ROPE64>(a, st);
    else launch_tile<Tile<8, 4, 3, 2>, LEPI_ROPE64>(a, st);
  } else {
    if (wide) launch_tile<Tile<8, 8, 4, 1>, LEPI_ROPE128>(a, st);
    else launch_tile<Tile<8, 4, 3, 2>, LEPI_ROPE128>(a, st);
  }
  return true;
}

static int sample_lds_grid(int n_tiles) { return grid_of<SampleTile>((size_t)(n_tiles + SampleTile::TN - 1) / SampleTile::TN); }
// Where a CU gets at least one block of 128 entries; the ring takes an even number of k-steps, no fewer than its stages.
int lmhead_sample_lds_groups(int n_tiles, int k_tiles, int m_tiles) {
  if (m_tiles <= 4 || m_tiles > SampleTile::TM || n_tiles < kCus * SampleTile::TN || k_tiles < SampleTile::ST || k_tiles % 2 != 0)
    return 0;
  return 2 * sample_lds_grid(n_tiles);
}
bool lmhead_sample_lds(const DecGemmArgs& a, hipStream_t st) {
  if (!lmhead_sample_lds_groups(a.n_tiles, a.k_tiles, a.m_tiles)) return false;
  static const bool configured = (allow_lds<SampleTile>(&k_lmhead_sample_lds), true);
  (void)configured;
  k_lmhead_sample_lds<<<sample_lds_grid(a.n_tiles), 256, SampleTile::kLds, st>>>(a);
  return true;
}

void gemm_lds(const LargeArgs& a, int epi, hipStream_t st) {
  double cost = 0.0;
  best_tile(a.n_tiles * 16, expected_rows(a), a.k_tiles, 1, epi != LEPI_SWIGLU, &cost).run(a, epi, st);
}

}  // namespace bf16
}  // namespace mtmc
