// Measurement probes: what this GPU sustains for a plain streaming read and for back-to-back matrix
// instructions on registers.  The benchmark reports both beside the published peaks.
#include "common.h"
#include "kernels.h"

namespace mtmc {

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t pv4u;
typedef __attribute__((ext_vector_type(8))) _Float16 pv8h;
typedef __attribute__((ext_vector_type(4))) float pv4f;

// Every workgroup reads its contiguous share of the range, eight independent 16-byte loads per lane in flight.
__global__ __launch_bounds__(512) void k_read_probe(const pv4u* __restrict__ src, size_t vec_per_wg, uint32_t* sink) {
  const pv4u* p = src + (size_t)blockIdx.x * vec_per_wg;
  pv4u acc = {0u, 0u, 0u, 0u};
  size_t i = threadIdx.x;
  for (; i + 7 * 512 < vec_per_wg; i += 8 * 512) {
    pv4u v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[i + (size_t)u * 512];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u];
  }
  for (; i < vec_per_wg; i += 512) acc ^= p[i];
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9e3779b9u) *sink = 1;  // keeps the loads alive
}

// One wavefront per SIMD with the register tile of the large-batch GEMM and nothing else: 8 x 8 accumulator blocks of
// 16 x 16 in the AGPR half of the register file; a round multiplies four A fragments with eight B fragments (32 instructions),
// the first and the last four of the eight in turn.  The fragments hold pseudo-random values of both signs spread over the
// fp16 exponents that real operands have: what the matrix pipes sustain depends on the data (the chip is power-limited
// there), and constant operands read about 40 % higher.
__global__ __launch_bounds__(256, 1) void k_mfma_probe(float* out, int iters) {
  pv4f acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[i][k] = pv4f{0.f, 0.f, 0.f, 0.f};
  pv8h a[8], b[8];
  uint32_t h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
#pragma unroll
  for (int f = 0; f < 8; ++f)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h ^= h << 13; h ^= h >> 17; h ^= h << 5;   // xorshift32
      a[f][i] = (_Float16)(((int)(h & 0xffff) - 32768) * (1.0f / 32768.0f) * (1.0f + (float)((h >> 16) & 3)));
      h ^= h << 13; h ^= h >> 17; h ^= h << 5;
      b[f][i] = (_Float16)(((int)(h & 0xffff) - 32768) * (0.05f / 32768.0f) * (1.0f + (float)((h >> 16) & 3)));
    }
  asm volatile("s_nop 7" ::: "memory");  // accumulator writes settle before the first (inline-asm) MFMA reads them
  auto round = [&](int i0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 8; ++k)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc[i0 + i][k]) : "v"(a[i0 + i]), "v"(b[k]));
  };
  for (int it = 1; it < iters; it += 2) {
    round(0);
    round(4);
  }
  if (iters & 1) round(0);
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // the last ones retire before their accumulators are read
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      asm volatile("" : "+a"(acc[i][k])::"memory");
#pragma unroll
      for (int j = 0; j < 4; ++j) s += acc[i][k][j];
    }
  out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

}  // namespace

void launch_read_probe(const void* src, size_t bytes, void* sink, hipStream_t st) {
  const int wgs = 1024;
  const size_t vec_per_wg = bytes / 16 / wgs;
  if (vec_per_wg == 0) return;
  k_read_probe<<<wgs, 512, 0, st>>>((const pv4u*)src, vec_per_wg, (uint32_t*)sink);
}

double launch_mfma_probe(float* out, int workgroups, int iters, hipStream_t st) {
  k_mfma_probe<<<workgroups, 256, 0, st>>>(out, iters);
  // 4 wavefronts x 32 instructions per round, 2 * 16 * 16 * 32 flops each
  return (double)workgroups * 4.0 * 32.0 * (double)iters * 16384.0;
}

}  // namespace mtmc
