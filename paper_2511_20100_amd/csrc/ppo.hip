// Clipped surrogate of the PPO update over scored samples (value and two diagnostics, no gradient).
// Per-workgroup partial sums in double, then one workgroup adds the partials; both reductions run in a fixed order, so the result
// does not depend on scheduling.
//
// What bounds calls of few samples that follow each other is the host: a launch costs it 2.5 us.  One instead of two takes a tag
// beside every partial sum: the call's own 64-bit number, stored when the sum is where others see it.  A workgroup that has stored
// its tag looks at all of them; the last one to store does see them all.  (Two that see them write the same result.)  It clears
// the tags behind itself, so that a launch that is replayed with the number it was recorded with starts without them.  Nobody
// waits.  The device pays for that with two trips to memory, and more the more workgroups look.  us a call, two launches -> one:
//   workgroups (1024 samples)      8            32           64           96           128          192          256          512
//   calls that follow each other   10.6 -> 7.9  10.6 -> 8.2  10.7 -> 8.3  10.9 -> 8.2  10.9 -> 8.3  10.9 -> 11.5 10.9 -> 8.8  10.9 -> 41
//   a call that is waited for      22.0 -> 21.8 21.8 -> 22.3 21.9 -> 23.0 21.6 -> 23.3 21.7 -> 23.7 21.7 -> 25.6 21.8 -> 24.3 22.6 -> 58
// Up to kPpoAlone the former gain more than the latter lose.
#include <atomic>
#include <chrono>
#include <mutex>
#include <random>

#include "common.h"
#include "kernels.h"

namespace mtmc {

namespace {

constexpr int kPpoBlocks = 1024;   // partial results at most
constexpr int kPpoThreads = 256;
constexpr int kPpoAlone = 128;     // ... that one launch adds up

struct PpoSums {
  double surrogate, clipped, kl, count;
};

// ... and as they lie in the workspace.  Counts are whole and below 2^32 (1024 workgroups share n samples, three floats each).
struct PpoPartial {
  double surrogate, kl;
  uint32_t clipped, count;
  uint64_t tag;
};
// ALONE: between workgroups of one launch
template <bool ALONE, class T>
__device__ __forceinline__ T ppo_load(const T* p) {
  if (!ALONE) return *p;
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool ALONE, class T>
__device__ __forceinline__ void ppo_store(T* p, T v) {
  if (ALONE) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

__device__ __forceinline__ PpoSums ppo_add(const PpoSums& a, const PpoSums& b) {
  return PpoSums{a.surrogate + b.surrogate, a.clipped + b.clipped, a.kl + b.kl, a.count + b.count};
}

// Sum over the workgroup in a fixed tree; the result is valid in thread 0.
__device__ __forceinline__ PpoSums ppo_block_sum(PpoSums v, PpoSums* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = kPpoThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = ppo_add(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  return red[0];
}

// The sum of n_partial partials in a fixed order, by one workgroup.
template <bool ALONE>
__device__ __forceinline__ void ppo_finish(PpoPartial* partial, int n_partial, PpoSums* red, double* out) {
  PpoSums s{0.0, 0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < n_partial; i += kPpoThreads) {
    PpoPartial* p = partial + i;
    s = ppo_add(s, PpoSums{ppo_load<ALONE>(&p->surrogate), (double)ppo_load<ALONE>(&p->clipped), ppo_load<ALONE>(&p->kl),
                           (double)ppo_load<ALONE>(&p->count)});
    if (ALONE) ppo_store<true>(&p->tag, (uint64_t)0);
  }
  s = ppo_block_sum(s, red);
  if (threadIdx.x == 0) {
    const double c = s.count > 0.0 ? s.count : 1.0;
    out[0] = -s.surrogate / c;
    out[1] = s.clipped / c;
    out[2] = s.kl / c;
    out[3] = s.count;
  }
}

template <bool ALONE>
__global__ __launch_bounds__(kPpoThreads) void k_ppo(const float* new_logp, const float* old_logp, const float* adv, const int* mask,
                                                     long long n, double eps, PpoPartial* partial, uint64_t tag, double* out) {
  __shared__ PpoSums red[kPpoThreads];
  PpoSums s{0.0, 0.0, 0.0, 0.0};
  for (long long i = (long long)blockIdx.x * kPpoThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kPpoThreads) {
    if (mask && mask[i] == 0) continue;
    const double d = (double)new_logp[i] - (double)old_logp[i];
    const double r = exp(d), a = (double)adv[i];
    const double rc = fmin(fmax(r, 1.0 - eps), 1.0 + eps);
    s.surrogate += fmin(r * a, rc * a);
    s.clipped += (fabs(r - 1.0) > eps) ? 1.0 : 0.0;
    s.kl -= d;
    s.count += 1.0;
  }
  s = ppo_block_sum(s, red);
  if (threadIdx.x == 0) {
    PpoPartial* p = partial + blockIdx.x;
    ppo_store<ALONE>(&p->surrogate, s.surrogate);
    ppo_store<ALONE>(&p->kl, s.kl);
    ppo_store<ALONE>(&p->clipped, (uint32_t)s.clipped);
    ppo_store<ALONE>(&p->count, (uint32_t)s.count);
    if (ALONE) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the sum is there before its tag
      ppo_store<true>(&p->tag, tag);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // and the tag before the look at the others
    }
  }
  if (!ALONE) return;
  __syncthreads();
  int all = 1;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += kPpoThreads) all &= ppo_load<true>(&partial[i].tag) == tag;
  if (!__syncthreads_and(all)) return;
  ppo_finish<true>(partial, gridDim.x, red, out);
}

__global__ __launch_bounds__(kPpoThreads) void k_ppo_final(PpoPartial* partial, int n_partial, double* out) {
  __shared__ PpoSums red[kPpoThreads];
  ppo_finish<false>(partial, n_partial, red, out);
}

// Partial sums of the entry point that takes no workspace: one copy of this array per GPU, part of the loaded
// code object, alive until the process ends.  Host code never uses the array's name as an address: it asks the
// runtime for the device address once per device (ppo_static_scratch) and passes that to the kernels.
static __device__ __align__(256) unsigned char scratch[kPpoBlocks * sizeof(PpoPartial)];

// A number that no other call of this or an earlier process has left in a workspace (never 0).
uint64_t ppo_tag() {
  static std::atomic<uint64_t> next{((uint64_t)std::random_device{}() << 32 | std::random_device{}()) ^
                                    (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count()};
  uint64_t z = next.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);  // splitmix64: a permutation of a counter
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z ? z : 1;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

size_t ppo_workspace_bytes() { return kPpoBlocks * sizeof(PpoPartial); }

// Device address of this GPU's copy of `scratch` (looked up on the first call on a device, with that device current).
int ppo_static_scratch(void** out) {
  int dev = -1;
  MTMC_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("device index " + std::to_string(dev) + " is beyond the " + std::to_string(kMaxDevices) +
              " devices the static scratch table covers");
    return MTMC_EINVAL;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    MTMC_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) {
      set_error("hipGetSymbolAddress returned no address for the static scratch array");
      return MTMC_EHIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return MTMC_OK;
}

void launch_ppo_clip_loss(const float* new_logp, const float* old_logp, const float* adv, const int* mask,
                          long long n, double eps, double* out, void* workspace, hipStream_t st) {
  const long long want = (n + 4 * kPpoThreads - 1) / (4 * kPpoThreads);
  const int blocks = (int)(want < 1 ? 1 : want > kPpoBlocks ? kPpoBlocks : want);
  PpoPartial* partial = reinterpret_cast<PpoPartial*>(workspace);
  if (blocks <= kPpoAlone) {
    k_ppo<true><<<blocks, kPpoThreads, 0, st>>>(new_logp, old_logp, adv, mask, n, eps, partial, ppo_tag(), out);
    return;
  }
  k_ppo<false><<<blocks, kPpoThreads, 0, st>>>(new_logp, old_logp, adv, mask, n, eps, partial, 0, out);
  k_ppo_final<<<1, kPpoThreads, 0, st>>>(partial, blocks, out);
}

}  // namespace mtmc
