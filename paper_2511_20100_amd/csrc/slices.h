// Sums of the slices that a split-K product leaves, by the kernels that read them.
#pragma once

#include <hip/hip_runtime.h>

namespace mtmc {

constexpr int kMaxSlices = 8;  // gemm_lds_splits() gives no more

// a + slice(0) + ... + slice(N - 1), in that order, all slices asked for before the first is added: the bits of a loop over them
template <int N, class T, class Slice>
__host__ __device__ __attribute__((always_inline)) inline T add_slices_of(T a, Slice slice) {
  T v[N];
#pragma unroll
  for (int s = 0; s < N; ++s) v[s] = slice(s);
#pragma unroll
  for (int s = 0; s < N; ++s) a = a + v[s];
  return a;
}
// The same for n slices (0 .. kMaxSlices), which only the launch knows: a loop over such a count asks for one slice after the other, a
// trip to memory each.
template <class T, class Slice>
__host__ __device__ __attribute__((always_inline)) inline T add_slices(T a, int n, Slice slice) {
  switch (n) {
    case 1: return add_slices_of<1>(a, slice);
    case 2: return add_slices_of<2>(a, slice);
    case 3: return add_slices_of<3>(a, slice);
    case 4: return add_slices_of<4>(a, slice);
    case 5: return add_slices_of<5>(a, slice);
    case 6: return add_slices_of<6>(a, slice);
    case 7: return add_slices_of<7>(a, slice);
    case 8: return add_slices_of<8>(a, slice);
    default: return a;
  }
}

}  // namespace mtmc
