// Four consecutive features of a row of any length and alignment with one 16-byte load.
#pragma once

#include <hip/hip_runtime.h>

namespace som {

typedef float f32x4r __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Features c .. c + 3 (c a multiple of 4), loaded on a 4-byte boundary and moved back where they would reach past the
// row; row_tail puts them in place then, with zeros behind.  The two are apart because what stands between a load and
// its use has the compiler wait for everything in flight.  kWide = false: rows of one to three features.
template <bool kWide>
__device__ __forceinline__ f32x4r row_load(const float *__restrict__ row, int c, int dim) {
  f32x4r v;
  if (kWide) {
    const f32x4u t = *reinterpret_cast<const f32x4u *>(row + min(c, dim - 4));
    v = f32x4r{t[0], t[1], t[2], t[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = row[min(c + e, dim - 1)];
  }
  return v;
}

template <bool kWide>
__device__ __forceinline__ void row_tail(f32x4r &v, int c, int dim) {
  if (kWide) {
    const int s = c - (dim - 4);                // how far the load was moved back, if at all
    if (s > 0) {
      const f32x4r t = (s & 1) ? f32x4r{v[1], v[2], v[3], 0.f} : v;
      const f32x4r u = (s & 2) ? f32x4r{t[2], t[3], 0.f, 0.f} : t;
      v = s >= 4 ? f32x4r{0.f, 0.f, 0.f, 0.f} : u;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = c + e < dim ? v[e] : 0.f;
  }
}

// Sum over the kLanes lanes (a power of two) of this lane's team, in all of them.
template <int kLanes, typename T>
__device__ __forceinline__ T team_sum(T v) {
#pragma unroll
  for (int o = kLanes / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace som
