// Shared by the dense and the sparse search in the subspace of the code book (bmu_subspace.hip, bmu_subspace_csr.hip).
#pragma once

#include "som_internal.hpp"

#include <math.h>

namespace som {

typedef _Float16 f16x8s __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4s __attribute__((ext_vector_type(4)));
typedef float f32x16s __attribute__((ext_vector_type(16)));

constexpr float kVScale = 256.f;           // V is stored times this: |V_rc| <= 1, and fp16's subnormals stay out of the way

__device__ __forceinline__ float pow2_over(float m, float *inverse) {      // power of two above m (1 for 0 and non-finite m)
  int e = 0;
  if (m > 0.f && m < INFINITY) {
    (void)frexpf(m, &e);
    e = e < -100 ? -100 : (e > 126 ? 126 : e);
  }
  *inverse = ldexpf(1.f, -e);
  return ldexpf(1.f, e);
}

// An upper bound of a norm from an fp32 sum of squares in units of `scale`.
__device__ __forceinline__ float norm_above(float sum, float scale) { return (sqrtf(sum) * (1.f + 4e-4f) + 1e-15f) * scale; }

// c_i as the sum of three halves, to 2^-35 of the largest (its scale leaves it below 2^10): the coordinates kSubConst .. + 2
// of hi, which holds the coordinates 24 .. 31.
static_assert(kSubConst % 8 + 3 <= 8, "the node constants share one group of eight coordinates");
__device__ __forceinline__ void put_constant(f16x8s &hi, float c) {
#pragma unroll
  for (int e = kSubConst % 8; e < kSubConst % 8 + 3; ++e) { hi[e] = (_Float16)c; c -= (float)hi[e]; }
}
__device__ __forceinline__ float constant_scale(float wmax2, float *inverse) {
  const float s = pow2_over(wmax2, inverse) * 0x1p-10f;
  *inverse *= 0x1p10f;
  return s;
}

// Rounding of the measured residual |w'_i - V^T u_i| (see k_subspace_coords): left[] = its norms after 16, 32, 48 and 64
// coordinates, wm = the largest |w'|, un = |u_i|, u1 = sum_r |u_ir|, vn = the largest |V_r|, sw = the scale of the node's planes.
__device__ __forceinline__ float residual_slack(const float (&left)[4], float wm, float un, float u1, float vn, float sw, int dim) {
  const float sums = wm + 3.f * (left[0] + left[1] + left[2]) + 2.f * left[3] + 8.f * 0x1p-10f * vn * u1;
  return 0x1p-24f * (2.5f * (sums + vn * u1) + 18.f * vn * un + 2.f * vn * u1) * (1.f + 1e-3f) + 0x1p-22f * wm +
         sqrtf((float)dim) * 0x1p-25f * sw;
}

// The factor of the node constants in an instance's coordinates of scale s (which it may raise, inv with it): a power of two
// that a half holds exactly.  xs = the unit of the coordinates before they are scaled.
__device__ __forceinline__ float constant_factor(float &s, float &inv, float xs, float uscale, float cscale) {
  const float over = cscale / (2.f * s * xs * uscale) * 0x1p-15f;
  if (over > 1.f) { s *= over; inv /= over; }
  return -cscale / (2.f * s * xs * uscale);
}
__device__ __forceinline__ bool factor_fits(float cfac) { return -cfac >= 0x1p-24f && -cfac <= 0x1p15f; }

// Maxima over the nodes, put together by the last workgroup of a launch: those of a workgroup go into its five words of `part`, the
// last one to count itself in *ticket gets the maxima of all (true, in f).  All threads call it; f is thread 0's.
template <int kThreads>
__device__ __forceinline__ bool last_maxima(float (&f)[5], float *__restrict__ part, int32_t *__restrict__ ticket) {
  __shared__ float s_fin[kThreads / 64][5];
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) {
#pragma unroll
    for (int e = 0; e < 5; ++e) __hip_atomic_store(part + 5 * blockIdx.x + e, f[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!s_last) return false;
#pragma unroll
  for (int e = 0; e < 5; ++e) f[e] = 0.f;
  for (int b = tid; b < (int)gridDim.x; b += kThreads)
#pragma unroll
    for (int e = 0; e < 5; ++e) f[e] = fmaxf(f[e], __hip_atomic_load(part + 5 * b + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
  for (int e = 0; e < 5; ++e) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) f[e] = fmaxf(f[e], __shfl_xor(f[e], o, 64));
    if (lane == 0) s_fin[wave][e] = f[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 5; ++e)
    for (int p = 0; p < kThreads / 64; ++p) f[e] = fmaxf(f[e], s_fin[p][e]);
  return true;
}

// The basis, up to its vectors (bmu_subspace.hip): W, mu -> sub_Vp, sub_Vt (sub_Vf).  W null: the sketch sub_S is there.  loss: the
// share of the largest |w'| that may lie outside, for the end of an attempt.
hipError_t launch_subspace_basis(som_ctx *c, const float *W, float loss);

}  // namespace som
