// fp32 rows as two fp16 planes, for the BMU filter that runs on the fp16 matrix cores
// (paper: BMU equation; "Parallelism": distances through linear algebra).
//
// A row v is divided by a power of two s > max|v_c| (so |v/s| < 1: no fp16 overflow, and the
// division is exact), then every element is written as hi + lo with
//     hi = fp16(v/s),   lo = fp16(v/s - hi)     (both round-to-nearest; the subtraction is exact)
// which leaves |v/s - hi - lo| <= max(2^-22 |v/s|, 2^-25): fp16 keeps 11 significant bits and its
// subnormals end at 2^-24 (the matrix cores honour subnormal inputs).  The product of two such
// numbers is hi*hi' + hi*lo' + lo*hi' up to 3 * 2^-22 relative: three fp16 MFMAs give an fp32-grade
// dot product at a third of the fp16 rate, which is still more than five times the fp32 MFMA rate.
//
// Storage: rows are padded to whole chunks of 32 columns, and chunk t of a row is 128 bytes:
// the 32 hi halves of columns 32 t .. 32 t + 31, then their 32 lo halves.  That is exactly the
// shape of one LDS tile row of the filter kernel (bmu_dense_h.hip).  Padding columns are zero.
// The coarse pass of the two-level search reads the hi halves alone: a second copy, rows padded to
// whole chunks of 64 columns, 128 bytes per chunk again.
#include "row_load.hpp"
#include "som_internal.hpp"

#include <math.h>

namespace som {

// Power of two strictly above m (1 for m = 0 or a non-finite m), exponent kept inside fp32's range.
__device__ __forceinline__ float pow2_above(float m, float *inverse) {
  int e = 0;
  if (m > 0.f && m < INFINITY) {
    (void)frexpf(m, &e);          // m = f * 2^e, f in [0.5, 1)
    e = e < -100 ? -100 : (e > 127 ? 127 : e);
  }
  *inverse = ldexpf(1.f, -e);
  return ldexpf(1.f, e);
}

// Norm of what the hi halves of a row leave out, from the fp32 sum of its squares in units of the scale, rounded up
// (a sum of at most 2^12 rounded terms per lane, all of one sign, and what falls below fp32's range).
__device__ __forceinline__ float lost_norm(float sum, float scale) { return (sqrtf(sum) * (1.f + 4e-4f) + 1e-15f) * scale; }

// Largest value of a workgroup of kWaves wavefronts (their lanes hold it) into *out: one atomic, and none where the
// word is that large already.
template <int kWaves>
__device__ __forceinline__ void publish_max(float v, float (&scratch)[kWaves], unsigned *out) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) v = fmaxf(v, scratch[w]);
    if (v > __uint_as_float(__hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) atomicMax(out, __float_as_uint(v));
  }
}

// kTeam threads per row (a wavefront for short rows, the workgroup for long ones).  With
// `global_max_bits` every row uses the same scale (the code book: one factor for all nodes, so
// that the scores of an instance stay comparable without a per-node multiplication) and the
// scale is also written to *scale_out; without it each row gets its own scale in scale_out[row].
// With `mu` the rows are centred first, a_c - mu_c in fp32 (the instances of the dense search: their
// scores then carry |x - mu| instead of |x| in the rounding bound).  src, out_hi, res_out, res_max as in k_row_planes.
template <int kTeam>
__global__ __launch_bounds__(256) void k_split_rows_f16(const float *__restrict__ A, int64_t nrows, int dim, int nK,
                                                        const unsigned *__restrict__ global_max_bits,
                                                        const float *__restrict__ mu,
                                                        _Float16 *__restrict__ out, float *__restrict__ scale_out,
                                                        _Float16 *__restrict__ out_hi, const int32_t *__restrict__ src,
                                                        float *__restrict__ res_out, unsigned *__restrict__ res_max,
                                                        const SubspaceState *__restrict__ off) {
  if (off && off->use) return;
  __shared__ float smax[4];
  float worst = 0.f;
  constexpr int kTeams = 256 / kTeam;
  const int tl = threadIdx.x % kTeam, team = threadIdx.x / kTeam;
  const int padded = nK * 32;
  const int padded_hi = (nK + 1) / 2 * 64;
  for (int64_t r = (int64_t)blockIdx.x * kTeams + team; r < nrows; r += (int64_t)gridDim.x * kTeams) {
    const float *a = A + (src ? (int64_t)src[r] : r) * dim;
    float m, lost = 0.f;
    if (global_max_bits) {
      m = __uint_as_float(*global_max_bits);
    } else {
      m = 0.f;
      for (int c = tl; c < dim; c += kTeam) m = fmaxf(m, fabsf(mu ? a[c] - mu[c] : a[c]));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
      if (kTeam == 256) {          // r depends on the block only: every thread gets here
        __syncthreads();
        if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = m;
        __syncthreads();
        m = fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]));
      }
    }
    float inv;
    const float s = pow2_above(m, &inv);
    if (tl == 0) {
      if (global_max_bits) { if (r == 0) *scale_out = s; }
      else scale_out[r] = s;
    }
    _Float16 *o = out + r * (int64_t)nK * 64;
    for (int c = tl; c < padded; c += kTeam) {
      const float v = c < dim ? (mu ? a[c] - mu[c] : a[c]) * inv : 0.f;
      const _Float16 hi = (_Float16)v;
      const _Float16 lo = (_Float16)(v - (float)hi);
      const int at = (c >> 5) * 64 + (c & 31);
      o[at] = hi;
      o[at + 32] = lo;
      lost += (v - (float)hi) * (v - (float)hi);
      if (out_hi) out_hi[r * (int64_t)padded_hi + c] = hi;
    }
    if (res_out || res_max) {
      lost = team_sum<64>(lost);
      if (kTeam == 256) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = lost;
        __syncthreads();
        lost = (smax[0] + smax[1]) + (smax[2] + smax[3]);
      }
      lost = lost_norm(lost, s);
      worst = fmaxf(worst, lost);
      if (res_out && tl == 0) res_out[r] = lost;
    }
    if (out_hi && padded_hi > padded) {
      for (int c = padded + tl; c < padded_hi; c += kTeam) out_hi[r * (int64_t)padded_hi + c] = (_Float16)0.f;
    }
  }
  if (res_max) publish_max(worst, smax, res_max);
}

// ---------------------------------------------------------------- rows of up to 2,048 features: held in registers
// A wavefront keeps a whole row in registers (R groups of four features per lane, all loads in flight at once), so the
// centred row's norm, its scale and its planes come from one read, where norms and planes used to read the instances
// three times (100,000 x 1,000 unregistered instances, three planes: 115 + 350 us -> 185, 1 GB at 5.4 TB/s).  The centring vector
// stays in registers over all rows of a wavefront.
constexpr int kPlaneThreads = 1024;

// c_i = |w'_i|^2 (the instances are centred too), optionally |w_i|^2 in fp64, the largest |w'_i|^2 and
// the largest |w'| element, w' = fl(w - mu); c_i goes to the node's place in the planes, pos_of[i] (null: i).  fp64 sums in a fixed order per row.  One pair of atomics per workgroup of
// sixteen wavefronts (an atomic on one address takes about 10 ns, whoever issues it; 2,500 x 1,000: 20 -> 9 us).
template <int R>
__global__ __launch_bounds__(kPlaneThreads) void k_node_stats(const float *__restrict__ W, int k, int dim,
                                                              const float *__restrict__ mu, float *__restrict__ cn,
                                                              unsigned *__restrict__ max_bits, double *__restrict__ wn64,
                                                              const int32_t *__restrict__ pos_of) {
  __shared__ float s_max[2][kPlaneThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int stride = gridDim.x * (kPlaneThreads / 64);
  const bool wide = dim >= 4;
  f32x4r m[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int c = 4 * (lane + 64 * r);
    m[r] = wide ? row_load<true>(mu, c, dim) : row_load<false>(mu, c, dim);
    if (wide) row_tail<true>(m[r], c, dim); else row_tail<false>(m[r], c, dim);
  }
  float vmax = 0.f, amax = 0.f;
  for (int i = blockIdx.x * (kPlaneThreads / 64) + wave; i < k; i += stride) {
    const float *w = W + (int64_t)i * dim;
    f32x4r x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = wide ? row_load<true>(w, 4 * (lane + 64 * r), dim) : row_load<false>(w, 4 * (lane + 64 * r), dim);
    double s2 = 0.0, sw = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (wide) row_tail<true>(x[r], 4 * (lane + 64 * r), dim); else row_tail<false>(x[r], 4 * (lane + 64 * r), dim);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = x[r][e] - m[r][e];
        amax = fmaxf(amax, fabsf(t));
        s2 += (double)t * (double)t;
        sw += (double)x[r][e] * (double)x[r][e];
      }
    }
    s2 = wave_sum(s2);
    if (wn64) sw = wave_sum(sw);
    vmax = fmaxf(vmax, (float)s2);
    if (lane == 0) {
      cn[pos_of ? pos_of[i] : i] = (float)s2;
      if (wn64) wn64[i] = sw;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
  if (lane == 0) { s_max[0][wave] = vmax; s_max[1][wave] = amax; }
  __syncthreads();
  if (threadIdx.x < 2) {
    float v = 0.f;
    for (int w = 0; w < kPlaneThreads / 64; ++w) v = fmaxf(v, s_max[threadIdx.x][w]);
    if (v > 0.f) atomicMax(max_bits + threadIdx.x, __float_as_uint(v));
  }
}

// The planes of a row, its scale and (instances) the squared norm of the centred row.  global_max_bits as in
// k_split_rows_f16; row j of the planes is row src[j] of A (null: j).  The norm of what the hi halves leave out,
// |x' - hi|, goes to res_out[j], or the largest of them to *res_max: the coarse pass's error bound is made of it.
// Bound by memory: it reads 4 and writes 4 to 6 bytes per element.  Sixteen wavefronts per workgroup where res_max is
// asked for: one atomic each, and those on one address take their 10 ns one after the other.  kLanes lanes per row: 16 up
// to 64 features, 32 up to 128 (91,834 x 30: 39 -> 13 us), else the wavefront.
template <int R, int kThreads, int kLanes>
__global__ __launch_bounds__(kThreads) void k_row_planes(const float *__restrict__ A, int64_t nrows, int dim, int nK,
                                                    const unsigned *__restrict__ global_max_bits,
                                                    const float *__restrict__ mu, _Float16 *__restrict__ out,
                                                    float *__restrict__ scale_out, _Float16 *__restrict__ out_hi,
                                                    float *__restrict__ norm_out, const int32_t *__restrict__ src,
                                                    float *__restrict__ res_out, unsigned *__restrict__ res_max) {
  constexpr int kWaves = kThreads / 64;
  __shared__ float smax[kWaves];
  float worst = 0.f;
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  constexpr int kTeams = kThreads / kLanes;
  const int lane = threadIdx.x % kLanes;
  const int64_t stride = (int64_t)gridDim.x * kTeams;
  const bool wide = dim >= 4;
  const int padded = nK * 32, padded_hi = (nK + 1) / 2 * 64;
  f32x4r m[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int c = 4 * (lane + kLanes * r);
    m[r] = wide ? row_load<true>(mu, c, dim) : row_load<false>(mu, c, dim);
    if (wide) row_tail<true>(m[r], c, dim); else row_tail<false>(m[r], c, dim);
  }
  for (int64_t j = (int64_t)blockIdx.x * kTeams + threadIdx.x / kLanes; j < nrows; j += stride) {
    const float *a = A + (src ? (int64_t)src[j] : j) * dim;
    f32x4r x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = wide ? row_load<true>(a, 4 * (lane + kLanes * r), dim) : row_load<false>(a, 4 * (lane + kLanes * r), dim);
    float top = 0.f;
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (wide) row_tail<true>(x[r], 4 * (lane + kLanes * r), dim); else row_tail<false>(x[r], 4 * (lane + kLanes * r), dim);
      x[r] -= m[r];                              // fp32 difference, as the planes hold it
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        top = fmaxf(top, fabsf(x[r][e]));
        s += (double)x[r][e] * (double)x[r][e];
      }
    }
    if (global_max_bits) {
      top = __uint_as_float(*global_max_bits);
    } else {
#pragma unroll
      for (int o = kLanes / 2; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, 64));
    }
    float inv;
    const float scale = pow2_above(top, &inv);
    if (norm_out) s = team_sum<kLanes>(s);
    if (lane == 0) {
      if (!global_max_bits) scale_out[j] = scale;
      else if (j == 0) *scale_out = scale;
      if (norm_out) norm_out[j] = (float)s;
    }
    _Float16 *o = out + j * (int64_t)nK * 64;
    float lost = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = 4 * (lane + kLanes * r);
      f16x4 hi, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = x[r][e] * inv;
        hi[e] = (_Float16)v;
        const float rest = v - (float)hi[e];
        lo[e] = (_Float16)rest;
        lost += rest * rest;
      }
      if (c < padded) {
        _Float16 *at = o + (c >> 5) * 64 + (c & 31);
        *reinterpret_cast<f16x4 *>(at) = hi;
        *reinterpret_cast<f16x4 *>(at + 32) = lo;
      }
      if (out_hi && c < padded_hi) *reinterpret_cast<f16x4 *>(out_hi + j * (int64_t)padded_hi + c) = hi;
    }
    if (res_out || res_max) {
      lost = lost_norm(team_sum<kLanes>(lost), scale);
      worst = fmaxf(worst, lost);
      if (res_out && lane == 0) res_out[j] = lost;
    }
  }
  if (res_max) publish_max(worst, smax, res_max);
}

static bool rows_fit_registers(const som_ctx *c) { return c->dim <= kPlaneMaxDim; }

#define SOM_BY_ROW_GROUPS(dim, CALL)                                   \
  do {                                                                 \
    const int groups_ = ((dim) + 255) / 256;                           \
    if (groups_ <= 1) { CALL(1); } else if (groups_ <= 2) { CALL(2); } \
    else if (groups_ <= 4) { CALL(4); } else { CALL(8); }              \
  } while (0)

static hipError_t launch_row_planes(som_ctx *c, const float *A, int64_t nrows, const unsigned *global_max_bits, const float *mu,
                                    _Float16 *out, float *scale_out, _Float16 *out_hi, float *norm_out,
                                    const int32_t *src, float *res_out, unsigned *res_max) {
  const int lanes = c->dim <= 64 ? 16 : c->dim <= 128 ? 32 : 64;
  const int threads = res_max ? kPlaneThreads : 256;
  int64_t blocks = (nrows + threads / lanes - 1) / (threads / lanes);
  const int64_t cap = (int64_t)c->n_cu * (4096 / threads);
  if (blocks > cap) blocks = cap;
#define SOM_ROW_PLANES_OF(R, T, L)                                                                                      \
  hipLaunchKernelGGL((k_row_planes<R, T, L>), dim3((unsigned)blocks), dim3(T), 0, c->stream, A, nrows, c->dim,           \
                     (c->dim + 31) / 32, global_max_bits, mu, out, scale_out, out_hi, norm_out, src, res_out, res_max)
#define SOM_ROW_PLANES(R)                                        \
  do {                                                           \
    if (res_max) SOM_ROW_PLANES_OF(R, kPlaneThreads, 64);        \
    else SOM_ROW_PLANES_OF(R, 256, 64);                          \
  } while (0)
  if (lanes == 16) { if (res_max) SOM_ROW_PLANES_OF(1, kPlaneThreads, 16); else SOM_ROW_PLANES_OF(1, 256, 16); }
  else if (lanes == 32) { if (res_max) SOM_ROW_PLANES_OF(1, kPlaneThreads, 32); else SOM_ROW_PLANES_OF(1, 256, 32); }
  else SOM_BY_ROW_GROUPS(c->dim, SOM_ROW_PLANES);
#undef SOM_ROW_PLANES
#undef SOM_ROW_PLANES_OF
  return hipGetLastError();
}

// Centred code book for the filters that run on planes: node constants, maxima, planes and scale.  coarse: the rows stand
// in the order of the two-level search (c->node_of), with the hi halves a second time and the largest of their losses.
hipError_t launch_codebook_planes(som_ctx *c, const float *W, bool want_wn64, bool coarse) {
  _Float16 *hi = coarse ? c->Wh1 : nullptr;
  const int32_t *node_of = coarse ? c->node_of : nullptr, *pos_of = coarse ? c->pos_of : nullptr;
  unsigned *lost = coarse ? c->wlost_bits : nullptr;
  if (!rows_fit_registers(c)) {
    hipError_t e = launch_center_codebook(c, W, true, want_wn64, true, pos_of);
    if (e != hipSuccess) return e;
    return launch_split_rows_f16(c, c->Wc, c->k, c->wmax_bits + 1, nullptr, c->Wh, c->wscale, 0, hi, node_of, nullptr, lost);
  }
  int blocks = (c->k + kPlaneThreads / 64 - 1) / (kPlaneThreads / 64);
  if (blocks > c->n_cu) blocks = c->n_cu;
#define SOM_NODE_STATS(R)                                                                                            \
  hipLaunchKernelGGL(k_node_stats<R>, dim3(blocks), dim3(kPlaneThreads), 0, c->stream, W, c->k, c->dim, c->mu, c->wn32, \
                     c->wmax_bits, want_wn64 ? c->wn64 : nullptr, pos_of)
  SOM_BY_ROW_GROUPS(c->dim, SOM_NODE_STATS);
#undef SOM_NODE_STATS
  return launch_row_planes(c, W, c->k, c->wmax_bits + 1, c->mu, c->Wh, c->wscale, hi, nullptr, node_of, nullptr, lost);
}

// Planes, scales and squared norms of centred instances; coarse: with the hi halves a second time and their losses
// (first: which of the context's rows A starts at).
hipError_t launch_instance_planes(som_ctx *c, const float *A, int64_t nrows, const float *mu, int64_t first, bool coarse,
                                  float *norm_out) {
  _Float16 *out = c->Xh + (size_t)first * ((c->dim + 31) / 32) * 64;
  _Float16 *out_hi = coarse ? c->Xh1 + (size_t)first * ((c->dim + 63) / 64) * 64 : nullptr;
  float *lost = coarse ? c->xlost + first : nullptr;
  if (rows_fit_registers(c))
    return launch_row_planes(c, A, nrows, nullptr, mu, out, c->xscale + first, out_hi, norm_out, nullptr, lost, nullptr);
  hipError_t e = launch_row_sqnorms(c, A, nrows, c->dim, mu, norm_out, nullptr, nullptr);
  if (e != hipSuccess) return e;
  return launch_split_rows_f16(c, A, nrows, nullptr, mu, out, c->xscale + first, 0, out_hi, nullptr, lost, nullptr);
}

hipError_t launch_split_rows_f16(som_ctx *c, const float *A, int64_t nrows, const unsigned *global_max_bits,
                                 const float *mu, _Float16 *out, float *scale_out, int dim, _Float16 *out_hi,
                                 const int32_t *src, float *res_out, unsigned *res_max, const SubspaceState *off) {
  if (dim <= 0) dim = c->dim;
  const int nK = (dim + 31) / 32;
  const int64_t cap = (int64_t)c->n_cu * (res_max ? 4 : 16);
  if (dim <= 2048) {
    int64_t blocks = (nrows + 3) / 4;
    if (blocks > cap) blocks = cap;
    hipLaunchKernelGGL(k_split_rows_f16<64>, dim3((unsigned)blocks), dim3(256), 0, c->stream, A, nrows, dim, nK,
                       global_max_bits, mu, out, scale_out, out_hi, src, res_out, res_max, off);
  } else {
    int64_t blocks = nrows < cap ? nrows : cap;
    hipLaunchKernelGGL(k_split_rows_f16<256>, dim3((unsigned)blocks), dim3(256), 0, c->stream, A, nrows, dim, nK,
                       global_max_bits, mu, out, scale_out, out_hi, src, res_out, res_max, off);
  }
  return hipGetLastError();
}

// One v_mfma_f32_32x32x16_f16 on caller-given operands: D = A B^T + C with A [32][16] and
// B [32][16] fp16 bit patterns, C and D [32][32] fp32.  Exists so that a test can check the
// rounding behaviour that the error bound of the filter assumes of this instruction.
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

__global__ __launch_bounds__(64) void k_probe_mfma_f16(const _Float16 *__restrict__ A, const _Float16 *__restrict__ B,
                                                       const float *__restrict__ C, float *__restrict__ D,
                                                       int count) {
  const int l = threadIdx.x;
  for (int t = blockIdx.x; t < count; t += gridDim.x) {
    const _Float16 *a = A + (int64_t)t * 512, *b = B + (int64_t)t * 512;
    const float *cc = C + (int64_t)t * 1024;
    float *d = D + (int64_t)t * 1024;
    f16x8_t av, bv;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      av[v] = a[(l & 31) * 16 + (l >> 5) * 8 + v];
      bv[v] = b[(l & 31) * 16 + (l >> 5) * 8 + v];
    }
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = cc[(8 * (v >> 2) + 4 * (l >> 5) + (v & 3)) * 32 + (l & 31)];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 16; ++v) d[(8 * (v >> 2) + 4 * (l >> 5) + (v & 3)) * 32 + (l & 31)] = acc[v];
  }
}

hipError_t launch_probe_mfma_f16(hipStream_t stream, const uint16_t *A, const uint16_t *B, const float *C, float *D,
                                 int count) {
  hipLaunchKernelGGL(k_probe_mfma_f16, dim3((unsigned)(count < 1024 ? count : 1024)), dim3(64), 0, stream,
                     reinterpret_cast<const _Float16 *>(A), reinterpret_cast<const _Float16 *>(B), C, D, count);
  return hipGetLastError();
}

}  // namespace som
