// Sparse best-matching-unit search in the subspace of the code book (paper: sparse kernel; BMU equation).
//
// The sparse sweep (bmu_csr.hip) gathers a 16-bit code-book entry for every (nonzero, node) pair, and what its gathers send
// past L2 bounds it.  While the radius is wide the code book lies in 64 directions to a few 1e-6 of its
// norm (bmu_subspace.hip), here too: a nonzero then costs 64 multiply-adds whatever the number of nodes, and what is left is a
// dense search of n x 64 against k x 64, which is the two-level search on the coordinates, its fine and collect pass
// included, with the bound on what the coordinates leave out in its margins.  The exact stage works on
// the rows themselves as ever.  The device decides after the nodes' coordinates are known: `use` closes the kernels of the
// sweep, otherwise the ones here are closed and the sweep runs.
//
// As in the sweep only the code book is centred: s_i = c_i - 2 x.w'_i with c_i = |w'_i|^2 + 2 mu.w'_i, w' = w - mu.
// The nodes are in the order of the two-level search (node_of).  Rows of W are long (tens of thousands of features) and few, so
// the passes over them split the features over workgroups:
//   k_csr_node_sums     u = V w' per piece of the features, with the sums for c_i, |w_i|^2 and |w'_i|^2;
//   k_csr_node_constants, k_csr_node_coords   the pieces added up;
//   k_csr_node_losses   |w' - V^T u|^2 per piece;
//   k_csr_subspace_decide   maxima and decision;
//   k_csr_project       y = V x per instance, in fp64.
// 100,000 rows of 100 nonzeros, 50,000 features, 50 x 50 nodes: search 3,750 us with the sweep, 1,370 here; the epoch 4,809 -> 2,500.
#include "row_load.hpp"
#include "subspace.hpp"

namespace som {

constexpr int kCsrNodes = 64;          // nodes per workgroup of the passes over W
constexpr int kCsrWaves = 4;

// Eight consecutive centred features of a row as hi/lo halves, divided by the planes' scale; zeros behind the row.
struct NodeHalves {
  f16x8s hi, lo;
};
__device__ __forceinline__ NodeHalves node_halves(const f32x4r (&x)[2], const f32x4r (&m)[2], float inv) {
  NodeHalves r;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float t = (x[e >> 2][e & 3] - m[e >> 2][e & 3]) * inv;
    r.hi[e] = (_Float16)t;
    r.lo[e] = (_Float16)(t - (float)r.hi[e]);
  }
  return r;
}
__device__ __forceinline__ void load8(const float *__restrict__ row, int c, int dim, f32x4r (&x)[2]) {
  x[0] = row_load<true>(row, c, dim);
  x[1] = row_load<true>(row, c + 4, dim);
}
__device__ __forceinline__ void tail8(f32x4r (&x)[2], int c, int dim) {
  row_tail<true>(x[0], c, dim);
  row_tail<true>(x[1], c + 4, dim);
}

// Bound of |c_i| = |w'_i|^2 + 2 mu.w'_i.
__device__ __forceinline__ float constant_bound(float wm2, float munorm2) { return (wm2 + 2.f * sqrtf(wm2) * sqrtf(munorm2)) * (1.f + 1e-5f); }

// Scale of the nodes' halves: the columns' quantisation steps say how large a centred element gets.
__device__ __forceinline__ float node_scale(const unsigned *qstep_max_bits, float *inverse) {
  return pow2_over(__uint_as_float(*qstep_max_bits) * 32768.f, inverse);
}

// upart [piece][k][64]: V w' over the piece's chunks of 32 features, in units of scale / 256; npart [piece][k][3]: sums of w'^2, mu w', w^2
// (fp64, as the sweep takes them); vpart [piece][64]: squared row norms of V (times 256^2).  64 nodes per workgroup, the chunks dealt to its
// wavefronts.
__global__ __launch_bounds__(64 * kCsrWaves) void k_csr_node_sums(const float *__restrict__ W, const float *__restrict__ mu,
                                                                  const int32_t *__restrict__ node_of, int k, int dim, int nK,
                                                                  int per_piece, const _Float16 *__restrict__ Vp,
                                                                  const unsigned *__restrict__ qstep_max_bits,
                                                                  const SubspaceState *__restrict__ state,
                                                                  float *__restrict__ upart, double *__restrict__ npart,
                                                                  float *__restrict__ vpart) {
  if (state->full) return;
  __shared__ float s_u[kCsrWaves][kSub][33];
  __shared__ double s_n[kCsrWaves][3][kCsrNodes];
  __shared__ float s_v[kCsrWaves][kSub];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int p0 = blockIdx.x * kCsrNodes, piece = blockIdx.y;
  float inv;
  (void)node_scale(qstep_max_bits, &inv);
  const float *w[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) w[nb] = W + (int64_t)node_of[min(p0 + 32 * nb + l32, k - 1)] * dim;
  const f32x16s zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16s u[2][2] = {{zero, zero}, {zero, zero}};      // [block of coordinates][block of nodes]
  double s2[2] = {0.0, 0.0}, sm[2] = {0.0, 0.0}, sw[2] = {0.0, 0.0};
  float vsq[2] = {0.f, 0.f};
  const int t_end = min(nK, (piece + 1) * per_piece);
  f32x4r xn[2][2][2], mn[2][2];                        // next chunk: [k-step][block of nodes]
  auto load = [&](int t) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = 32 * t + 16 * ks + 8 * lhi;
      load8(mu, c, dim, mn[ks]);
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) load8(w[nb], c, dim, xn[ks][nb]);
    }
  };
  int t = piece * per_piece + wave;
  if (t < t_end) load(t);
  for (; t < t_end; t += kCsrWaves) {
    f32x4r x[2][2][2], m[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        m[ks][h] = mn[ks][h];
        x[ks][0][h] = xn[ks][0][h];
        x[ks][1][h] = xn[ks][1][h];
      }
    const _Float16 *v = Vp + ((int64_t)(t >> 1) * 2 * kSub + l32) * 64 + (t & 1) * 32 + 8 * lhi;
    f16x8s vh[2][2], vl[2][2];                         // [k-step][block of coordinates]
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        vh[ks][rb] = *reinterpret_cast<const f16x8s *>(v + rb * 32 * 64 + 16 * ks);
        vl[ks][rb] = *reinterpret_cast<const f16x8s *>(v + (kSub + rb * 32) * 64 + 16 * ks);
      }
    if (t + kCsrWaves < t_end) load(t + kCsrWaves);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = 32 * t + 16 * ks + 8 * lhi;
      tail8(m[ks], c, dim);
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        tail8(x[ks][nb], c, dim);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float xv = x[ks][nb][e >> 2][e & 3], mv = m[ks][e >> 2][e & 3], d = xv - mv;
          s2[nb] += (double)d * (double)d;
          sm[nb] += (double)mv * (double)d;
          sw[nb] += (double)xv * (double)xv;
        }
        const NodeHalves h = node_halves(x[ks][nb], m[ks], inv);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          u[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl[ks][rb], h.hi, u[rb][nb], 0, 0, 0);
          u[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[ks][rb], h.lo, u[rb][nb], 0, 0, 0);
          u[rb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[ks][rb], h.hi, u[rb][nb], 0, 0, 0);
        }
      }
      if (blockIdx.x == 0) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float f = (float)vh[ks][rb][e] + (float)vl[ks][rb][e];
            vsq[rb] += f * f;
          }
      }
    }
  }
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    s2[nb] += __shfl_xor(s2[nb], 32, 64);
    sm[nb] += __shfl_xor(sm[nb], 32, 64);
    sw[nb] += __shfl_xor(sw[nb], 32, 64);
    vsq[nb] += __shfl_xor(vsq[nb], 32, 64);
    if (lhi == 0) {
      s_n[wave][0][32 * nb + l32] = s2[nb];
      s_n[wave][1][32 * nb + l32] = sm[nb];
      s_n[wave][2][32 * nb + l32] = sw[nb];
      s_v[wave][32 * nb + l32] = vsq[nb];
    }
  }
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int e = 0; e < 16; ++e) s_u[wave][rb * 32 + 8 * (e >> 2) + 4 * lhi + (e & 3)][l32] = u[rb][nb][e];
    __syncthreads();
    for (int o = tid; o < 32 * kSub; o += 64 * kCsrWaves) {
      const int r = o & 63, nd = o >> 6, p = p0 + 32 * nb + nd;
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < kCsrWaves; ++q) s += s_u[q][r][nd];
      if (p < k) upart[((int64_t)piece * k + p) * kSub + r] = s;
    }
  }
  if (tid < 3 * kCsrNodes) {
    const int which = tid >> 6, nd = tid & 63;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kCsrWaves; ++q) s += s_n[q][which][nd];
    if (p0 + nd < k) npart[((int64_t)piece * k + p0 + nd) * 3 + which] = s;
  }
  if (blockIdx.x == 0 && tid < kSub) {
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < kCsrWaves; ++q) s += s_v[q][tid];
    vpart[piece * kSub + tid] = s;
  }
}

// c_i at the node's place, |w_i|^2 under its number, the largest |w'_i|^2.  Sixteen lanes per node take the pieces in turn.
__global__ __launch_bounds__(256) void k_csr_node_constants(const double *__restrict__ npart, int pieces, int k,
                                                            const int32_t *__restrict__ node_of,
                                                            const SubspaceState *__restrict__ state, float *__restrict__ cn,
                                                            double *__restrict__ wn64, unsigned *__restrict__ wmax_bits) {
  if (state->full) return;
  const int part = threadIdx.x & 15, p = blockIdx.x * 16 + (threadIdx.x >> 4);
  double s2 = 0.0, sm = 0.0, sw = 0.0;
  if (p < k)
    for (int q = part; q < pieces; q += 16) {
      const double *at = npart + ((int64_t)q * k + p) * 3;
      s2 += at[0]; sm += at[1]; sw += at[2];
    }
  s2 = team_sum<16>(s2);
  sm = team_sum<16>(sm);
  sw = team_sum<16>(sw);
  float vmax = 0.f;
  if (p < k) {
    if (part == 0) {
      cn[p] = (float)(s2 + 2.0 * sm);
      wn64[node_of[p]] = sw;
    }
    vmax = (float)s2;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o, 64));
  if ((threadIdx.x & 63) == 0 && vmax > 0.f) atomicMax(wmax_bits, __float_as_uint(vmax));
}

// The coordinates, added over the pieces, as planes: eight per thread.  nstat [k][3]: sums of u^2, |u| and lo(u)^2 over a node's
// coordinates, in units of the coordinates' scale.
__global__ __launch_bounds__(256) void k_csr_node_coords(const float *__restrict__ upart, int pieces, int k,
                                                         const unsigned *__restrict__ qstep_max_bits,
                                                         const unsigned *__restrict__ wmax_bits,
                                                         const float *__restrict__ mu_norm2, const float *__restrict__ cn,
                                                         const SubspaceState *__restrict__ state, _Float16 *__restrict__ U1,
                                                         _Float16 *__restrict__ U2, float *__restrict__ nstat) {
  if (state->full) return;
  const int g = threadIdx.x & 7, p = blockIdx.x * 32 + (threadIdx.x >> 3);
  float inv, uinv, cinv;
  const float sw = node_scale(qstep_max_bits, &inv);
  const float wm2 = __uint_as_float(*wmax_bits);
  (void)pow2_over(sqrtf(wm2) * (1.f + 1e-3f), &uinv);
  (void)constant_scale(constant_bound(wm2, *mu_norm2), &cinv);
  float u[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (p < k)
    for (int q = 0; q < pieces; ++q) {
      const f32x4r *at = reinterpret_cast<const f32x4r *>(upart + ((int64_t)q * k + p) * kSub + 8 * g);
      const f32x4r a = at[0], b = at[1];
#pragma unroll
      for (int e = 0; e < 4; ++e) { u[e] += a[e]; u[4 + e] += b[e]; }
    }
  f16x8s hi, lo;
  float su = 0.f, s1 = 0.f, sl = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = u[e] * (sw * uinv) * (1.f / kVScale);
    hi[e] = (_Float16)v;
    lo[e] = (_Float16)(v - (float)hi[e]);
    su += v * v;
    s1 += fabsf(v);
    sl += (float)lo[e] * (float)lo[e];
  }
  su = team_sum<8>(su);
  s1 = team_sum<8>(s1);
  sl = team_sum<8>(sl);
  if (p >= k) return;
  if (g == 0) { nstat[3 * p] = su; nstat[3 * p + 1] = s1; nstat[3 * p + 2] = sl; }
  _Float16 *u2 = U2 + (int64_t)p * 2 * kSub + (g >> 2) * 64 + (g & 3) * 8;
  *reinterpret_cast<f16x8s *>(u2) = hi;
  *reinterpret_cast<f16x8s *>(u2 + 32) = lo;
  if (g == kSubConst / 8) put_constant(hi, cn[p] * cinv);
  *reinterpret_cast<f16x8s *>(U1 + (int64_t)p * kSub + 8 * g) = hi;
}

// epart [piece][k][4]: squared norms of what 16, 32, 48 and 64 coordinates leave of w' over the piece, in units of (coordinates' scale / 256)^2.
// V^T u - w' on the matrix cores, w' through products with the identity, as in k_subspace_coords.
__global__ __launch_bounds__(64 * kCsrWaves) void k_csr_node_losses(const float *__restrict__ W, const float *__restrict__ mu,
                                                                    const int32_t *__restrict__ node_of, int k, int dim, int nK,
                                                                    int per_piece, const _Float16 *__restrict__ Vt,
                                                                    const _Float16 *__restrict__ U2,
                                                                    const unsigned *__restrict__ qstep_max_bits,
                                                                    const unsigned *__restrict__ wmax_bits,
                                                                    const SubspaceState *__restrict__ state,
                                                                    float *__restrict__ epart) {
  if (state->full) return;
  __shared__ float s_e[kCsrWaves][4][kCsrNodes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int p0 = blockIdx.x * kCsrNodes, piece = blockIdx.y;
  float inv, uinv;
  const float sw = node_scale(qstep_max_bits, &inv);
  (void)pow2_over(sqrtf(__uint_as_float(*wmax_bits)) * (1.f + 1e-3f), &uinv);
  f16x8s ident[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) ident[ks][e] = (_Float16)(l32 == 16 * ks + 8 * lhi + e ? -kVScale * (sw * uinv) : 0.f);
  const float *w[2];
  f16x8s uh[2][4], ul[2][4];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int p = min(p0 + 32 * nb + l32, k - 1);
    w[nb] = W + (int64_t)node_of[p] * dim;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const _Float16 *at = U2 + (int64_t)p * 2 * kSub + (ks >> 1) * 64 + (ks & 1) * 16 + 8 * lhi;
      uh[nb][ks] = *reinterpret_cast<const f16x8s *>(at);
      ul[nb][ks] = *reinterpret_cast<const f16x8s *>(at + 32);
    }
  }
  float esq[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  const int t_end = min(nK, (piece + 1) * per_piece);
  f32x4r xn[2][2][2], mn[2][2];
  auto load = [&](int t) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = 32 * t + 16 * ks + 8 * lhi;
      load8(mu, c, dim, mn[ks]);
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) load8(w[nb], c, dim, xn[ks][nb]);
    }
  };
  int t = piece * per_piece + wave;
  if (t < t_end) load(t);
  for (; t < t_end; t += kCsrWaves) {
    const _Float16 *v = Vt + (int64_t)(t * 32 + l32) * 2 * kSub + 8 * lhi;
    f16x8s vh[4], vl[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      vh[ks] = *reinterpret_cast<const f16x8s *>(v + 16 * ks);
      vl[ks] = *reinterpret_cast<const f16x8s *>(v + kSub + 16 * ks);
    }
    f32x16s d[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) d[nb] = f32x16s{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = 32 * t + 16 * ks + 8 * lhi;
      f32x4r m[2] = {mn[ks][0], mn[ks][1]};
      tail8(m, c, dim);
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        f32x4r x[2] = {xn[ks][nb][0], xn[ks][nb][1]};
        tail8(x, c, dim);
        const NodeHalves h = node_halves(x, m, inv);
        d[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ident[ks], h.hi, d[nb], 0, 0, 0);
        d[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ident[ks], h.lo, d[nb], 0, 0, 0);
      }
    }
    if (t + kCsrWaves < t_end) load(t + kCsrWaves);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        d[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[ks], uh[nb][ks], d[nb], 0, 0, 0);
        d[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl[ks], uh[nb][ks], d[nb], 0, 0, 0);
        d[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[ks], ul[nb][ks], d[nb], 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e) esq[nb][ks] += d[nb][e] * d[nb][e];
      }
  }
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      esq[nb][ks] += __shfl_xor(esq[nb][ks], 32, 64);
      if (lhi == 0) s_e[wave][ks][32 * nb + l32] = esq[nb][ks];
    }
  __syncthreads();
  for (int o = tid; o < 4 * kCsrNodes; o += 64 * kCsrWaves) {
    const int ks = o & 3, nd = o >> 2;
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < kCsrWaves; ++q) s += s_e[q][ks][nd];
    if (p0 + nd < k) epart[((int64_t)piece * k + p0 + nd) * 4 + ks] = s;
  }
}

// Bounds per node, their maxima, and whether the search goes this way.
__global__ __launch_bounds__(256) void k_csr_subspace_decide(const float *__restrict__ epart, int pieces, int k, int dim,
                                                             const float *__restrict__ nstat, const float *__restrict__ vpart,
                                                             const unsigned *__restrict__ qstep_max_bits,
                                                             const unsigned *__restrict__ wmax_bits,
                                                             const float *__restrict__ mu_norm2, float *__restrict__ part,
                                                             int32_t *__restrict__ ticket, SubspaceState *__restrict__ state) {
  if (state->full) return;
  __shared__ float s_top[4][5], s_vn;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float inv, uinv, cinv;
  const float sw = node_scale(qstep_max_bits, &inv);
  const float wm2 = __uint_as_float(*wmax_bits), wm = sqrtf(wm2) * (1.f + 1e-6f);
  const float unit = pow2_over(sqrtf(wm2) * (1.f + 1e-3f), &uinv);
  if (wave == 0) {
    float v = 0.f;
#pragma unroll 8
    for (int q = 0; q < pieces; ++q) v += vpart[q * kSub + lane];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    if (lane == 0) s_vn = sqrtf(v) * (1.f + 4e-4f) / kVScale;
  }
  __syncthreads();
  const float vn = s_vn;
  float f[5] = {0.f, 0.f, 0.f, 0.f, 0.f};      // losses of 64, |u|, |u|_1, lo(u), losses of 32
  for (int p0 = blockIdx.x * 32; p0 < k; p0 += gridDim.x * 32) {      // eight threads per node
    const int p = min(p0 + (tid >> 3), k - 1);
    float left[4] = {0.f, 0.f, 0.f, 0.f};
    for (int q = tid & 7; q < pieces; q += 8) {
      const f32x4r v = *reinterpret_cast<const f32x4r *>(epart + ((int64_t)q * k + p) * 4);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) left[ks] += v[ks];
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) left[ks] = norm_above(team_sum<8>(left[ks]), unit * (1.f / kVScale));
    const float un = norm_above(nstat[3 * p], unit), u1 = nstat[3 * p + 1] * unit * (1.f + 1e-4f);
    const float slack = residual_slack(left, wm, un, u1, vn, sw, dim);
    const float e64 = left[3] + slack, e32 = left[1] + slack;
    f[0] = e64 < INFINITY ? fmaxf(f[0], e64) : INFINITY;         // NaN counts as infinite
    f[1] = fmaxf(f[1], un);
    f[2] = fmaxf(f[2], u1);
    f[3] = fmaxf(f[3], norm_above(nstat[3 * p + 2], unit));
    f[4] = e32 < INFINITY ? fmaxf(f[4], e32) : INFINITY;
  }
#pragma unroll
  for (int e = 0; e < 5; ++e) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) f[e] = fmaxf(f[e], __shfl_xor(f[e], o, 64));
    if (lane == 0) s_top[wave][e] = f[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 5; ++e) f[e] = fmaxf(fmaxf(s_top[0][e], s_top[1][e]), fmaxf(s_top[2][e], s_top[3][e]));
  if (last_maxima<256>(f, part, ticket) && tid == 0) {
    const int use = !(f[0] <= kSubspaceLossCsr * wm && f[1] < INFINITY) ? 0 : f[4] <= kSubspaceLoss32 * wm ? 1 : 2;
    state->use = use;
    state->fine = use != 0;
    state->e = use == 1 ? f[4] : f[0];
    state->e32 = f[4];
    state->e64 = f[0];
    state->u = f[1];
    state->u1 = f[2] * vn;
    state->ulost = f[3];
    state->wm = wm;
    state->uscale = unit;
    state->cmax = constant_bound(wm2, *mu_norm2);
    state->cscale = constant_scale(state->cmax, &cinv);
  }
}

// ---------------------------------------------------------------- the instances
// y = V x, a wavefront per row, a coordinate per lane; nonzeros handed round with v_readlane as in the sweep, eight rows of V (256
// contiguous bytes each) in flight.  In fp64: in fp32 the roundings of a row of 100 nonzeros alone would be several times what 64
// coordinates leave out.
__global__ __launch_bounds__(256) void k_csr_project(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                     const float *__restrict__ values, int64_t n, int dim,
                                                     const float *__restrict__ Vf, const float *__restrict__ xn32,
                                                     const SubspaceState *__restrict__ state, _Float16 *__restrict__ Y1,
                                                     _Float16 *__restrict__ Y2, float *__restrict__ yscale, float *__restrict__ err,
                                                     float *__restrict__ err2) {
  const int use = state->use;
  if (!use) return;
  constexpr int kAhead = 8;
  const int lane = threadIdx.x & 63;
  const float um = state->u, ulost = state->ulost, e1 = state->e, e64 = state->e64;
  const float uscale = state->uscale, cscale = state->cscale;
  const float *vl = Vf + lane;
  for (int64_t j = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); j < n; j += (int64_t)gridDim.x * 4) {
    const int64_t rs = indptr[j];
    const int len = (int)(indptr[j + 1] - rs);
    double y = 0.0;
    for (int p0 = 0; p0 < len; p0 += 64) {
      int c = 0;
      float v = 0.f;
      if (p0 + lane < len) {
        c = indices[rs + p0 + lane];
        c = c < 0 ? 0 : (c >= dim ? dim - 1 : c);
        v = values[rs + p0 + lane];
      }
      const int m = min(64, len - p0);
      int q = 0;
      for (; q + kAhead <= m; q += kAhead) {
        float a[kAhead];
#pragma unroll
        for (int t = 0; t < kAhead; ++t) a[t] = vl[(int64_t)__builtin_amdgcn_readlane(c, q + t) * kSub];
#pragma unroll
        for (int t = 0; t < kAhead; ++t)
          y = fma((double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), q + t)), (double)a[t], y);
      }
      for (; q < m; ++q)
        y = fma((double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), q)),
                (double)vl[(int64_t)__builtin_amdgcn_readlane(c, q) * kSub], y);
    }
    const float yf = (float)y;
    float top = fabsf(yf);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o, 64));
    float inv;
    float s = pow2_over(top, &inv);
    const float cfac = constant_factor(s, inv, 1.f, uscale, cscale);
    const float ys = yf * inv;
    _Float16 hi = (_Float16)ys;
    const float rest = ys - (float)hi;
    Y2[j * 2 * kSub + (lane >> 5) * 64 + (lane & 31)] = hi;
    Y2[j * 2 * kSub + (lane >> 5) * 64 + 32 + (lane & 31)] = (_Float16)rest;
    float ysq = ys * ys, lost = rest * rest;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      ysq += __shfl_xor(ysq, o, 64);
      lost += __shfl_xor(lost, o, 64);
    }
    if (lane >= kSubConst && lane < kSubConst + 3) hi = (_Float16)cfac;
    if (use == 1) { if (lane < 32) Y1[j * 32 + lane] = hi; }
    else Y1[j * kSub + lane] = hi;
    if (lane == 0) {
      const float xn = sqrtf(xn32[j]) * (1.f + 1e-6f), yn = norm_above(ysq, s), yl = norm_above(lost, s);
      yscale[j] = s;
      // as in the dense projection; y itself is off by its rounding to fp32 and by that of its chain, len 2^-53 |x| |V_r| a coordinate
      // and eight times that (|V_r| is 1 to a few 1e-3, so sixteen) over the 64
      const float b = (0x1p-23f * yn + (float)len * 0x1p-49f * xn) * um;
      err[j] = factor_fits(cfac)
                   ? (b + xn * e1 + yl * um + (yn + yl) * (ulost + 21.f * 0x1p-24f * um) + 12.f * 0x1p-24f * state->cmax) * (1.f + 1e-3f)
                   : INFINITY;
      err2[j] = (b + xn * e64 + (0x1p-22f * yn + 8.f * 0x1p-25f * s) * um + (42.f + 12.f) * 0x1p-24f * yn * um) * (1.f + 1e-3f);
    }
  }
}

// ---------------------------------------------------------------- host side
// Workgroups along the features of the passes over W: about five per CU in all.
static int csr_pieces(const som_ctx *c) {
  const int tiles = (c->k + kCsrNodes - 1) / kCsrNodes, nK = (c->dim + 31) / 32;
  int pieces = (5 * c->n_cu + tiles - 1) / tiles;
  if (pieces > kCtMaxSlabs) pieces = kCtMaxSlabs;
  if (pieces > (nK + kCsrWaves - 1) / kCsrWaves) pieces = (nK + kCsrWaves - 1) / kCsrWaves;
  if (pieces < 1) pieces = 1;
  const int per = (nK + pieces - 1) / pieces;
  return (nK + per - 1) / per;
}
size_t subspace_csr_part_floats(const som_ctx *c) { return (size_t)csr_pieces(c) * c->k * (kSub + 4) + (size_t)kCtMaxSlabs * kSub + 3 * (size_t)c->k; }

// Worth its scratch for n rows of nnz nonzeros?  The sweep takes 0.13 ps per nonzero and node (hot block included); this 0.25 ms, three more
// reads of the code book and 30 ps per nonzero, all measured at 50 x 50 nodes.  It has to promise three times its own cost, and
// half as much again where the two-level search is asked for by name (epochs, sweep / coordinates: 20,000 rows of 20,000 features on 2,500 nodes,
// which is 1.4 times, 1,356 / 1,046 us; 2,000 of 5,000 on 900 nodes, 0.1 times, 288 / 339).  On a toroid the distance across the seam has a kink that every chosen node carries over the map: 1e-2 of the code book of a text-like
// set stays outside 64 directions at any radius, so planar maps only.  Grows with n and nnz.
bool subspace_csr_eligible(const som_ctx *c, int64_t n, int64_t nnz) {
  const int64_t blocks = (c->k + 127) / 128;
  if (c->nb_function != SOM_NEIGHBORHOOD_GAUSSIAN || c->nb_compact) return false;
  if (c->map_type != SOM_MAP_PLANAR || c->dim < kSubspaceCsrDim || blocks * c->n_cap * 4 > kTwoLevelMaxTable) return false;
  if (c->sub_always) return true;
  if (c->filter != SOM_FILTER_TWO_LEVEL && (c->filter != SOM_FILTER_AUTO || blocks < kTwoLevelMinBlocks)) return false;
  const double own = 0.25e-3 + 3e-12 * (double)c->k * (double)c->dim + 3e-11 * (double)nnz;
  return 1.3e-13 * (double)nnz * (double)c->k >= (c->filter == SOM_FILTER_AUTO ? 3.0 : 1.4) * own;
}

// The code book left by an epoch of this radius or more lies in 64 directions to 3e-5 of its norm up to 16 to 17 nodes per squared
// radius on planar maps (text-like rows, square and hexagonal, 400 to 10,000 nodes: 1e-5 at 15, 8e-5 at 21).
bool subspace_csr_likely(const som_ctx *c, double radius) {
  return radius > 0.0 && (double)c->rows * (double)c->cols <= kSubspaceCsrMaxArea * radius * radius;
}

hipError_t launch_csr_subspace(som_ctx *c, const int64_t *indptr, const int32_t *indices, const float *values, int64_t n, const float *W) {
  const hipError_t e = launch_subspace_basis(c, nullptr, 2.f * kSubspaceLossCsr);      // (an attempt costs a ninth of what it may save)
  if (e != hipSuccess) return e;
  const int nK = (c->dim + 31) / 32, pieces = csr_pieces(c), per = (nK + pieces - 1) / pieces;
  const int tiles = (c->k + kCsrNodes - 1) / kCsrNodes;
  float *upart = c->sub_cpart, *epart = upart + (size_t)pieces * c->k * kSub, *vpart = epart + (size_t)pieces * c->k * 4;
  float *nstat = vpart + (size_t)kCtMaxSlabs * kSub;
  hipLaunchKernelGGL(k_csr_node_sums, dim3(tiles, pieces), dim3(64 * kCsrWaves), 0, c->stream, W, c->mu, c->node_of, c->k, c->dim, nK, per,
                     c->sub_Vp, c->qstep_max_bits, c->sub_state, upart, c->ct_partial, vpart);
  hipLaunchKernelGGL(k_csr_node_constants, dim3((c->k + 15) / 16), dim3(256), 0, c->stream, c->ct_partial, pieces, c->k, c->node_of,
                     c->sub_state, c->wn32, c->wn64, c->wmax_bits);
  hipLaunchKernelGGL(k_csr_node_coords, dim3((c->k + 31) / 32), dim3(256), 0, c->stream, upart, pieces, c->k, c->qstep_max_bits,
                     c->wmax_bits, c->mu_norm2, c->wn32, c->sub_state, c->sub_U1, c->sub_U2, nstat);
  hipLaunchKernelGGL(k_csr_node_losses, dim3(tiles, pieces), dim3(64 * kCsrWaves), 0, c->stream, W, c->mu, c->node_of, c->k, c->dim, nK,
                     per, c->sub_Vt, c->sub_U2, c->qstep_max_bits, c->wmax_bits, c->sub_state, epart);
  int blocks = (c->k + 31) / 32;
  if (blocks > kSubspaceParts) blocks = kSubspaceParts;
  hipLaunchKernelGGL(k_csr_subspace_decide, dim3(blocks), dim3(256), 0, c->stream, epart, pieces, c->k, c->dim, nstat, vpart,
                     c->qstep_max_bits, c->wmax_bits, c->mu_norm2, c->sub_part, c->list_counts + kSubTicketWord, c->sub_state);
  int64_t rows = (n + 3) / 4;
  if (rows > (int64_t)c->n_cu * 16) rows = (int64_t)c->n_cu * 16;
  hipLaunchKernelGGL(k_csr_project, dim3((unsigned)rows), dim3(256), 0, c->stream, indptr, indices, values, n, c->dim, c->sub_Vf,
                     c->xn32, c->sub_state, c->sub_Y1, c->sub_Y2, c->sub_yscale, c->sub_err, c->sub_err2);
  return hipGetLastError();
}

}  // namespace som
