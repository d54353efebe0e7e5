// Dense best-matching-unit search: the coarse pass in the subspace that the code book spans (paper: BMU equation;
// batch and neighbourhood equations, which is where the subspace comes from).
//
// A batch update leaves every weight vector a weighted mean of the same few sums, the weights smooth over the map: while
// the radius is wide, the k x dim code book is numerically of rank far below both k and dim (50 x 50 nodes at a radius
// of a third of the map: its part outside 64 directions is 2e-6 of its norm).  With V [64][dim] nearly orthonormal rows
// that span it, u_i the coordinates of node i and y = V x' those of an instance,
//     x'.w'_i = y.u_i + x'.e_i,      e_i = w'_i - V^T u_i   (whatever u and V are),
// so |x'| max|e_i| bounds what a score from 64 products instead of dim leaves out.  The coarse pass of the two-level
// search (bmu_coarse.hip) only has to bound every block's best score; it takes these 64-feature operands in the
// place of the full ones wherever the measured max|e_i| is small, and the block selection adds the bound to its margin.
// The fine pass and the exact stage work on the full rows as before: the BMUs do not depend on any of this.
//
//   k_subspace_sketch   S[r] = sum of +- w'_i over the nodes i = r mod 61: 61 random combinations whose span is the
//                       code book's as far as so many directions go (as good as dense random signs in every case
//                       tried, and one pass over the code book); three rows in between stay zero, their coordinates
//                       carry the node constants through the coarse pass;
//   k_subspace_gram     S S^T in fp64;
//   k_subspace_factor   its Cholesky factor's inverse, directions below 1e-6 of the largest dropped;
//   k_subspace_vectors  V = L^-1 S as fp16 hi/lo planes, in the two orders that the next two kernels read;
//   k_subspace_coords   u = V w' and |w' - V^T u| per node on the matrix cores (split fp16, three products), the maxima over the
//                       nodes, and the decision;
//   k_subspace_project  y = V x' for every instance, from the hi halves of its planes, and the bound on its scores.
// Measured (MI355X, a whole epoch, without -> with): 100,000 x 1,000 on 50 x 50 nodes 860 -> 561 us (coarse pass 518 ->
// 31, the six kernels 155), 50,000 x 256 on 200 x 200 1,541 -> 982 (1,163 -> 266 + 145), 1,000,000 x 128 on 100 x 100 4,000 ->
// 2,009 (3,060 -> 708 + 165).
#include "subspace.hpp"

namespace som {

constexpr double kDropPivot = 1e-12;       // (relative norm)^2 below which a sketch row adds no direction
constexpr int kGramCols = 128;             // features per workgroup of the Gram matrix

// ---------------------------------------------------------------- basis
// A workgroup per (bucket, 64 features); eight node subgroups.  Bound by the read of the code book out of L2.
__global__ __launch_bounds__(512) void k_subspace_sketch(const float *__restrict__ W, int k, int dim, int dimp,
                                                         const float *__restrict__ mu, float *__restrict__ S) {
  __shared__ float s_part[8][64];
  const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int r = blockIdx.x, c = blockIdx.y * 64 + lane;
  const int first = r < kSubConst ? r : r < kSubConst + 3 ? k : r - 3;
  const bool in = c < dim;
  const float m = in ? mu[c] : 0.f;
  float acc = 0.f;
#pragma unroll 4
  for (int64_t i = first + (int64_t)kSketchBuckets * sub; i < k; i += kSketchBuckets * 8) {
    const float v = in ? W[i * dim + c] - m : 0.f;
    acc += sketch_sign((int)i) ? v : -v;
  }
  s_part[sub][lane] = acc;
  __syncthreads();
  if (sub == 0) {
#pragma unroll
    for (int p = 1; p < 8; ++p) acc += s_part[p][lane];
    S[(int64_t)r * dimp + c] = acc;          // zeros behind the row's end
  }
}

// G = S S^T in fp64 on the matrix cores, kGramCols features per workgroup and a partial matrix for each such piece (their sum: k_gram_sum,
// or the factor itself where there are few).  A wavefront owns the 16 rows 16 wave .. of G; lane l16 holds a row, its quad four features of every 16, and
// instruction e takes feature 4 quad + e of both operands (vector code with the rows in LDS: 48 us at 50,000 features).
__global__ __launch_bounds__(256) void k_subspace_gram(const float *__restrict__ S, int dimp, double *__restrict__ G) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, quad = lane >> 4;
  const int c_end = min(dimp, ((int)blockIdx.x + 1) * kGramCols);      // (a multiple of 64)
  f64x4 acc[4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll 4
  for (int c = blockIdx.x * kGramCols + 4 * quad; c < c_end; c += 16) {
    f32x4 b[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) b[t] = *reinterpret_cast<const f32x4 *>(S + (int64_t)(16 * t + l16) * dimp + c);
    const f32x4 a = *reinterpret_cast<const f32x4 *>(S + (int64_t)(16 * wave + l16) * dimp + c);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[e], (double)b[t][e], acc[t], 0, 0, 0);
  }
  G += (int64_t)blockIdx.x * kSub * kSub;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) G[(16 * wave + 4 * v + quad) * kSub + 16 * t + l16] = acc[t][v];
}

__global__ __launch_bounds__(256) void k_gram_sum(double *__restrict__ G, int pieces) {      // into the first piece
  __shared__ double s_part[4][64];
  const int o = blockIdx.x * 64 + (threadIdx.x & 63), part = threadIdx.x >> 6;
  double s = 0.0;
#pragma unroll 8
  for (int p = part; p < pieces; p += 4) s += G[(int64_t)p * kSub * kSub + o];
  s_part[part][threadIdx.x & 63] = s;
  __syncthreads();
  if (part == 0) G[o] = (s_part[0][threadIdx.x] + s_part[1][threadIdx.x]) + (s_part[2][threadIdx.x] + s_part[3][threadIdx.x]);
}

// Linv^T of G = L L^T by elimination on [G | I], one workgroup, both matrices in registers (4 x 4 entries of each per
// thread); per step the pivot's column and the right half's row go round through LDS.  A pivot under the
// floor (or NaN) gives no direction: its row of L^-1 is zero.  Bound by 64 dependent steps: the reciprocal is a Newton
// iteration (any basis will do that is nearly orthonormal), the square roots are left for the end, and blocks of 16 rows
// and columns that are done or still zero are left out; two pivots are exchanged at a time, and the pieces of G are read sixteen entries at once (30.7 -> 21 us).
// An attempt that the nodes' losses would end anyway ends here where the pivots say so: the last eight are what the directions before
// each leave of a random combination of the nodes, and the largest loss was 1.3 to 3.4 times their root mean square wherever it was within
// a factor of two of kSubspaceLoss (230 trained code books, 2,500 to 40,000 nodes, dense and text-like), so half of
// `loss` draws the line: of 105 books of 50 to 80 clusters on toroids it ended 59 of the 70 hopeless attempts and 3 of the
// 35 others, all three at the very edge.  A last direction of a sixteenth of the limit says that the rank ends here.  40,000 nodes of 64
// clusters, radius a quarter of the map: an epoch without an attempt 1,637 us, with one that the losses ended 1,717, with one that ends here 1,640.
__global__ __launch_bounds__(256) void k_subspace_factor(const double *__restrict__ G, int pieces, float loss, double *__restrict__ LinvT,
                                                         SubspaceState *__restrict__ state) {
  __shared__ double s_col[2][2][kSub], s_row[2][2][kSub], s_linv[kSub][kSub + 1], s_pivot[kSub];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  double m[4][4], w[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      m[a][b] = 0.0;
      w[a][b] = ty + 16 * a == tx + 16 * b ? 1.0 : 0.0;
    }
#pragma unroll 2
  for (int p = 0; p < pieces; ++p)               // sixteen loads of a piece in flight
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) m[a][b] += G[(int64_t)p * kSub * kSub + (ty + 16 * a) * kSub + tx + 16 * b];
  if (tx == ty) {                                // the diagonal
#pragma unroll
    for (int a = 0; a < 4; ++a) s_pivot[ty + 16 * a] = m[a][a];
  }
  __syncthreads();
  double top = s_pivot[tid & 63];               // the largest pivot
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
  __syncthreads();
  const double floor_p = top * kDropPivot;
  auto reciprocal = [&](double p) {              // zero for a pivot that gives no direction
    double inv = __builtin_amdgcn_rcp(p);
    inv = fma(fma(-p, inv, 1.0), inv, inv);
    inv = fma(fma(-p, inv, 1.0), inv, inv);
    return p > floor_p && p < INFINITY ? inv : 0.0;
  };
#pragma unroll
  for (int tb = 0; tb < 4; ++tb) {
#pragma unroll 1
    for (int tt = 0; tt < 16; tt += 2) {         // two pivots per exchange: the second one's column and row are brought up to date by every reader
      const int t = 16 * tb + tt, par = (tt >> 1) & 1;
      if ((tx & ~1) == tt) {
#pragma unroll
        for (int a = 0; a < 4; ++a) s_col[par][tx & 1][ty + 16 * a] = m[a][tb];
      }
      if ((ty & ~1) == tt) {
#pragma unroll
        for (int b = 0; b < 4; ++b) s_row[par][ty & 1][tx + 16 * b] = w[tb][b];
      }
      __syncthreads();
      const double *col0 = s_col[par][0], *col1 = s_col[par][1], *row0 = s_row[par][0], *row1 = s_row[par][1];
      const double p0 = col0[t], c01 = col0[t + 1];            // (m is symmetric: column t at row t + 1 is column t + 1 at row t)
      const double inv0 = reciprocal(p0), g = c01 * inv0;
      const double p1 = fma(-g, c01, col1[t + 1]), inv1 = reciprocal(p1);
      if (tid < kSub) {
        s_linv[t][tid] = row0[tid];
        s_linv[t + 1][tid] = fma(-g, row0[tid], row1[tid]);
        if (tid == 0) {
          s_pivot[t] = inv0 != 0.0 ? p0 : 0.0;
          s_pivot[t + 1] = inv1 != 0.0 ? p1 : 0.0;
        }
      }
      double cj0[4], cj1[4], rj0[4], rj1[4];
#pragma unroll
      for (int b = tb; b < 4; ++b) {
        cj0[b] = col0[tx + 16 * b];
        cj1[b] = fma(-g, cj0[b], col1[tx + 16 * b]);
      }
#pragma unroll
      for (int b = 0; b <= tb; ++b) {
        rj0[b] = row0[tx + 16 * b];
        rj1[b] = fma(-g, rj0[b], row1[tx + 16 * b]);
      }
#pragma unroll
      for (int a = tb; a < 4; ++a) {
        const int i = ty + 16 * a;
        const double ci = col0[i];
        const double f0 = i > t ? ci * inv0 : 0.0;
        const double f1 = i > t + 1 ? fma(-g, ci, col1[i]) * inv1 : 0.0;
#pragma unroll
        for (int b = tb; b < 4; ++b) m[a][b] = fma(-f1, cj1[b], fma(-f0, cj0[b], m[a][b]));
#pragma unroll
        for (int b = 0; b <= tb; ++b) w[a][b] = fma(-f1, rj1[b], fma(-f0, rj0[b], w[a][b]));
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    double least = top, sum = 0.0;
    for (int t = kSub - 8; t < kSub; ++t) {
      least = fmin(least, s_pivot[t]);
      sum += s_pivot[t];
    }
    const double limit = top * ((double)loss * (double)loss);
    state->use = state->fine = 0;
    state->full = !(sum <= 8.0 * 0.25 * limit || least <= limit / 256.0);
    state->e32 = state->e64 = -1.f;      // not measured
  }
  if (tid < kSub) s_pivot[tid] = s_pivot[tid] > 0.0 ? 1.0 / sqrt(s_pivot[tid]) : 0.0;
  __syncthreads();
  const double norm = s_pivot[tid & 63];
  for (int s = tid >> 6; s < kSub; s += 4) LinvT[s * kSub + (tid & 63)] = norm > 0.0 ? s_linv[tid & 63][s] * norm : 0.0;
}

// V = L^-1 S times kVScale, as hi/lo halves: Vp [chunk of 64 features][plane][64 r][64 features] and
// Vt [feature][plane][64 r].  A workgroup per 64 features, eight rows of V per wavefront.
__global__ __launch_bounds__(512) void k_subspace_vectors(const float *__restrict__ S, int dimp, const double *__restrict__ LinvT,
                                                          const SubspaceState *__restrict__ state,
                                                          _Float16 *__restrict__ Vp, _Float16 *__restrict__ Vt,
                                                          float *__restrict__ Vf) {
  if (state->full) return;
  const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blockIdx.x * 64 + lane;
  double v[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 16
  for (int s = 0; s < kSub; ++s) {
    const double x = (double)S[(int64_t)s * dimp + c];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += LinvT[s * kSub + 8 * g + e] * x;
  }
  f16x8s hi, lo;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float f = (float)v[e] * kVScale;
    hi[e] = (_Float16)f;
    lo[e] = (_Float16)(f - (float)hi[e]);
    _Float16 *at = Vp + ((int64_t)blockIdx.x * 2 * kSub + 8 * g + e) * 64 + lane;
    at[0] = hi[e];
    at[kSub * 64] = lo[e];
  }
  if (Vf) {                                     // sparse rows gather the vectors feature by feature
#pragma unroll
    for (int e = 0; e < 8; ++e) Vf[(int64_t)c * kSub + 8 * g + e] = ((float)hi[e] + (float)lo[e]) * (1.f / kVScale);
  }
  *reinterpret_cast<f16x8s *>(Vt + (int64_t)c * 2 * kSub + 8 * g) = hi;
  *reinterpret_cast<f16x8s *>(Vt + (int64_t)c * 2 * kSub + kSub + 8 * g) = lo;
}

// ---------------------------------------------------------------- the nodes
// 32 nodes per workgroup and step, the chunks of 32 features dealt to its eight wavefronts, twice: u = V w' (summed over
// the wavefronts through LDS), then w' - V^T u, whose squares are added up.  In both products a lane holds one node.  The
// residual is formed by the matrix cores alone: w' enters through products with 256 s over that power times the identity.
// Units: planes hold w'/s (s = *wscale), V times 256, u divided by a power of two above the largest |w'|.
// Roundings of the residual: w' is put together exactly; then a matrix instruction rounds by 2.5 u of the accumulator it finds and of its
// products' magnitudes at most, and by 9 u of its largest product (the model of the filter passes; those of the four groups of 16 add up to 2 |u| |V_r| at most); accumulators are no longer
// than what so many coordinates leave, which is measured after every 16 (plus products with a lo half, 2^-10 of |u|_1), and the
// magnitudes add up to |u|_1 |V_r|.  The dropped lo.lo products are below 2^-23 |u|_1 |V_r|, the planes' own residual below 2^-22 |w'| and
// 2^-25 s per element.  With all magnitudes priced in every instruction instead the bound was seven times as large, and the
// fine pass could not have used the coordinates.  Per wavefront and 32 features 12 + 16 matrix instructions on 12 KB from
// L2: the latency of those loads bounds it on small maps.
__global__ __launch_bounds__(512) void k_subspace_coords(const _Float16 *__restrict__ Wh, int k, int dim, int nK,
                                                         const _Float16 *__restrict__ Vp, const _Float16 *__restrict__ Vt,
                                                         const float *__restrict__ wscale, const unsigned *__restrict__ wmax_bits,
                                                         const float *__restrict__ cn, _Float16 *__restrict__ U1, _Float16 *__restrict__ U2,
                                                         int may_fine, float *__restrict__ part,
                                                         int32_t *__restrict__ ticket, SubspaceState *__restrict__ state) {
  __shared__ float s_u[4][kSub][33];
  __shared__ __attribute__((aligned(16))) _Float16 s_un[2][32][kSub + 8];     // -u as hi/lo planes
  __shared__ float s_sum[3][8][32], s_e[4][8][32], s_v[8][2][64];
  if (state->full) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const float sw = *wscale;
  const float wm = sqrtf(__uint_as_float(*wmax_bits)) * (1.f + 1e-6f);
  float uinv, cinv;
  const float unit = pow2_over(wm * (1.f + 1e-3f), &uinv);        // of the u planes
  const float cscale = constant_scale(__uint_as_float(*wmax_bits), &cinv);
  f16x8s ident[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) ident[ks][e] = (_Float16)(l32 == 16 * ks + 8 * lhi + e ? kVScale * (sw * uinv) : 0.f);
  const f32x16s zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float top_e = 0.f, top_e32 = 0.f, top_u = 0.f, top_u1 = 0.f, top_lost = 0.f, vn = 0.f;
  const int tiles = (k + 31) / 32;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int node = min(tile * 32 + l32, k - 1);
    const _Float16 *w = Wh + (int64_t)node * nK * 64 + 8 * lhi;
    f32x16s u[2] = {zero, zero};
    float vsq[2] = {0.f, 0.f};
    // a chunk's operands: [k-step][hi, lo] of the nodes, [k-step][block of 32 rows][hi, lo] of V; the next chunk's are
    // in flight while one is multiplied
    f16x8s wn[2][2], vn8[2][2][2];
    auto load_u = [&](int t) {
      const _Float16 *v = Vp + ((int64_t)(t >> 1) * 2 * kSub + l32) * 64 + (t & 1) * 32 + 8 * lhi;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
          wn[ks][pl] = *reinterpret_cast<const f16x8s *>(w + t * 64 + 32 * pl + 16 * ks);
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) vn8[ks][rb][pl] = *reinterpret_cast<const f16x8s *>(v + (pl * kSub + rb * 32) * 64 + 16 * ks);
        }
    };
    if (wave < nK) load_u(wave);
    for (int t = wave; t < nK; t += 8) {
      f16x8s wc[2][2], vc[2][2][2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
          wc[ks][pl] = wn[ks][pl];
          vc[ks][0][pl] = vn8[ks][0][pl];
          vc[ks][1][pl] = vn8[ks][1][pl];
        }
      if (t + 8 < nK) load_u(t + 8);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          const f16x8s vh = vc[ks][rb][0], vl = vc[ks][rb][1];
          u[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl, wc[ks][0], u[rb], 0, 0, 0);
          u[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, wc[ks][1], u[rb], 0, 0, 0);
          u[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, wc[ks][0], u[rb], 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float f = (float)vh[e] + (float)vl[e];
            vsq[rb] += f * f;
          }
        }
    }
    // operands of the residual: the planes of the nodes again and V in the other order
    f16x8s wr[2][2], vr[4][2];
    auto load_e = [&](int t) {
      const _Float16 *v = Vt + (int64_t)(t * 32 + l32) * 2 * kSub + 8 * lhi;
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) wr[ks][pl] = *reinterpret_cast<const f16x8s *>(w + t * 64 + 32 * pl + 16 * ks);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) vr[ks][pl] = *reinterpret_cast<const f16x8s *>(v + pl * kSub + 16 * ks);
      }
    };
    if (wave < nK) load_e(wave);
    __syncthreads();                                 // the previous step's readers are done
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      if (wave >= 4) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s_u[wave - 4][rb * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3)][l32] = u[rb][v];
      }
      s_v[wave][rb][lane] = vsq[rb];
    }
    __syncthreads();
    if (wave < 4) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) s_u[wave][rb * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3)][l32] += u[rb][v];
    }
    __syncthreads();
    if (tid < 256) {
      const int nd = tid & 31, g = tid >> 5;         // eight coordinates of one node
      float su = 0.f, s1 = 0.f, sl = 0.f;
      f16x8s hi, lo, nhi, nlo;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = 8 * g + e;
        float un = 0.f;
#pragma unroll
        for (int p = 0; p < 4; ++p) un += s_u[p][r][nd];
        un *= sw * uinv * (1.f / kVScale);
        hi[e] = (_Float16)un;
        lo[e] = (_Float16)(un - (float)hi[e]);
        nhi[e] = -hi[e];
        nlo[e] = -lo[e];
        su += un * un;
        s1 += fabsf(un);
        sl += (float)lo[e] * (float)lo[e];
      }
      *reinterpret_cast<f16x8s *>(&s_un[0][nd][8 * g]) = nhi;
      *reinterpret_cast<f16x8s *>(&s_un[1][nd][8 * g]) = nlo;
      s_sum[0][g][nd] = su;
      s_sum[1][g][nd] = s1;
      s_sum[2][g][nd] = sl;
      if (tile * 32 + nd < k) {
        _Float16 *u2 = U2 + (int64_t)(tile * 32 + nd) * 2 * kSub + (g >> 2) * 64 + (g & 3) * 8;
        *reinterpret_cast<f16x8s *>(u2) = hi;
        *reinterpret_cast<f16x8s *>(u2 + 32) = lo;
        if (g == kSubConst / 8) put_constant(hi, cn[tile * 32 + nd] * cinv);
        *reinterpret_cast<f16x8s *>(U1 + (int64_t)(tile * 32 + nd) * kSub + 8 * g) = hi;
      }
    }
    {                                                // largest row norm of V: row 32 rb + l32 is spread over waves and halves
      float f = 0.f;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        float s = 0.f;
#pragma unroll
        for (int p = 0; p < 8; ++p) s += s_v[p][rb][l32] + s_v[p][rb][32 + l32];
        f = fmaxf(f, s);
      }
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) f = fmaxf(f, __shfl_xor(f, o, 64));
      vn = sqrtf(f) * (1.f + 4e-4f) / kVScale;
    }
    __syncthreads();
    f16x8s uh[4], ul[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      uh[ks] = *reinterpret_cast<const f16x8s *>(&s_un[0][l32][16 * ks + 8 * lhi]);
      ul[ks] = *reinterpret_cast<const f16x8s *>(&s_un[1][l32][16 * ks + 8 * lhi]);
    }
    float esq[4] = {0.f, 0.f, 0.f, 0.f};
    for (int t = wave; t < nK; t += 8) {
      f32x16s d = zero;
      f16x8s vc[4][2];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) { vc[ks][0] = vr[ks][0]; vc[ks][1] = vr[ks][1]; }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        d = __builtin_amdgcn_mfma_f32_32x32x16_f16(ident[ks], wr[ks][0], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x16_f16(ident[ks], wr[ks][1], d, 0, 0, 0);
      }
      if (t + 8 < nK) load_e(t + 8);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const f16x8s vh = vc[ks][0], vl = vc[ks][1];
        d = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, uh[ks], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl, uh[ks], d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, ul[ks], d, 0, 0, 0);
#pragma unroll
        for (int v2 = 0; v2 < 16; ++v2) esq[ks] += d[v2] * d[v2];      // what 16, 32, 48, 64 coordinates leave
      }
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      esq[ks] += __shfl_xor(esq[ks], 32, 64);
      if (lhi == 0) s_e[ks][wave][l32] = esq[ks];
    }
    __syncthreads();
    if (tid < 32) {
      float su = 0.f, s1 = 0.f, sl = 0.f;
#pragma unroll
      for (int g = 0; g < 8; ++g) { su += s_sum[0][g][tid]; s1 += s_sum[1][g][tid]; sl += s_sum[2][g][tid]; }
      float left[4];                                 // norms
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        left[ks] = 0.f;
#pragma unroll
        for (int p = 0; p < 8; ++p) left[ks] += s_e[ks][p][tid];
        left[ks] = norm_above(left[ks], unit * (1.f / kVScale));
      }
      const float u1 = s1 * unit * (1.f + 1e-4f);
      const float un = sqrtf(su) * (1.f + 1e-4f) * unit;
      const float slack = residual_slack(left, wm, un, u1, vn, sw, dim);
      const float e2 = left[3] + slack, e32 = left[1] + slack;
      top_e = e2 < INFINITY ? fmaxf(top_e, e2) : INFINITY;     // NaN counts as infinite
      top_e32 = e32 < INFINITY ? fmaxf(top_e32, e32) : INFINITY;
      top_u = fmaxf(top_u, un);
      top_u1 = fmaxf(top_u1, u1);
      top_lost = fmaxf(top_lost, (sqrtf(sl) * (1.f + 1e-4f) + 1e-15f) * unit);
    }
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) {
    top_e = fmaxf(top_e, __shfl_xor(top_e, o, 64));
    top_e32 = fmaxf(top_e32, __shfl_xor(top_e32, o, 64));
    top_u = fmaxf(top_u, __shfl_xor(top_u, o, 64));
    top_u1 = fmaxf(top_u1, __shfl_xor(top_u1, o, 64));
    top_lost = fmaxf(top_lost, __shfl_xor(top_lost, o, 64));
  }
  float f[5] = {top_e, top_u, top_u1, top_lost, top_e32};
  if (last_maxima<512>(f, part, ticket) && tid == 0) {
    const int use = !(f[1] < INFINITY) ? 0 : f[4] <= kSubspaceLoss32 * wm ? 1 : f[0] <= kSubspaceLoss * wm ? 2 : 0;
    state->use = use;
    state->fine = may_fine && use && f[0] <= kSubspaceLossFine * wm;
    state->e = use == 1 ? f[4] : f[0];
    state->e32 = f[4];
    state->e64 = f[0];
    state->u = f[1];
    state->u1 = f[2] * vn;
    state->ulost = f[3];
    state->wm = wm;
    state->cmax = __uint_as_float(*wmax_bits);
    state->uscale = unit;
    state->cscale = cscale;
  }
}

// ---------------------------------------------------------------- the instances
// y = V hi(x') of 256 instances per workgroup, 64 per wavefront: V a chunk of 64 features at a time through LDS (16-byte slots swizzled as in
// the coarse pass), the instances' halves straight from memory into the operand registers, one chunk ahead.  Bound by
// the read of the hi planes (2 bytes per element).
// A lane holds one instance; err[j] bounds |x'.w'_i - (the coarse pass's y.u_i)| for every node i.
template <int kRB, bool kFine>
__device__ __forceinline__ void project_rows(const _Float16 *__restrict__ Xp, int64_t n, int dim, const _Float16 *__restrict__ Vp,
                                             const float *__restrict__ xscale, const float *__restrict__ xn32,
                                             const float *__restrict__ xlost, const SubspaceState *__restrict__ state,
                                             _Float16 *__restrict__ Y1, _Float16 *__restrict__ Y2, float *__restrict__ yscale,
                                             float *__restrict__ err, float *__restrict__ err2, _Float16 (&s_v)[2][2 * kSub * 64],
                                             const int64_t tile) {
  constexpr int kXPlanes = kFine ? 2 : 1, kIB = kFine ? 1 : 2;      // blocks of 32 instances per wavefront
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int nK = (dim + 63) / 64, nK32 = (dim + 31) / 32;
  const int64_t inst0 = (tile * 4 + wave) * (32 * kIB);
  if (tile * (128 * kIB) >= n) return;     // uniform over the workgroup
  const _Float16 *x[kIB];
#pragma unroll
  for (int ib = 0; ib < kIB; ++ib) {
    int64_t j = inst0 + ib * 32 + l32;
    if (j > n - 1) j = n - 1;
    x[ib] = Xp + j * (int64_t)(kFine ? nK32 : nK) * 64 + 8 * lhi;
  }
  // loader: the chunk's 128 rows (64 hi, 64 lo) of 128 bytes, four 16-byte slots per thread
  int st_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int slot = i * 256 + tid, row = slot >> 3, pos = slot & 7;
    st_off[i] = row * 64 + 8 * (pos ^ ((row & 7) ^ ((row >> 3) & 1)));
  }
  const int swz = (l32 & 7) ^ ((l32 >> 3) & 1);
  const f32x16s zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16s acc[kRB][kIB], tot[kFine ? kRB : 1][kIB];
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
    for (int ib = 0; ib < kIB; ++ib) {
      acc[rb][ib] = zero;
      if (kFine) tot[rb][ib] = zero;
    }
  f16x8s v[4], xr[kIB][4][kXPlanes];
  auto load = [&](int t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const f16x8s *>(Vp + (int64_t)t * 2 * kSub * 64 + 8 * (i * 256 + tid));
#pragma unroll
    for (int ib = 0; ib < kIB; ++ib)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        if (kFine) {           // chunks of 32: [32 hi | 32 lo]; the second one of the last 64 may not be there (V is zero there)
          const _Float16 *at = x[ib] + min(2 * t + (ks >> 1), nK32 - 1) * 64 + (ks & 1) * 16;
          xr[ib][ks][0] = *reinterpret_cast<const f16x8s *>(at);
          xr[ib][ks][kXPlanes - 1] = *reinterpret_cast<const f16x8s *>(at + 32);
        } else {
          xr[ib][ks][0] = *reinterpret_cast<const f16x8s *>(x[ib] + t * 64 + 16 * ks);
        }
      }
  };
  // every workgroup starts at another chunk: rows are a power of two apart where dim is one or is padded to one, and workgroups
  // that all read the same columns would queue at the same few memory channels
  const int turn = (int)(tile % nK);
  load(turn);
  for (int t = 0; t < nK; ++t) {
    _Float16 *sv = s_v[t & 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<f16x8s *>(sv + st_off[i]) = v[i];
    f16x8s xc[kIB][4][kXPlanes];
#pragma unroll
    for (int ib = 0; ib < kIB; ++ib)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int pl = 0; pl < kXPlanes; ++pl) xc[ib][ks][pl] = xr[ib][ks][pl];
    if (t + 1 < nK) load(t + 1 + turn < nK ? t + 1 + turn : t + 1 + turn - nK);
    __syncthreads();           // one barrier per chunk: the other stage's readers passed the previous one
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int pl = 1; pl >= 0; --pl)
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb) {
          const int row = pl * kSub + rb * 32 + l32;
          const f16x8s a = *reinterpret_cast<const f16x8s *>(sv + row * 64 + 8 * ((2 * ks + lhi) ^ swz));
#pragma unroll
          for (int ib = 0; ib < kIB; ++ib) {
            acc[rb][ib] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, xc[ib][ks][0], acc[rb][ib], 0, 0, 0);
            if (kFine && pl == 0) acc[rb][ib] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, xc[ib][ks][kXPlanes - 1], acc[rb][ib], 0, 0, 0);
          }
        }
    if (kFine) {               // short chains: their roundings are most of the fine pass's margin
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
        for (int ib = 0; ib < kIB; ++ib) {
          tot[rb][ib] += acc[rb][ib];
          acc[rb][ib] = zero;
        }
    }
  }
  const float wm = state->wm, um = state->u, u1 = state->u1, ulost = state->ulost;
  const float uscale = state->uscale, cscale = state->cscale;
  const bool first32 = state->use == 1;
  // roundings of a coordinate: a chain of 8 nK matrix instructions, or (fine) chains of 12, their sum, and the dropped lo.lo products
  const float chain = kFine ? 2.5f * 12.f + 11.f + (float)nK + 4.f : 2.5f * (float)(8 * nK) + 11.f;
#pragma unroll
  for (int ib = 0; ib < kIB; ++ib) {
    const int64_t j = inst0 + ib * 32 + l32;
    if (kFine) {
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb) acc[rb][ib] = tot[rb][ib];
    }
    float top = 0.f;
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
      for (int i = 0; i < 16; ++i) top = fmaxf(top, fabsf(acc[rb][ib][i]));
    top = fmaxf(top, __shfl_xor(top, 32, 64));
    float inv;
    float s = pow2_over(top, &inv);
    const float xs = (j < n ? xscale[j] : 1.f) * (1.f / kVScale);
    const float cfac = constant_factor(s, inv, xs, uscale, cscale);      // (an instance it does not fit keeps every block)
    float ysq = 0.f, lost = 0.f;
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f16x4s h, l;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float y = acc[rb][ib][4 * g + i] * inv;
          h[i] = (_Float16)y;
          const float d = y - (float)h[i];
          l[i] = (_Float16)d;
          ysq += y * y;
          lost += d * d;
        }
        if (kFine && j < n) {
          _Float16 *at = Y2 + j * 2 * kSub + rb * 64 + 8 * g + 4 * lhi;
          *reinterpret_cast<f16x4s *>(at) = h;
          *reinterpret_cast<f16x4s *>(at + 32) = l;
        }
        if (rb == 0) {                       // coordinates kSubConst .. kSubConst + 2
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 8 * g + 4 * lhi + i;
            if (r >= kSubConst && r < kSubConst + 3) h[i] = (_Float16)cfac;
          }
        }
        if (j < n && (rb == 0 || !first32)) *reinterpret_cast<f16x4s *>(Y1 + j * (first32 ? 32 : 64) + rb * 32 + 8 * g + 4 * lhi) = h;
      }
    ysq += __shfl_xor(ysq, 32, 64);
    lost += __shfl_xor(lost, 32, 64);
    if (j < n && lhi == 0) {
      const float unit = s * xs;
      const float lx = xlost[j], xn = sqrtf(xn32[j]) * (1.f + 1e-6f) + lx;
      const float yn = (sqrtf(ysq) * (1.f + 1e-4f) + 1e-15f) * unit, yl = (sqrtf(lost) * (1.f + 4e-4f) + 1e-15f) * unit;
      yscale[j] = unit;
      // what the planes that were multiplied leave of x', times w', and the roundings of y, times u
      const float left = kFine ? 0x1p-22f * xn + sqrtf((float)dim) * 0x1p-25f * xscale[j] : lx;
      const float b = left * wm + chain * 0x1p-24f * xn * u1;
      // coarse: hi.e_i + (y - hi(y)).u + hi(y).(u - hi(u)) + the coarse pass's chain of up to four instructions, over the
      // products and over half of c_i
      const float b1 = b + xn * state->e + yl * um + (yn + yl) * (ulost + 21.f * 0x1p-24f * um) + 12.f * 0x1p-24f * state->cmax;
      err[j] = factor_fits(cfac) ? b1 * (1.f + 1e-3f) : INFINITY;
      // fine: the residual, what hi + lo leave of y, a chain of 12 instructions, its flush and the dropped products
      if (kFine) err2[j] = (b + xn * state->e64 + (0x1p-22f * yn + 8.f * 0x1p-25f * unit) * um + (42.f + 12.f) * 0x1p-24f * yn * um) * (1.f + 1e-3f);
    }
  }
}

// (three workgroups per CU: 168 registers, 20 bytes spilled once, against 204 and two; 100,000 x 1,000 with the fine pass's planes 123 -> 116 us,
// 1,000,000 x 128 93 -> 82)
__global__ __launch_bounds__(256, 3) void k_subspace_project(const _Float16 *__restrict__ Xh1, const _Float16 *__restrict__ Xh, int64_t n,
                                                          int dim, const _Float16 *__restrict__ Vp, const float *__restrict__ xscale,
                                                          const float *__restrict__ xn32, const float *__restrict__ xlost,
                                                          const SubspaceState *__restrict__ state, _Float16 *__restrict__ Y1,
                                                          _Float16 *__restrict__ Y2, float *__restrict__ yscale,
                                                          float *__restrict__ err, float *__restrict__ err2) {
  __shared__ __attribute__((aligned(16))) _Float16 s_v[2][2 * kSub * 64];
  if (state->fine) project_rows<2, true>(Xh, n, dim, Vp, xscale, xn32, xlost, state, Y1, Y2, yscale, err, err2, s_v, (int64_t)blockIdx.x);
  else if (state->use == 1) project_rows<1, false>(Xh1, n, dim, Vp, xscale, xn32, xlost, state, Y1, Y2, yscale, err, err2, s_v, (int64_t)blockIdx.x);
  else if (state->use == 2) project_rows<2, false>(Xh1, n, dim, Vp, xscale, xn32, xlost, state, Y1, Y2, yscale, err, err2, s_v, (int64_t)blockIdx.x);
}

// ---------------------------------------------------------------- host side
// Is the subspace worth its scratch for searches of n instances?  By default where the coarse pass would take some 150 us
// more on the full rows (2 ns per million multiply-adds) than the basis and the coordinates take (80 us, and the read of the
// hi planes), by whatever name the two-level search is asked for (below that it costs: 5,000 x 100 on 400 nodes, 117 us an epoch
// without and 161 with it, 20,000 x 200 on 1,600 nodes 197 and 226).  Grows with n, so that scratch for the largest call serves every smaller one.
// alone: for a search outside an epoch.  Under the other neighbourhoods a code book has as many directions as nodes.
bool subspace_eligible(const som_ctx *c, int64_t n, bool alone) {
  if (c->dim <= kSub || c->dim > kPlaneMaxDim || c->nb_function != SOM_NEIGHBORHOOD_GAUSSIAN || c->nb_compact) return false;
  return c->sub_always || (double)n * (double)c->k * (double)(c->dim - kSub) >= (alone ? kSubspaceAloneWork : kSubspaceMinWork);
}

// Is the code book likely to lie in 64 directions?  One that enters an epoch was left by an epoch of about its radius
// or more, and the number of directions grows with the number of radii the map is long and wide.  A search
// outside an epoch (radius 0) may bring any: it is tried where the work it may save is several times what a
// failure costs (13 us for 2,500 nodes and 22 for 40,000 where the factor finds out, 75 to 110 where the nodes' losses do).
bool subspace_likely(const som_ctx *c, int64_t n, double radius) {
  if (radius <= 0.0) return subspace_eligible(c, n, true);
  return (double)c->rows * (double)c->cols <= kSubspaceMaxArea * radius * radius;
}

size_t subspace_vector_halves(const som_ctx *c) { return (size_t)((c->dim + 63) / 64) * 64 * 2 * kSub; }

int subspace_gram_pieces(const som_ctx *c) { return ((c->dim + 63) / 64 * 64 + kGramCols - 1) / kGramCols; }

hipError_t launch_subspace_basis(som_ctx *c, const float *W, float loss) {
  const int nK = (c->dim + 63) / 64, dimp = nK * 64, pieces = subspace_gram_pieces(c);
  double *linv = c->sub_G + (size_t)pieces * kSub * kSub;
  if (W) hipLaunchKernelGGL(k_subspace_sketch, dim3(kSub, nK), dim3(512), 0, c->stream, W, c->k, c->dim, dimp, c->mu, c->sub_S);
  hipLaunchKernelGGL(k_subspace_gram, dim3(pieces), dim3(256), 0, c->stream, c->sub_S, dimp, c->sub_G);
  if (pieces > 8) hipLaunchKernelGGL(k_gram_sum, dim3(kSub), dim3(256), 0, c->stream, c->sub_G, pieces);
  hipLaunchKernelGGL(k_subspace_factor, dim3(1), dim3(256), 0, c->stream, c->sub_G, pieces > 8 ? 1 : pieces, loss, linv, c->sub_state);
  hipLaunchKernelGGL(k_subspace_vectors, dim3(nK), dim3(512), 0, c->stream, c->sub_S, dimp, linv, c->sub_state, c->sub_Vp, c->sub_Vt,
                     c->sub_Vf);
  return hipGetLastError();
}

hipError_t launch_subspace(som_ctx *c, const float *W, int64_t n) {
  const hipError_t e = launch_subspace_basis(c, W, kSubspaceLoss);
  if (e != hipSuccess) return e;
  int blocks = (c->k + 31) / 32;
  if (blocks > kSubspaceParts) blocks = kSubspaceParts;
  hipLaunchKernelGGL(k_subspace_coords, dim3(blocks), dim3(512), 0, c->stream, c->Wh, c->k, c->dim, (c->dim + 31) / 32, c->sub_Vp,
                     c->sub_Vt, c->wscale, c->wmax_bits, c->wn32, c->sub_U1, c->sub_U2,
                     c->sub_Y2 != nullptr, c->sub_part, c->list_counts + kSubTicketWord, c->sub_state);
  const int64_t per = c->sub_Y2 ? 128 : 256;      // instances per workgroup (without the fine pass's planes half of 128 leave at once)
  hipLaunchKernelGGL(k_subspace_project, dim3((unsigned)((n + per - 1) / per)), dim3(256), 0, c->stream, c->Xh1, c->Xh, n, c->dim,
                     c->sub_Vp, c->xscale, c->xn32, c->xlost, c->sub_state, c->sub_Y1, c->sub_Y2, c->sub_yscale, c->sub_err,
                     c->sub_err2);
  return hipGetLastError();
}

}  // namespace som
