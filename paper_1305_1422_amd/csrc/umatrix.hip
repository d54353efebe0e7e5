// U-matrix (paper: U-matrix equation): U(j) = mean over the immediate neighbours i of node j of
// the Euclidean distance |w_i - w_j|.  Immediate neighbours are the other nodes at grid distance
// <= 1: up to four on a square grid, up to six on a hexagonal one, fewer on the border of a
// planar map; on a toroid the map wraps.  Distances summed in fp64.
// Bound by the chain of loads where rows are short, by the neighbours' rows out of the caches where they are long; so four neighbours'
// rows stream beside the node's, 512 features of each on the way at a time, and a node is shared by four wavefronts where the map
// does not fill the chip with one each (square map, one neighbour and 64 features at a
// time / now: 50 x 50 nodes of 1,000 features 27 / 12 us, of 50,000 1,419 / 270, 10 x 10 of 50,000 891 / 27).
#include "row_load.hpp"
#include "som_internal.hpp"

#include <math.h>

namespace som {

// kTeam wavefronts of a workgroup of four take a node, kGroup neighbours at a time.  kShort: rows of a few features per lane, taken one by one.
template <int kTeam, int kGroup, bool kShort>
__global__ __launch_bounds__(256) void k_umatrix(const float *__restrict__ W, int rows, int cols, int dim,
                                                 int toroid, int hex, float *__restrict__ U) {
  constexpr int kTeams = 4 / kTeam, kAhead = 2;
  __shared__ double s_part[4][kGroup];
  // (one neighbour at a time: the search for the neighbours is most of it, and faster in vector registers)
  const int lane = threadIdx.x & 63, wave = kGroup == 1 ? (int)threadIdx.x >> 6 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int team = wave / kTeam, part = wave % kTeam;
  const int k = rows * cols;
  for (int j0 = blockIdx.x * kTeams; j0 < k; j0 += gridDim.x * kTeams) {      // (with a team of four j0 is the node: uniform over the workgroup)
    const int j = j0 + team;
    if (j >= k) continue;
    const int yj = j / cols, xj = j - yj * cols;
    int nb[8];
    int cnt = 0;
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        if (dx == 0 && dy == 0) continue;
        int x = xj + dx, y = yj + dy;
        if (toroid) {
          x = (x + cols) % cols;
          y = (y + rows) % rows;
        } else if (x < 0 || x >= cols || y < 0 || y >= rows) {
          continue;
        }
        const int i = y * cols + x;
        if (i == j || grid_q(rows, cols, toroid, hex, x, y, xj, yj) > 4) continue;
        bool seen = false;
        for (int t = 0; t < cnt; ++t) seen |= (nb[t] == i);      // tiny toroids alias offsets
        if (!seen) nb[cnt++] = i;
      }
    double sum = 0.0;
    const float *wj = W + (int64_t)j * dim;
    for (int t0 = 0; t0 < cnt; t0 += kGroup) {
      const float *wi[kGroup];
#pragma unroll
      for (int t = 0; t < kGroup; ++t) wi[t] = W + (int64_t)nb[min(t0 + t, cnt - 1)] * dim;      // (the last one again where there are fewer)
      double s[kGroup] = {};
      if (kShort) {
        for (int c = lane; c < dim; c += kWave) {
          const double a = (double)wj[c];
          float b[kGroup];
#pragma unroll
          for (int t = 0; t < kGroup; ++t) b[t] = wi[t][c];
#pragma unroll
          for (int t = 0; t < kGroup; ++t) {
            const double d = (double)b[t] - a;
            s[t] += d * d;
          }
        }
      } else for (int c0 = 4 * (lane + kWave * part); c0 < dim; c0 += 4 * kWave * kTeam * kAhead) {
        f32x4r a[kAhead], b[kAhead][kGroup];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int c = c0 + u * 4 * kWave * kTeam;
          a[u] = row_load<true>(wj, c, dim);
#pragma unroll
          for (int t = 0; t < kGroup; ++t) b[u][t] = row_load<true>(wi[t], c, dim);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int c = c0 + u * 4 * kWave * kTeam;
          row_tail<true>(a[u], c, dim);
#pragma unroll
          for (int t = 0; t < kGroup; ++t) {
            row_tail<true>(b[u][t], c, dim);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double d = (double)b[u][t][e] - (double)a[u][e];
              s[t] += d * d;
            }
          }
        }
      }
#pragma unroll
      for (int t = 0; t < kGroup; ++t) s[t] = wave_sum(s[t]);
      if (kTeam > 1) {
        if (lane == 0) {
#pragma unroll
          for (int t = 0; t < kGroup; ++t) s_part[wave][t] = s[t];
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < kGroup; ++t) s[t] = (s_part[0][t] + s_part[1][t]) + (s_part[2][t] + s_part[3][t]);
        __syncthreads();
      }
#pragma unroll
      for (int t = 0; t < kGroup; ++t)
        if (t0 + t < cnt) sum += sqrt(s[t]);
    }
    if (lane == 0 && part == 0) U[j] = cnt ? (float)(sum / cnt) : 0.f;
  }
}

template <int kTeam, int kGroup, bool kShort>
static void launch_umatrix_form(som_ctx *c, const float *W, float *U) {
  constexpr int kTeams = 4 / kTeam;
  int blocks = (c->k + kTeams - 1) / kTeams;
  if (blocks > c->n_cu * 16) blocks = c->n_cu * 16;
  hipLaunchKernelGGL((k_umatrix<kTeam, kGroup, kShort>), dim3(blocks), dim3(256), 0, c->stream, W, c->rows, c->cols, c->dim,
                     c->map_type == SOM_MAP_TOROID, c->grid_type == SOM_GRID_HEXAGONAL, U);
}

hipError_t launch_umatrix(som_ctx *c, const float *W, float *U) {
  // Square map, us: short rows, one by one / sixteen bytes a lane: 2,500 nodes of 300 features 9.9 / 10.3, of 500 11.3 / 10.4.  Where several
  // nodes wait for every wavefront, one neighbour at a time has the fewer instructions: 40,000 of 30 65 against 76 four at a time; the
  // line, one / four neighbours at a time, square planar and hexagonal toroid: 3,600 of 30 9.7 / 9.6, 14.2 / 14.0, of 200 11.1 / 10.2, 16.6 / 15.3;
  // 4,356 of 30 10.8 / 11.0, 16.0 / 16.7, of 64 10.8 / 10.9, 15.7 / 16.4, of 200 12.0 / 11.1, 18.3 / 17.6; 6,084 of 30 11.9 / 12.0, 17.9 / 19.1, of 200
  // 13.8 / 13.2, 20.2 / 20.1.  Four wavefronts a node / one: 100 nodes of 50,000 27 / 81, 400 of 20,000 25 / 38, 2,500 of 5,000 40 / 32, 400 of
  // 1,000 9.3 / 8.7.  (Hexagonal toroids of 385 features and more, one neighbour and 64 features / this: 2,500 nodes of 385 16 / 14, of 1,000
  // 38 / 17, of 20,000 613 / 176; 40,000 of 400 128 / 113; 100 of 50,000 1,350 / 47.)
  if (c->dim <= 384 && c->k > (c->dim <= 128 ? 16 : 24) * c->n_cu) launch_umatrix_form<1, 1, true>(c, W, U);
  else if (c->dim <= 384) launch_umatrix_form<1, 4, true>(c, W, U);
  else if (c->k <= 4 * c->n_cu && c->dim >= 4096) launch_umatrix_form<4, 4, false>(c, W, U);
  else launch_umatrix_form<1, 4, false>(c, W, U);
  return hipGetLastError();
}

}  // namespace som
