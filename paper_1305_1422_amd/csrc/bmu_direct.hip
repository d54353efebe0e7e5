// Dense best-matching-unit search for small problems, in double precision from the start (paper: BMU
// equation, ties to the lowest node index).
//
// The filter passes (bmu_dense_h.hip, bmu_coarse.hip) win on large searches, but behind each of them stand a
// dozen launches - centring, planes, block selection, ordering, certification, the exact stage - of 3 to 15
// microseconds each, however small the search.  Up to a size (direct_search_pays) one kernel does it all: the
// scores s_i = |w_i|^2 - 2 x.w_i from v_mfma_f64_16x16x4 on the operands as they are, converted in registers,
// with |w_i|^2 and |x|^2 summed on the way.
//
// A score is off by at most 2^-53 (2 dim + 4)(2 |x| |w| + |w|^2), so where no other node's score comes within
//     tau = 2^-50 (dim + 8)(2 |x| Wmax + Wmax^2)
// of the best one, the best one is the BMU.  Otherwise (equal or nearly equal rows, an instance with a
// non-finite component: tau is then infinite or a NaN, which counts as "within") the tiles are swept once more,
// the nodes within tau are listed, and the plain sums sum_c (x_c - w_c)^2 of those decide, added in the same
// order for every node, so that identical rows tie and the lowest index wins (a list that overflows: the plain
// sums of all nodes; no finite distance at all gives node 0).
//
// A wavefront works on 16 instances and tiles of 16 NT nodes (NT = 4 reads each instance operand once per four
// node operands; NT = 1 where there are too few tiles to occupy the chip).  Output lane (l16, g) holds node l16 of
// a 16-node tile and the instances 4 v + g: minima over nodes stay in the lane until the end.  Rows of up to
// 64 features are kept in registers whole (the instances for the whole sweep, the next tile's nodes while the
// present one is multiplied: kSteps = steps of 16 features); longer ones stream, two steps ahead.
// Sharing out the work: a wavefront per 16 instances sweeps all nodes (many instances), the 8 wavefronts of a
// workgroup share the nodes of 16 instances, or (few instances) the nodes are shared out over grid.y as well,
// long rows over the four wavefronts of a workgroup besides, and a second kernel merges the groups.
#include "row_load.hpp"
#include "som_internal.hpp"

#include <math.h>

namespace som {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kDirectList = 64;       // nodes listed per open instance

// The best score of an instance over a set of nodes, the second best (its value alone), and the largest |w|^2 of
// the set.
struct DirectBest {
  double best, second, wmax;
  int arg;
};

__device__ __forceinline__ DirectBest direct_none() { return DirectBest{INFINITY, INFINITY, 0.0, 0x7fffffff}; }

__device__ __forceinline__ void direct_merge(DirectBest &a, const DirectBest &b) {
  const bool other = b.best < a.best || (b.best == a.best && b.arg < a.arg);
  a.second = fmin(fmin(a.second, b.second), other ? a.best : b.best);
  a.best = other ? b.best : a.best;
  a.arg = other ? b.arg : a.arg;
  a.wmax = fmax(a.wmax, b.wmax);
}

// Data-parallel-primitive moves within rows of 16 lanes (no LDS crossbar): quad_perm [1,0,3,2], [2,3,0,1], half-row
// and row mirror; combining with each in turn leaves the row's total in all 16 lanes.
template <int kCtrl>
__device__ __forceinline__ int direct_dpp(int v) { return __builtin_amdgcn_update_dpp(v, v, kCtrl, 0xf, 0xf, false); }
template <int kCtrl>
__device__ __forceinline__ double direct_dpp(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)direct_dpp<kCtrl>((int)u), hi = (unsigned)direct_dpp<kCtrl>((int)(u >> 32));
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
template <int kCtrl>
__device__ __forceinline__ void direct_row_step(DirectBest &r) {
  const DirectBest b{direct_dpp<kCtrl>(r.best), direct_dpp<kCtrl>(r.second), direct_dpp<kCtrl>(r.wmax), direct_dpp<kCtrl>(r.arg)};
  direct_merge(r, b);
}
__device__ __forceinline__ void direct_row_merge(DirectBest &r) {
  direct_row_step<0xB1>(r);
  direct_row_step<0x4E>(r);
  direct_row_step<0x141>(r);
  direct_row_step<0x140>(r);
}

// Lanes of the set below this one.
__device__ __forceinline__ int lanes_below(unsigned long long set) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(set >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)set, 0u));
}

// A value that is the same in all lanes, in scalar registers.
__device__ __forceinline__ double direct_uniform(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)u), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(u >> 32));
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}

// Scores up to this one may belong to the BMU.
__device__ __forceinline__ double direct_limit(const DirectBest &r, double xn, int dim) {
  return r.best + 8.881784197001252e-16 * (double)(dim + 8) * (2.0 * sqrt(xn) * sqrt(r.wmax) + r.wmax);      // 2^-50
}

__device__ __forceinline__ bool direct_decided(const DirectBest &r, double limit) {
  return r.arg != 0x7fffffff && r.second > limit;          // false on NaNs
}

// Adds the nodes node(lo) .. node(hi - 1) to the lanes' running plain minima.  A node is taken by a team of lanes, four
// features a lane (rows of up to 4 features: a lane per node; beyond 128: the wavefront), four nodes per team at once,
// so that a short row leaves no lanes idle (1,000,000 x 10 on 100 nodes, 20 copies of 5 rows: 3,670 -> 910 us); the additions of a node come in the same order whichever team has it.
template <bool kWide, typename Node>
__device__ __forceinline__ void direct_plain(const float *__restrict__ x, const float *__restrict__ W, int lo, int hi, Node node,
                                             int dim, int lane, double &best, int &arg) {
  int team = 1;
  while (team < kWave && 4 * team < dim) team *= 2;            // uniform
  const int teams = kWave / team, own = lane / team, part = 4 * (lane & (team - 1));
  for (int i = lo; i < hi; i += 4 * teams) {
    int id[4];
    double d2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      id[u] = node(min(i + u * teams + own, hi - 1));
      d2[u] = 0.0;
    }
    for (int c0 = 0; c0 < dim; c0 += 4 * team) {
      const int c = c0 + part;
      f32x4r xv = row_load<kWide>(x, c, dim), wv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) wv[u] = row_load<kWide>(W + (int64_t)id[u] * dim, c, dim);
      row_tail<kWide>(xv, c, dim);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        row_tail<kWide>(wv[u], c, dim);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double d = (double)xv[e] - (double)wv[u][e];
          d2[u] += d * d;
        }
      }
    }
    for (int o = team / 2; o > 0; o >>= 1)
#pragma unroll
      for (int u = 0; u < 4; ++u) d2[u] += __shfl_xor(d2[u], o, kWave);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (nearer(d2[u], id[u], best, arg)) { best = d2[u]; arg = id[u]; }
  }
}

// The minima of 64 lanes as one, in all of them.
__device__ __forceinline__ void direct_plain_merge(double &best, int &arg) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double b = __shfl_xor(best, o, kWave);
    const int a = __shfl_xor(arg, o, kWave);
    if (nearer(b, a, best, arg)) { best = b; arg = a; }
  }
}

// 16 features: lane group g holds features c0 + 4 g .. + 3 of its rows, matrix instruction e takes feature
// c0 + 4 g + e from both operands.
template <int NT>
__device__ __forceinline__ void direct_step(const f32x4r &xs, const f32x4r (&ws)[NT], f64x4 (&acc)[NT], double (&wn)[NT]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const double xd = (double)xs[e];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const double wd = (double)ws[t][e];
      wn[t] = fma(wd, wd, wn[t]);
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd, wd, acc[t], 0, 0, 0);
    }
  }
}

// mask: +inf at nodes that need not be looked at (copies of a lower-indexed node, dedup.hip), or null.
// kShare: 1 = a wavefront per 16 instances; kWaves = the workgroup's wavefronts share the nodes of 16 instances
// (tile by tile); 0 = they share the FEATURES of every tile (long rows).  kSteps: rows of up to 16 kSteps features
// held in registers, 0 = longer rows.
// grid = (instance tiles / (kShare == 1 ? kWaves : 1), groups); with one group the BMUs are written, else a record per
// (group, instance).
template <int kWaves, int kShare, int NT, int kSteps, bool kWide>
__global__ __launch_bounds__(64 * kWaves) void k_direct_search(const float *__restrict__ X, int64_t n,
                                                               const float *__restrict__ W, int k, int dim,
                                                               const float *__restrict__ mask, int tiles_per_group,
                                                               int32_t *__restrict__ bmus,
                                                               DirectBest *__restrict__ rec, double *__restrict__ xn_out,
                                                               int32_t *__restrict__ list_counts) {
  static_assert(kShare == 0 || kShare == 1 || kShare == kWaves, "a tile belongs to one wavefront or to the whole workgroup");
  constexpr bool kOwn = kShare == 1, kSplit = kShare == 0;
  constexpr int kTeams = kOwn ? kWaves : 1;      // instance tiles per workgroup
  __shared__ DirectBest s_rec[kWaves][16];
  __shared__ double s_lim[kTeams][16];
  __shared__ int s_cnt[kTeams][16], s_list[kTeams][16][kDirectList];
  __shared__ f64x4 s_acc[kSplit ? kWaves : 1][kSplit ? NT : 1][kSplit ? 64 : 1];
  __shared__ double s_wn[kSplit ? kWaves : 1][kSplit ? NT : 1][kSplit ? 64 : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int team = kOwn ? wave : 0;
  const int l16 = lane & 15, g = lane >> 4;
  const int64_t j0 = ((int64_t)blockIdx.x * kTeams + team) * 16;
  if (j0 >= n) return;               // uniform over the workgroup, or (kOwn) without barriers below
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 3) list_counts[threadIdx.x] = 0;      // nothing for the exact stage
  const float *xr = X + (j0 + l16 < n ? j0 + l16 : n - 1) * dim;
  const int ntiles = (k + 16 * NT - 1) / (16 * NT);
  const int t0 = blockIdx.y * tiles_per_group;
  const int t1 = min(t0 + tiles_per_group, ntiles);
  const int first = kShare == kWaves && !kOwn ? t0 + wave : t0;
  constexpr int kStride = kShare == kWaves && !kOwn ? kWaves : 1;

  // |x|^2 of instance l16, and the instances themselves if their rows are short
  constexpr int kHold = kSteps > 0 ? kSteps : 1;
  f32x4r xs[kHold];
  double xn = 0.0;
  if (kSteps > 0) {
#pragma unroll
    for (int a = 0; a < kSteps; ++a) {
      xs[a] = row_load<kWide>(xr, 16 * a + 4 * g, dim);
      row_tail<kWide>(xs[a], 16 * a + 4 * g, dim);
#pragma unroll
      for (int e = 0; e < 4; ++e) xn = fma((double)xs[a][e], (double)xs[a][e], xn);
    }
  }
  // the part of the features this wavefront multiplies
  const int steps = (dim + 15) / 16;
  const int per_wave = kSplit ? (steps + kWaves - 1) / kWaves : steps;
  const int c_lo = kSplit ? 16 * per_wave * wave : 0;
  const int c_hi = kSplit ? min(c_lo + 16 * per_wave, dim) : dim;

  double best[4], second[4], limit[4];
  int arg[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) { best[v] = second[v] = INFINITY; limit[v] = 0.0; arg[v] = 0x7fffffff; }
  double wmax = 0.0;
  // The scores of one 16-node tile: into the minima, or (second sweep) the nodes within the limit into the lists.
  auto consume = [&](bool collect, int node, const f64x4 &acc, double wn) {
    const bool out = node >= k || (mask && mask[min(node, k - 1)] == INFINITY);
    if (!collect) {
      const double w2 = out ? INFINITY : wn;
      wmax = fmax(wmax, out ? 0.0 : wn);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double s = fma(-2.0, acc[v], w2);
        second[v] = fmin(second[v], fmax(best[v], s));      // (a NaN score is no candidate; behind a finite one it leaves the instance open)
        arg[v] = s < best[v] ? node : arg[v];
        best[v] = fmin(best[v], s);
      }
    } else if (!out) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double s = fma(-2.0, acc[v], wn);
        if (!(s > limit[v])) {                 // -inf at decided instances; a NaN lists the node
          const int at = atomicAdd(&s_cnt[team][4 * v + g], 1);
          if (at < kDirectList) s_list[team][4 * v + g][at] = node;
        }
      }
    }
  };
  auto sweep = [&](bool collect) {
    f32x4r wv[2][kHold][NT];
    auto row_of = [&](int tile, int t) { return W + (int64_t)min(tile * 16 * NT + 16 * t + l16, k - 1) * dim; };
    auto load_tile = [&](f32x4r (&dst)[kHold][NT], int tile) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float *wr = row_of(tile, t);
#pragma unroll
        for (int a = 0; a < kHold; ++a) dst[a][t] = row_load<kWide>(wr, 16 * a + 4 * g, dim);
      }
    };
    if (kSteps > 0 && first < t1) load_tile(wv[0], first);
    for (int tile = first; tile < t1; tile += kStride) {
      f64x4 acc[NT];
      double wn[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) { acc[t] = f64x4{0.0, 0.0, 0.0, 0.0}; wn[t] = 0.0; }
      if (kSteps > 0) {
        load_tile(wv[1], tile + kStride);      // (past the last tile: the last rows again)
#pragma unroll
        for (int a = 0; a < kSteps; ++a) {
          if (16 * a + 16 > dim)               // uniform
#pragma unroll
            for (int t = 0; t < NT; ++t) row_tail<kWide>(wv[0][a][t], 16 * a + 4 * g, dim);
          direct_step<NT>(xs[a], wv[0][a], acc, wn);
        }
      } else {
        f32x4r xa[2], wa[2][NT];
        const float *wr[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) wr[t] = row_of(tile, t);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          xa[b] = row_load<kWide>(xr, c_lo + 16 * b + 4 * g, dim);
#pragma unroll
          for (int t = 0; t < NT; ++t) wa[b][t] = row_load<kWide>(wr[t], c_lo + 16 * b + 4 * g, dim);
        }
        xn = 0.0;
        for (int c0 = c_lo; c0 < c_hi; c0 += 32) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            f32x4r x1 = xa[b], w1[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) w1[t] = wa[b][t];
            const int c = c0 + 16 * b + 4 * g;
            xa[b] = row_load<kWide>(xr, c + 32, dim);
#pragma unroll
            for (int t = 0; t < NT; ++t) wa[b][t] = row_load<kWide>(wr[t], c + 32, dim);
            if (c0 + 16 * b + 16 > dim) {        // uniform
              row_tail<kWide>(x1, c, dim);
#pragma unroll
              for (int t = 0; t < NT; ++t) row_tail<kWide>(w1[t], c, dim);
            }
            if (kSplit && c0 + 16 * b >= c_hi) {      // an odd number of steps: the next wavefront's features
              x1 = f32x4r{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int t = 0; t < NT; ++t) w1[t] = f32x4r{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) xn = fma((double)x1[e], (double)x1[e], xn);
            direct_step<NT>(x1, w1, acc, wn);
          }
        }
      }
      if (kSplit) {
        // wavefront t adds up the four parts of 16-node tile t
        static_assert(!kSplit || NT == kWaves, "a 16-node tile per wavefront");
#pragma unroll
        for (int t = 0; t < NT; ++t) { s_acc[wave][t][lane] = acc[t]; s_wn[wave][t][lane] = wn[t]; }
        __syncthreads();
        f64x4 a = s_acc[0][wave][lane];
        double w2 = s_wn[0][wave][lane];
#pragma unroll
        for (int v = 1; v < kWaves; ++v) { a += s_acc[v][wave][lane]; w2 += s_wn[v][wave][lane]; }
        __syncthreads();
        w2 += __shfl_xor(w2, 16, kWave);
        w2 += __shfl_xor(w2, 32, kWave);
        consume(collect, tile * 16 * NT + 16 * wave + l16, a, w2);
      } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          wn[t] += __shfl_xor(wn[t], 16, kWave);
          wn[t] += __shfl_xor(wn[t], 32, kWave);
          consume(collect, tile * 16 * NT + 16 * t + l16, acc[t], wn[t]);
        }
      }
      if (kSteps > 0) {
#pragma unroll
        for (int a = 0; a < kHold; ++a)
#pragma unroll
          for (int t = 0; t < NT; ++t) wv[0][a][t] = wv[1][a][t];
      }
    }
  };

  sweep(false);
  // over the 16 lanes of a group; the record of instance 4 v + g is the same in all of them
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    DirectBest q{best[v], second[v], wmax, arg[v]};
    direct_row_merge(q);
    if (l16 == v) s_rec[wave][4 * v + g] = q;
  }
  xn += __shfl_xor(xn, 16, kWave);
  xn += __shfl_xor(xn, 32, kWave);
  if (kSplit) {
    if (g == 0) s_wn[wave][0][l16] = xn;
    __syncthreads();
    xn = 0.0;
    for (int v = 0; v < kWaves; ++v) xn += s_wn[v][0][l16];
  } else if (kOwn) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  } else {
    __syncthreads();
  }
  DirectBest r = s_rec[kOwn ? wave : 0][l16];
  if (!kOwn)
    for (int v = 1; v < kWaves; ++v) direct_merge(r, s_rec[v][l16]);
  if (rec) {
    if (threadIdx.x < 16 && j0 + l16 < n) {
      rec[(int64_t)blockIdx.y * n + j0 + l16] = r;
      if (blockIdx.y == 0) xn_out[j0 + l16] = xn;
    }
    return;
  }
  const bool leader = kOwn || wave == 0;
  if (!kOwn && !kSplit && kSteps == 0) {       // only a wavefront that had a tile knows |x|^2: wavefront 0 has one
    if (wave == 0 && g == 0) s_lim[0][l16] = xn;
    __syncthreads();
    xn = s_lim[0][l16];
    __syncthreads();
  }
  const double lim = direct_limit(r, xn, dim);
  const bool live = j0 + l16 < n;
  const bool is_open = live && !direct_decided(r, lim);
  if (leader && g == 0 && live && !is_open) bmus[j0 + l16] = r.arg;
  unsigned long long open = __ballot(is_open) & 0xffffull;
  if (!open) return;                            // uniform: every wavefront of the workgroup holds the same records
  if (leader && g == 0) { s_lim[team][l16] = is_open ? lim : -INFINITY; s_cnt[team][l16] = 0; }
  if (kOwn) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); else __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) limit[v] = s_lim[team][4 * v + g];
  sweep(true);
  if (kOwn) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); else __syncthreads();
  for (int turn = 0; open; open &= open - 1, ++turn) {
    if (!kOwn && turn % kWaves != wave) continue;
    const int q = __ffsll((long long)open) - 1;
    const int cnt = __builtin_amdgcn_readfirstlane(s_cnt[team][q]);
    double b = INFINITY;
    int a = 0x7fffffff;
    const int *listed = &s_list[team][q][0];
    if (cnt <= kDirectList) direct_plain<kWide>(X + (j0 + q) * dim, W, 0, cnt, [&](int p) { return listed[p]; }, dim, lane, b, a);
    else direct_plain<kWide>(X + (j0 + q) * dim, W, 0, k, [](int p) { return p; }, dim, lane, b, a);
    direct_plain_merge(b, a);
    if (lane == 0) bmus[j0 + q] = a == 0x7fffffff ? 0 : a;
  }
}

// Merges the groups' records.  A wavefront per instance merges them, a lane per record; the instances they leave open are
// then decided by the whole workgroup, by plain distances: of a group's best node alone where only
// that one is inside the limit, else of all nodes of the group.  What bounds that is the latency of one load after the
// other, so the nodes of all groups in question are shared out evenly over the wavefronts, and a workgroup
// takes no more instances than two workgroups per CU leave it (per_block <= 16); where several are open, up to four at a
// time, since sixteen wavefronts on one spend a good part on their meetings (5,000 x 256 on 400 equal nodes: 473 us one at a
// time, 438 so).  Measured, search and merge, a wavefront
// per open instance from 1,024 instances on and 64 nodes one after the other / as it is now: 5,000 x 20 on a trained map
// of 2,500 nodes 162 / 52 us, 1,500 x 20 on 2,500 nodes of which each has 19 exact copies 677 / 80.
// With nothing open it is a launch of 2 to 3 us: the open ones come from one read, and 64 registers let two workgroups
// share a CU (4,097 x 33 on 1,073 nodes, the whole search: 31.7 us with more registers and a look at each instance, 30.2).
constexpr int kMergeWaves = 16;      // 2^4

template <bool kWide>
__global__ __launch_bounds__(64 * kMergeWaves, kWide ? 8 : 4) void k_direct_merge(const DirectBest *__restrict__ rec, const double *__restrict__ xn,
                                                                   int groups, int nodes_per_group, int per_block,
                                                                   const float *__restrict__ X, int64_t n,
                                                                   const float *__restrict__ W, int k, int dim,
                                                                   int32_t *__restrict__ bmus) {
  __shared__ double s_limit[kMergeWaves], s_d2[kMergeWaves];
  __shared__ int s_open[kMergeWaves], s_id[kMergeWaves], s_one[4][kWave], s_first[4][kWave];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t j0 = (int64_t)blockIdx.x * per_block;
  if (wave < per_block && j0 + wave < n) {
    const int64_t j = j0 + wave;
    DirectBest r = direct_none();
    for (int v = lane; v < groups; v += kWave) direct_merge(r, rec[(int64_t)v * n + j]);
    direct_row_merge(r);
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const DirectBest b{__shfl_xor(r.best, o, kWave), __shfl_xor(r.second, o, kWave), __shfl_xor(r.wmax, o, kWave),
                         __shfl_xor(r.arg, o, kWave)};
      direct_merge(r, b);
    }
    const double limit = direct_limit(r, xn[j], dim);
    const bool decided = direct_decided(r, limit);
    if (lane == 0) {
      s_open[wave] = !decided;
      s_limit[wave] = limit;
      if (decided) bmus[j] = r.arg;
    }
  } else if (lane == 0) {
    s_open[wave] = 0;
  }
  __syncthreads();
  // (one read for all of them; uniform)
  unsigned long long open = __ballot(lane < per_block && s_open[lane & (kMergeWaves - 1)]);
  while (open) {
    // one, two or four instances at once, the wavefronts in as many crews
    const int left = __popcll(open), halvings = left >= 4 ? 2 : left >= 2 ? 1 : 0, hands = kMergeWaves >> halvings;
    const int crew = wave >> (4 - halvings), hand = wave & (hands - 1);
    int q = 0;
    for (int t = 0; t < 1 << halvings; ++t, open &= open - 1)
      if (t == crew) q = __ffsll((long long)open) - 1;       // (crews never outnumber the instances left)
    const int64_t j = j0 + q;
    const double limit = direct_uniform(s_limit[q]);
    double b = INFINITY;
    int a = 0x7fffffff;
    for (int v0 = 0; v0 < groups; v0 += kWave) {
      const int v = v0 + lane;
      const DirectBest r = v < groups ? rec[(int64_t)v * n + j] : direct_none();
      const bool kept = v < groups && !(r.best > limit);            // (a NaN limit keeps every group)
      const bool one = kept && r.second > limit && (unsigned)r.arg < (unsigned)k;
      const unsigned long long ones = __ballot(one), whole = __ballot(kept && !one);
      int *s_ones = s_one[crew], *s_firsts = s_first[crew];
      if (hand == 0) {
        if (one) s_ones[lanes_below(ones)] = r.arg;
        else if (kept) s_firsts[lanes_below(whole)] = v * nodes_per_group;
      }
      __syncthreads();
      const int singles = __popcll(ones), total = singles + __popcll(whole) * nodes_per_group;
      const int share = (total + hands - 1) >> (4 - halvings), at = hand * share;
      direct_plain<kWide>(X + j * dim, W, at, min(at + share, total), [&](int p) {
        if (p < singles) return s_ones[p];
        const int g = (p - singles) / nodes_per_group;
        return min(s_firsts[g] + (p - singles) - g * nodes_per_group, k - 1);      // (the last group may be short)
      }, dim, lane, b, a);
      __syncthreads();
    }
    direct_plain_merge(b, a);
    if (lane == 0) { s_d2[wave] = b; s_id[wave] = a; }
    __syncthreads();
    if (hand == 0) {
      b = lane < hands ? s_d2[wave + lane] : INFINITY;
      a = lane < hands ? s_id[wave + lane] : 0x7fffffff;
      direct_plain_merge(b, a);
      if (lane == 0) bmus[j] = a == 0x7fffffff ? 0 : a;
    }
    __syncthreads();
  }
}

struct DirectPlan {
  int share;          // kShare of k_direct_search
  int nt, tiles, groups, per_group;
};

// Launch geometry (see the head of the file).
static DirectPlan direct_plan(const som_ctx *c, int64_t n) {
  DirectPlan p;
  const int64_t nt16 = (n + 15) / 16;
  const int64_t tiles16 = ((int64_t)c->k + 15) / 16;
  const int64_t steps = (c->dim + 15) / 16;
  const int64_t cu = c->n_cu;
  p.nt = nt16 * tiles16 >= 32 * cu ? 4 : 1;
  p.groups = 1;
  p.share = 8;
  if (nt16 >= 16 * cu) {                 // four wavefronts per SIMD with an instance tile each
    p.share = 1;
  } else {
    // in units of one (16 x 16 x 16)-step on a SIMD (0.23 us with the conversions and the minima); a second launch
    // costs about 22 of them.  Eight wavefronts per workgroup are two per SIMD, one workgroup per CU.
    const int64_t rounds = (nt16 + cu - 1) / cu;
    const int64_t tiles = (tiles16 + p.nt - 1) / p.nt;
    const int64_t single = rounds * 2 * ((tiles + 7) / 8) * p.nt * steps;
    const int64_t spread = nt16 * tiles16 * steps / (4 * cu) * 6 / 5 + p.nt * steps + 22;
    if (single > spread) {
      p.share = c->dim >= 512 ? 0 : 4;          // (the exchange between the wavefronts costs about eight steps)
      if (p.share == 0) p.nt = 4;
    }
  }
  p.tiles = (int)((c->k + 16 * p.nt - 1) / (16 * p.nt));
  p.per_group = p.tiles;
  if (p.share == 0 || p.share == 4) {
    const int unit = p.share == 4 ? 4 : 1;          // tiles a workgroup takes at once
    int64_t want = (5 * cu + nt16 - 1) / nt16;      // five workgroups per CU
    const int most = (p.tiles + unit - 1) / unit;
    if (want > most) want = most;
    if (want < 1) want = 1;
    p.per_group = (int)((p.tiles + want - 1) / want);
    p.per_group = (p.per_group + unit - 1) / unit * unit;
    p.groups = (p.tiles + p.per_group - 1) / p.per_group;
  }
  return p;
}

// Where the direct search wins: estimates of both searches in microseconds, fitted to timings over maps of 100 to 40,000
// nodes, rows of 10 to 1,000 features and 64 to 4,000,000 instances (unordered and trained code books, and such of
// which every row has 19 copies).
// Direct, in (16 x 16 x 16)-steps per SIMD, by the ways of sharing out: 0.2 a step, and besides what a wavefront waits
// for between its tiles.  Where groups are merged, 1.45 times that, for the plain distances of open instances there: a
// trained map leaves up to a third of them open (1,500 x 100 on 2,500 nodes: unordered 39, trained 60, all rows copied
// 252 against 124 / 167 / 164 filtered).  The second sweep of the other forms needs no such allowance, since the
// filtered search's exact stage grows by as much on such maps (12,000 x 64 on 400 nodes: 50 / 49 / 96 against
// 62 / 92 / 123).
static double direct_search_us(const som_ctx *c, int64_t n) {
  const DirectPlan p = direct_plan(c, n);
  const double nt16 = (double)((n + 15) / 16), steps = (double)((c->dim + 15) / 16), cu = (double)c->n_cu;
  const double row = (double)p.nt * steps;               // steps of a tile of nodes with 16 instances
  if (p.share == 1)                                      // (and the instances' rows, read once)
    return 4.0 + nt16 / cu * 0.256 * (0.21 * p.tiles * row + 0.5 + 0.8 * fmin(steps, 4.0));
  if (p.share == 8)
    return 6.0 + fmax(nt16 / cu, 1.0) * (0.44 * ((p.tiles + 7) / 8) * row + (p.nt == 1 ? 1.7 : c->dim <= 64 ? 2.0 * steps : 0.0));
  if (p.share == 4)                                      // whole turns of four tiles
    return (p.groups > 1 ? 1.45 : 1.0) * (11.0 + (p.groups > 1 ? 0.26 : 0.36) * nt16 * ((p.tiles + 3) / 4 * 4) * row / (4.0 * cu));
  return 1.45 * (14.0 + 0.21 * nt16 * p.tiles * row / (4.0 * cu));
}

// Filtered, on an unordered code book (a trained one costs up to half as much again): launches, the code book's planes,
// per instance the exact stage and the matrix work; instances that are not registered bring their own planes.
static double filtered_search_us(const som_ctx *c, int64_t n, bool registered) {
  const double k = (double)c->k, dim = (double)c->dim;
  const bool two_level = (c->k + 127) / 128 >= kTwoLevelMinBlocks;
  double fixed = (two_level ? 84.0 : 40.0 + 0.004 * k) + 0.02 * dim + 2e-5 * k * dim;
  double each = two_level ? 0.3e-6 * k + 0.5e-8 * k * dim : 0.04e-3 + 0.6e-6 * k + 0.6e-8 * k * dim;
  if (!registered) {
    fixed += 9.0;
    each += 0.08e-3 + 1.5e-6 * dim;
  }
  return fixed + each * (double)n;
}

// The line lies where the two meet on an unordered code book, and 15 % beyond, since most maps are ordered ones.
// Direct / filtered on both sides of it, registered, unordered: 12,000 x 64 on 400 nodes 50 / 48, 20,000 x 64 77 / 55;
// 70,000 x 64 on 100 nodes 51 / 53, 150,000 x 64 105 / 65, 1,000,000 x 64 648 / 198; 400,000 x 16 on 400 nodes 174 / 182,
// 1,000,000 x 16 413 / 318; 12,000 x 20 on 2,500 nodes 67 / 116, 35,000 x 20 195 / 156.
bool direct_search_pays(const som_ctx *c, int64_t n, bool registered) {
  return direct_search_us(c, n) <= 1.15 * filtered_search_us(c, n, registered);
}

// Room for the records of any number of instances, so that no call has to grow it: there are groups for fewer than 5 cu
// instance tiles, no more of them than (5 cu - 1) / tiles + 1 nor than quarters of the tiles of 16 nodes (1.5 MB on 256
// CUs at most).
size_t direct_record_doubles(const som_ctx *c) {
  const size_t cu = (size_t)c->n_cu, most = (((size_t)c->k + 15) / 16 + 3) / 4;
  if (most < 2) return 1;
  const size_t tiles = 10 * cu < 5 * cu * most ? 10 * cu : 5 * cu * most;
  return 16 * (tiles * (sizeof(DirectBest) / sizeof(double)) + 5 * cu);
}

hipError_t launch_direct_search(som_ctx *c, const float *X, int64_t n, const float *W, const float *mask, int32_t *bmus) {
  const DirectPlan p = direct_plan(c, n);
  const unsigned nt16 = (unsigned)((n + 15) / 16);
  const unsigned gx = p.share == 1 ? (nt16 + 3) / 4 : nt16;
  DirectBest *rec = p.groups > 1 ? reinterpret_cast<DirectBest *>(c->direct_rec) : nullptr;
  double *xn = p.groups > 1 ? reinterpret_cast<double *>(rec + (size_t)p.groups * (size_t)n) : nullptr;      // behind them
  const int held = c->dim <= 64 ? (c->dim + 15) / 16 : 0;      // steps of 16 features kept in registers
#define SOM_DIRECT(WV, SH, NTV, ST, WIDE)                                                                             \
  hipLaunchKernelGGL((k_direct_search<WV, SH, NTV, ST, WIDE>), dim3(gx, (unsigned)p.groups), dim3(64 * WV), 0, c->stream, \
                     X, n, W, c->k, c->dim, mask, p.per_group, bmus, rec, xn, c->list_counts)
#define SOM_DIRECT_HELD(WV, SH, NTV)                \
  switch (held) {                                   \
    case 0: SOM_DIRECT(WV, SH, NTV, 0, true); break; \
    case 1:                                         \
      if (c->dim >= 4) SOM_DIRECT(WV, SH, NTV, 1, true); \
      else SOM_DIRECT(WV, SH, NTV, 1, false);       \
      break;                                        \
    case 2: SOM_DIRECT(WV, SH, NTV, 2, true); break; \
    case 3: SOM_DIRECT(WV, SH, NTV, 3, true); break; \
    default: SOM_DIRECT(WV, SH, NTV, 4, true);      \
  }
  if (p.share == 0) SOM_DIRECT(4, 0, 4, 0, true);
  else if (p.share == 1) { if (p.nt == 4) SOM_DIRECT_HELD(4, 1, 4) else SOM_DIRECT_HELD(4, 1, 1) }
  else if (p.share == 8) { if (p.nt == 4) SOM_DIRECT_HELD(8, 8, 4) else SOM_DIRECT_HELD(8, 8, 1) }
  else { if (p.nt == 4) SOM_DIRECT_HELD(4, 4, 4) else SOM_DIRECT_HELD(4, 4, 1) }
#undef SOM_DIRECT_HELD
#undef SOM_DIRECT
  if (p.groups > 1) {
    int64_t per_block = (n + 2 * (int64_t)c->n_cu - 1) / (2 * (int64_t)c->n_cu);
    if (per_block > kMergeWaves) per_block = kMergeWaves;
    const dim3 grid((unsigned)((n + per_block - 1) / per_block));
    if (c->dim >= 4)
      hipLaunchKernelGGL(k_direct_merge<true>, grid, dim3(64 * kMergeWaves), 0, c->stream, rec, xn, p.groups,
                         p.per_group * 16 * p.nt, (int)per_block, X, n, W, c->k, c->dim, bmus);
    else
      hipLaunchKernelGGL(k_direct_merge<false>, grid, dim3(64 * kMergeWaves), 0, c->stream, rec, xn, p.groups,
                         p.per_group * 16 * p.nt, (int)per_block, X, n, W, c->k, c->dim, bmus);
  }
  return hipGetLastError();
}

}  // namespace som
