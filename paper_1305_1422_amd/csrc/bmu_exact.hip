// Exact stage of the best-matching-unit search (paper: BMU equation, d = Euclidean distance).
//
// The fp32 pass leaves, per instance, a few candidate nodes with their scores
// s = |w'|^2 - 2 x'.w' (x' = x - mu, w' = w - mu) and the smallest score it dropped.  Here:
//   certify  - bounds the rounding error of those scores; an instance whose best score beats
//              everything else by more than twice the bound is decided on the spot;
//   refine   - otherwise the candidates inside the bound are compared by their squared
//              distances sum_c (x_c - w_c)^2 evaluated in fp64 on the original (uncentred)
//              vectors, lowest node index on exact ties (sparse rows: a regrouped sum over the
//              nonzeros, and the plain sum over all coordinates where that one would cancel);
//   collect  - if a dropped score lies inside the bound too, the fp32 sweep is repeated for
//              that instance and every node under the threshold is listed (bmu_dense.hip),
//              then the list is compared exactly;
//   rescan   - if even that list overflows, all nodes are compared exactly.
// The instance lists are built with atomic counters, so their order varies between runs;
// every instance is decided independently, so the BMUs do not.
//
// (The split-fp16 pass multiplies centred instances x' = fl(x - mu): there X = |x'| and the terms in M
// fall away.)
// Error bound of one dense fp32 score s = c_i - 2 x.w'_i (u = 2^-24, g = roundings a product term
// can suffer, X = |x|, M = |mu|, Wm = max |w'| over the nodes, w' = fl(w - mu)):
//   |s_fp32 - s_exact| <= u [ (2 g + 4) X Wm + 4 Wm^2 + 6 M Wm ]
// made of: the dot product, g u sum|x_c w'_c| <= g u X Wm, doubled by the factor -2; the rounding
// of the stored c_i, u (Wm^2 + 2 M Wm); the final multiply-add, u (Wm^2 + 2 M Wm + 2 X Wm); and the
// rounding of w - mu itself, which moves a squared distance by at most 2 u (X + M + Wm) Wm.
// MFMA pass with two-level accumulation: g = block + ceil(dim / block) + 2.
// Sparse scores |w|^2 - 2 x.w from an FMA chain of len terms, no centring: g = len,
//   |s_fp32 - s_exact| <= u [ (2 g + 2) X Wm + 2 Wm^2 ].
#include "margin.hpp"
#include "row_load.hpp"

namespace som {

// `groups` candidate lists per instance (one per node group of the fp32 pass), stored
// [group][instance][kCand]; the kept candidates are written back into group 0's slots.
__global__ __launch_bounds__(256) void k_certify(CandView cand, int groups, const float *__restrict__ xn32,
                                                 const unsigned *__restrict__ wmax_bits,
                                                 const float *__restrict__ mu_norm2, MarginModel mm, int64_t n, int k,
                                                 int32_t *__restrict__ bmus, int32_t *__restrict__ cand_n,
                                                 int32_t *__restrict__ refine_list,
                                                 int32_t *__restrict__ collect_rows,
                                                 float *__restrict__ collect_thr,
                                                 int32_t *__restrict__ collect_cnt,
                                                 int32_t *__restrict__ list_counts, UnitWork work,
                                                 const int32_t *__restrict__ order,
                                                 const SubspaceState *__restrict__ state, int runs_if) {
  if (state && (state->use != 0) != (runs_if != 0)) return;
  // with `order` the instances are visited in that order, so that neighbours in it are appended to the
  // lists together: the second sweep's tiles then hold instances with similar block sets (two-level
  // search).  List slots are reserved per workgroup - one atomic per list and workgroup, the positions
  // inside from ballots - because a million instances' worth of wavefront-wide atomics on one counter
  // (16,000 of them) were what this kernel spent its time on.
  __shared__ int s_wave_cnt[2][4], s_base[2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = p < n;
  const int64_t j = live ? (order ? (int64_t)order[p] : p) : 0;
  static_assert(kCand == 4, "the candidate lists are read as 16-byte vectors");
  const float4 *val4 = reinterpret_cast<const float4 *>(cand.val);
  const int4 *idx4 = reinterpret_cast<const int4 *>(cand.idx);
  float smin = INFINITY, omin = INFINITY;
  double thr = 0.0;
  int keep[kCand] = {0, 0, 0, 0};
  int cnt = 0;
  if (live) {
    // the lists of kBatch groups, and what the margin is made of, in flight together: one at a time, the chain of their
    // latencies was the kernel (1,000,000 instances of 8 groups 106 -> 77 us, 100,000 18 -> 14.7; 12,347 of 72 groups 241 -> 172); the last list is read again where fewer are left
    constexpr int kBatch = 4;
    float4 v4[kBatch];
    int4 id4[kBatch];
    float over[kBatch];
    auto load = [&](int q0) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int64_t at = (int64_t)min(q0 + u, groups - 1) * n + j;
        v4[u] = val4[at];
        id4[u] = idx4[at];
        over[u] = cand.over[at];
      }
    };
    load(0);
    const double margin = score_margin(mm, j, (double)xn32[j], (double)__uint_as_float(*wmax_bits), (double)*mu_norm2);
    for (int q0 = 0; q0 < groups; q0 += kBatch) {
      if (q0) load(q0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if ((unsigned)id4[u].x < (unsigned)k) smin = fminf(smin, v4[u].x);
        if ((unsigned)id4[u].y < (unsigned)k) smin = fminf(smin, v4[u].y);
        if ((unsigned)id4[u].z < (unsigned)k) smin = fminf(smin, v4[u].z);
        if ((unsigned)id4[u].w < (unsigned)k) smin = fminf(smin, v4[u].w);
        omin = fminf(omin, over[u]);
      }
    }
    thr = (double)smin + margin;
    for (int q0 = 0; q0 < groups; q0 += kBatch) {
      if (groups > kBatch) load(q0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const float v[kCand] = {v4[u].x, v4[u].y, v4[u].z, v4[u].w};
        const int id[kCand] = {id4[u].x, id4[u].y, id4[u].z, id4[u].w};
#pragma unroll
        for (int t = 0; t < kCand; ++t) {
          if (q0 + u < groups && (unsigned)id[t] < (unsigned)k && (double)v[t] <= thr) {
            if (cnt < kCand) keep[cnt] = id[t];
            ++cnt;
          }
        }
      }
    }
  }
  const bool overflow = (double)omin <= thr || cnt > kCand;
  const bool to_collect = live && (overflow || cnt == 0);
  const bool to_refine = live && !to_collect && cnt > 1;
  // slots: [0] refine list, [1] collect list
  const unsigned long long bal_r = __ballot(to_refine), bal_c = __ballot(to_collect);
  if (lane == 0) {
    s_wave_cnt[0][wave] = __popcll(bal_r);
    s_wave_cnt[1][wave] = __popcll(bal_c);
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int total = s_wave_cnt[threadIdx.x][0] + s_wave_cnt[threadIdx.x][1] + s_wave_cnt[threadIdx.x][2] +
                      s_wave_cnt[threadIdx.x][3];
    s_base[threadIdx.x] = total ? atomicAdd(&list_counts[threadIdx.x], total) : 0;
  }
  __syncthreads();
  const unsigned long long below = (1ull << lane) - 1ull;
  int before_r = s_base[0], before_c = s_base[1];
  for (int w = 0; w < wave; ++w) {
    before_r += s_wave_cnt[0][w];
    before_c += s_wave_cnt[1][w];
  }
  if (to_collect) {
    const int slot = before_c + __popcll(bal_c & below);
    collect_rows[slot] = (int32_t)j;
    float t32 = (float)thr;                     // round the threshold up: no score inside the margin is lost
    if ((double)t32 < thr) t32 = nextafterf(t32, INFINITY);
    collect_thr[slot] = cnt == 0 ? INFINITY : t32;
    int filled = 0;
    if (work.sweeps > 0) {
      // sparse search: only the node ranges whose third-best score is inside the threshold have to be
      // swept again; the others are known completely through their two best nodes, listed here
      const double lim = cnt == 0 ? (double)INFINITY : thr;
      for (int q = 0; q < groups; ++q) {
        if ((double)cand.over[(int64_t)q * n + j] <= lim) {
          const int slice = q / work.sweeps;
          const int pos = atomicAdd(&work.counts[slice], 1);
          work.units[(int64_t)slice * work.cap + pos] = (int64_t)slot * work.sweeps + (q - slice * work.sweeps);
        } else {
          const int64_t base = ((int64_t)q * n + j) * kCand;
#pragma unroll
          for (int t = 0; t < kCand; ++t) {
            const int id = cand.idx[base + t];
            if ((unsigned)id < (unsigned)k && (double)cand.val[base + t] <= lim) {
              if (filled < kListCap) work.list[(int64_t)slot * kListCap + filled] = id;
              ++filled;
            }
          }
        }
      }
    }
    collect_cnt[slot] = filled;
  } else if (to_refine) {
    for (int t = 0; t < cnt; ++t) cand.idx[j * kCand + t] = keep[t];
    cand_n[j] = cnt;
    refine_list[before_r + __popcll(bal_r & below)] = (int32_t)j;
  } else if (live) {
    bmus[j] = keep[0];
  }
}

// sum_c (x_c - w_c)^2 in fp64, columns dealt to lanes round-robin, butterfly reduction: the
// same order for every node, so identical weight vectors give bit-identical results.
__device__ __forceinline__ double sqdist_dense_wave(const float *__restrict__ x, const float *__restrict__ w,
                                                    int dim, int lane) {
  double s = 0.0;
  for (int c = lane; c < dim; c += kWave) {
    const double d = (double)x[c] - (double)w[c];
    s += d * d;
  }
  return wave_sum(s);
}

// Four such distances at once, each with the summation order of sqdist_dense_wave (same bits).
__device__ __forceinline__ void sqdist_dense_wave4(const float *__restrict__ x, const float *__restrict__ W,
                                                   const int (&id)[4], int dim, int lane, double (&out)[4]) {
  const float *w0 = W + (int64_t)id[0] * dim, *w1 = W + (int64_t)id[1] * dim;
  const float *w2 = W + (int64_t)id[2] * dim, *w3 = W + (int64_t)id[3] * dim;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (int c = lane; c < dim; c += kWave) {
    const double xv = (double)x[c];
    const double d0 = xv - (double)w0[c], d1 = xv - (double)w1[c];
    const double d2 = xv - (double)w2[c], d3 = xv - (double)w3[c];
    s0 += d0 * d0;
    s1 += d1 * d1;
    s2 += d2 * d2;
    s3 += d3 * d3;
  }
  out[0] = wave_sum(s0);
  out[1] = wave_sum(s1);
  out[2] = wave_sum(s2);
  out[3] = wave_sum(s3);
}

// The same distance for a sparse row with implicit zeros, regrouped so that only the nonzeros are
// visited: |w|^2 + sum_nz ((v - w_c)^2 - w_c^2).  Equal to the plain sum in exact arithmetic; in fp64
// its absolute error is about (dim + len) 2^-53 (|w|^2 + |x|^2), which is harmless unless the
// distance itself is that small (sqdist_csr_wave below).
// kN nodes at a time: the gathers of their weights are what it waits for, so they go together, 128 nonzeros of each.
// The term is rounded the same for any kN (lists of 100,000 rows of 100 nonzeros on 2,500 nodes: 190 -> 163 us; lists of two to four, which
// many wavefronts wait for side by side, 106 -> 105).
__device__ __forceinline__ double regrouped_term(double v, double wc) {
#pragma clang fp contract(off)
  const double d = v - wc;
  return __builtin_fma(d, d, -(wc * wc));
}

template <int kN>
__device__ __forceinline__ void sqdist_csr_regrouped_wave(const int32_t *__restrict__ idx,
                                                          const float *__restrict__ val, int len,
                                                          const float *__restrict__ W, const int (&node)[kN],
                                                          const double *__restrict__ wn64, int dim, int lane, double (&out)[kN]) {
  double s[kN] = {};
  for (int p0 = 0; p0 < len; p0 += 2 * kWave) {
    int c[2];
    float v[2], w[2][kN];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int p = min(p0 + u * kWave + lane, len - 1);
      c[u] = idx[p];
      v[u] = val[p];
      c[u] = c[u] < 0 ? 0 : (c[u] >= dim ? dim - 1 : c[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (p0 + u * kWave + lane < len) {
#pragma unroll
        for (int t = 0; t < kN; ++t) w[u][t] = W[(int64_t)node[t] * dim + c[u]];
      }
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (p0 + u * kWave + lane < len) {
#pragma unroll
        for (int t = 0; t < kN; ++t) s[t] += regrouped_term((double)v[u], (double)w[u][t]);
      }
  }
#pragma unroll
  for (int t = 0; t < kN; ++t) out[t] = wn64[node[t]] + wave_sum(s[t]);
}

// The BMU equation's sum as it is printed: every coordinate once, an unlisted one as zero, all
// terms non-negative, so nothing cancels and an instance that coincides with the weight vector
// is at distance exactly 0.  Lanes take the coordinates round-robin; each keeps a cursor into the
// row's (sorted) column list, which only ever moves forward.  dim loads: the rare path.
__device__ __forceinline__ double sqdist_csr_plain_wave(const int32_t *__restrict__ idx,
                                                        const float *__restrict__ val, int len,
                                                        const float *__restrict__ w, int dim, int lane) {
  double s = 0.0;
  int p = 0;
  for (int c = lane; c < dim; c += kWave) {
    while (p < len && idx[p] < c) ++p;
    const double x = (p < len && idx[p] == c) ? (double)val[p] : 0.0;
    const double d = x - (double)w[c];
    s += d * d;
  }
  return wave_sum(s);
}

// Squared norm of a sparse row in fp64 (every lane gets the sum).
__device__ __forceinline__ double csr_row_sqnorm_wave(const float *__restrict__ val, int len, int lane) {
  double s = 0.0;
  for (int p = lane; p < len; p += kWave) s += (double)val[p] * (double)val[p];
  return wave_sum(s);
}

// Exact distance of a sparse row: the regrouped sum wherever its rounding is at least 2^23 times
// smaller than the result (relative error below 1.2e-7, a hundredth of the tolerance band of the
// decision), the plain sum otherwise.  wn = |w|^2, xn = |x|^2.  Every lane holds the same bits of
// the regrouped value, so the branch is uniform over the wavefront; bit-identical weight vectors
// take the same branch and get the same bits.
template <int kN>
__device__ __forceinline__ void sqdist_csr_wave(const int32_t *__restrict__ idx, const float *__restrict__ val,
                                                int len, const float *__restrict__ W, const int (&node)[kN],
                                                const double *__restrict__ wn64, double xn, int dim, int lane, double (&d2)[kN]) {
  sqdist_csr_regrouped_wave<kN>(idx, val, len, W, node, wn64, dim, lane, d2);
#pragma unroll
  for (int t = 0; t < kN; ++t) {
    const double noise = ((double)dim + (double)len + 2.0) * 1.862645149230957e-09 * (wn64[node[t]] + xn);   // 2^-29 = 2^-52 * 2^23
    if (d2[t] < noise) d2[t] = sqdist_csr_plain_wave(idx, val, len, W + (int64_t)node[t] * dim, dim, lane);
  }
}

// The nearest of some nodes to a sparse row, by a wavefront: four at a time, then two, then one.
template <int kN>
__device__ __forceinline__ void nearest_csr_step(const int32_t *__restrict__ idx, const float *__restrict__ val, int len,
                                                 const float *__restrict__ W, const int32_t *__restrict__ lst,
                                                 const double *__restrict__ wn64, double xn, int dim, int k, int lane, double &best, int &arg) {
  int node[kN];
  double d2[kN];
#pragma unroll
  for (int t = 0; t < kN; ++t) node[t] = min(max(lst[t], 0), k - 1);      // lists only ever hold valid nodes; never trust memory
  sqdist_csr_wave<kN>(idx, val, len, W, node, wn64, xn, dim, lane, d2);
#pragma unroll
  for (int t = 0; t < kN; ++t)
    if (nearer(d2[t], node[t], best, arg)) { best = d2[t]; arg = node[t]; }
}

__device__ __forceinline__ int nearest_csr(const int32_t *__restrict__ idx, const float *__restrict__ val, int len,
                                           const float *__restrict__ W, const int32_t *__restrict__ lst, int cn,
                                           const double *__restrict__ wn64, int dim, int k, int lane) {
  const double xn = csr_row_sqnorm_wave(val, len, lane);
  double best = INFINITY;
  int arg = 0x7fffffff, t = 0;
  for (; t + 4 <= cn; t += 4) nearest_csr_step<4>(idx, val, len, W, lst + t, wn64, xn, dim, k, lane, best, arg);
  if (t + 2 <= cn) {
    nearest_csr_step<2>(idx, val, len, W, lst + t, wn64, xn, dim, k, lane, best, arg);
    t += 2;
  }
  if (t < cn) nearest_csr_step<1>(idx, val, len, W, lst + t, wn64, xn, dim, k, lane, best, arg);
  return arg;
}

__global__ __launch_bounds__(256) void k_refine_dense(const float *__restrict__ X, const float *__restrict__ W,
                                                      int dim, const int32_t *__restrict__ cand_idx,
                                                      const int32_t *__restrict__ cand_n,
                                                      const int32_t *__restrict__ refine_list,
                                                      const int32_t *__restrict__ list_counts,
                                                      int32_t *__restrict__ bmus) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int nwaves = gridDim.x * (blockDim.x / kWave);
  const int count = list_counts[0];
  for (int e = wave; e < count; e += nwaves) {
    const int64_t j = refine_list[e];
    const int cn = cand_n[j];
    double best = INFINITY;
    int arg = 0x7fffffff;
    for (int t = 0; t < cn; ++t) {
      const int i = cand_idx[j * kCand + t];
      const double d2 = sqdist_dense_wave(X + j * dim, W + (int64_t)i * dim, dim, lane);
      if (nearer(d2, i, best, arg)) { best = d2; arg = i; }
    }
    if (lane == 0) bmus[j] = arg == 0x7fffffff ? 0 : arg;      // no finite distance (non-finite input): node 0, as a plain scan gives
  }
}

// Next entry of a work list for this wavefront.  The lists differ in length by two orders of magnitude (2 to
// 256 nodes), and a fixed assignment of entries to wavefronts left most of the chip idle behind the wavefronts
// that had drawn the long ones (5 resident wavefronts per CU on average, out of 32); so entries are handed out
// from counters that the search zeroes with the list lengths.  One counter serialises: an atomic on one address
// takes about 10 ns whoever issues it, more than the comparison of a list of 128-feature rows.  Hence eight
// counters in different memory channels: workgroup b draws from counter b mod 8, which hands out the entries
// e = b mod 8 (mod 8).
__device__ inline int next_entry(int32_t *list_counts, int lane) {
  const int slice = blockIdx.x & (kListTickets - 1);
  int t = 0;
  // (opaque: where a loop ends in another "lane 0 only", the compiler may join the two and take the other lanes to the
  // broadcast below without lane 0, whose entry they would never get)
  asm volatile("" : "+v"(lane));
  if (lane == 0) t = atomicAdd(list_counts + kListCounts + slice * kListTicketStride, 1);
  return __builtin_amdgcn_readfirstlane(t) * kListTickets + slice;
}

// The same for a list that is usually shorter than the wavefronts are many: the first entry of each is given by its number, so that
// nothing is drawn at all then (8,192 wavefronts that all draw from eight counters to find the list empty: 10 us).
struct ListEntries {
  int32_t *counters;
  int at, drawn;             // the entry in hand; how many are given by number
  __device__ ListEntries(int32_t *list_counts)
      : counters(list_counts), at((int)(threadIdx.x / kWave * gridDim.x + blockIdx.x)), drawn((int)(gridDim.x * (blockDim.x / kWave))) {
    at = __builtin_amdgcn_readfirstlane(at);
  }
  __device__ void next(int count, int lane) { at = count <= drawn ? count : drawn + next_entry(counters, lane); }
};

// One collected list compared exactly by a wavefront: the nearest of its nodes (0x7fffffff: none at a finite distance) and how near.
__device__ __forceinline__ int nearest_listed(const float *__restrict__ x, const float *__restrict__ W, int dim, int k,
                                              const int32_t *__restrict__ lst, int cn, int lane, double &best) {
  best = INFINITY;
  int arg = 0x7fffffff;
  // four listed nodes at a time: their rows stream together and the instance is read once for the four
  // (a list can be long, and one distance at a time left the kernel waiting on its own loads); every
  // distance is still summed in the order of sqdist_dense_wave
  int t = 0;
  for (; t + 4 <= cn; t += 4) {
    int id[4];
    double d2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) id[u] = min(max(lst[t + u], 0), k - 1);   // lists only ever hold valid nodes; never trust memory
    sqdist_dense_wave4(x, W, id, dim, lane, d2);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (nearer(d2[u], id[u], best, arg)) { best = d2[u]; arg = id[u]; }
  }
  if (cn - t > 1) {                                // two or three left: as four, the last one again
    int id[4];
    double d2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) id[u] = min(max(lst[min(t + u, cn - 1)], 0), k - 1);
    sqdist_dense_wave4(x, W, id, dim, lane, d2);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (nearer(d2[u], id[u], best, arg)) { best = d2[u]; arg = id[u]; }
  } else if (t < cn) {
    const int i = min(max(lst[t], 0), k - 1);
    const double d2 = sqdist_dense_wave(x, W + (int64_t)i * dim, dim, lane);
    if (nearer(d2, i, best, arg)) { best = d2; arg = i; }
  }
  return arg;
}

// Exact comparison of the collected lists, a wavefront each.  A list that overflowed its capacity sends the instance on to the full
// rescan.  This is the form for lists that come in no particular order (the one-level filters): bound by the nodes' rows out of
// L2, with as many wavefronts as fit to wait for them.
__global__ __launch_bounds__(256) void k_refine_lists_each(const float *__restrict__ X, const float *__restrict__ W, int dim, int k,
                                                           const int32_t *__restrict__ collect_rows,
                                                           const int32_t *__restrict__ collect_cnt,
                                                           const int32_t *__restrict__ collect_list,
                                                           int32_t *__restrict__ rescan_list,
                                                           int32_t *__restrict__ list_counts, int32_t *__restrict__ bmus) {
  const int lane = threadIdx.x & (kWave - 1);
  const int count = list_counts[1];
  for (ListEntries it(list_counts); it.at < count; it.next(count, lane)) {
    const int e = it.at;
    const int64_t j = collect_rows[e];
    const int cn = collect_cnt[e];
    if (cn > kListCap || cn == 0) {
      if (lane == 0) rescan_list[atomicAdd(&list_counts[2], 1)] = (int32_t)j;
      continue;
    }
    double best;
    const int arg = nearest_listed(X + j * dim, W, dim, k, collect_list + (int64_t)e * kListCap, cn, lane, best);
    if (lane == 0) bmus[j] = arg == 0x7fffffff ? 0 : arg;      // no finite distance (non-finite input): node 0, as a plain scan gives
  }
}

// The same for the two-level search, whose lists were appended in its order: neighbours name much the same nodes, and comparing each
// list by itself read every node's row out of L2 once per instance (14.7 GB for 100,000 x 1,000 on a trained map of 2,500 nodes:
// 1,900 us at 7.7 TB/s).  From kListTileMin lists on, a workgroup takes 16 consecutive ones and compares their
// union with all 16 instances as one fp64 matrix product of rows relative to one of the nodes,
//   d2 = |x~|^2 + |w~|^2 - 2 x~.w~,   x~ = x - w_0, w~ = w - w_0,
// whose rounding is below (dim + 8) 2^-50 (|x~| + |w~|)^2; the nodes it cannot tell apart from the nearest - usually there are none - are compared
// by the plain sums as before, so the decision is the same to the bit.  Bound by the fp64 matrix pipe; the product in fp32 took
// half the time and left a dozen near-copies per instance to the plain sums (3,000 us).  The nodes left go four at a time: 1,000 -> 935 us.  A union of more than kUnionCap
// nodes, or of more than half of what the lists hold together, is not worth it.  Those lists, and any fewer than
// kListTileMin, are left to the launch that also rescans (k_lists_left_and_rescan): here, with the three workgroups
// per CU that the union's LDS leaves room for, 225 such tiles of 1,408 took as long as all the others (30,000 x 1,000 on a trained map
// of 3,600 nodes: a search 1,933 -> 1,316 us, 1,624 with every list by itself).  kListTileMin is the wavefronts that the chip holds: with fewer lists each
// has one or more to itself, and is done before a tile's chain of loads is (searches, tiles / one by one: 4,304 lists of 500 features
// 829 / 741 us, 7,732 of 1,000 1,233 / 1,105, 4,860 733 / 521; but 6,962 of 300 280 / 312; 10,427 of 300 316 / 364, 11,708 of 1,000 509 / 760).
constexpr int kListTileMin = 8192;
constexpr int kUnionCap = 320, kUnionHash = 1024;

template <bool kWide>
__global__ __launch_bounds__(256) void k_refine_lists_dense(const float *__restrict__ X, const float *__restrict__ W,
                                                            int dim, int k, const int32_t *__restrict__ collect_rows,
                                                            const int32_t *__restrict__ collect_cnt,
                                                            const int32_t *__restrict__ collect_list,
                                                            int32_t *__restrict__ rescan_list,
                                                            int32_t *__restrict__ list_counts,
                                                            int32_t *__restrict__ tiles_left,
                                                            int32_t *__restrict__ bmus) {
  __shared__ int s_hash[kUnionHash], s_node[kUnionCap], s_row[16], s_cnt[16], s_n, s_listed, s_slot;
  __shared__ double s_d2[16][kUnionCap + 1], s_xn[16], s_wn[kUnionCap];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int count = list_counts[1];
  if (count < kListTileMin) {
    for (int e = blockIdx.x * 256 + tid; e < count; e += gridDim.x * 256)
      if (collect_cnt[e] > kListCap || collect_cnt[e] == 0) rescan_list[atomicAdd(&list_counts[2], 1)] = collect_rows[e];
    return;
  }
  const int l16 = lane & 15, quad = lane >> 4;
  for (;;) {
    __syncthreads();                               // the previous tile's readers are done
    if (wave == 0) {
      const int t = next_entry(list_counts, lane); // of the tiles
      if (lane == 0) { s_slot = t; s_n = 0; s_listed = 0; }
    }
    for (int h = tid; h < kUnionHash; h += 256) s_hash[h] = -1;
    __syncthreads();
    const int e0 = s_slot * 16;
    if (e0 >= count) return;                       // uniform over the workgroup
    if (tid < 16) {
      const bool live = e0 + tid < count;
      const int cn = live ? collect_cnt[e0 + tid] : 0;
      s_row[tid] = live ? collect_rows[e0 + tid] : -1;
      s_cnt[tid] = cn > kListCap ? 0 : cn;
      if (live && (cn > kListCap || cn == 0)) rescan_list[atomicAdd(&list_counts[2], 1)] = s_row[tid];
    }
    __syncthreads();
    // union of the lists
    for (int r = wave; r < 16; r += 4) {
      const int cn = s_cnt[r];
      if (lane == 0) atomicAdd(&s_listed, cn);
      for (int t = lane; t < cn; t += kWave) {
        const int i = min(max(collect_list[(int64_t)(e0 + r) * kListCap + t], 0), k - 1);
        unsigned h = ((unsigned)i * 2654435761u) >> 22;                      // 10 bits
        for (int probe = 0; probe < kUnionHash; ++probe, h = (h + 1) & (kUnionHash - 1)) {
          if (s_n > kUnionCap) break;              // (a torn view of the counter only ends the search a little later)
          const int was = atomicCAS(&s_hash[h], -1, i);
          if (was == i) break;
          if (was == -1) {
            const int at = atomicAdd(&s_n, 1);
            if (at < kUnionCap) s_node[at] = i;
            break;
          }
        }
      }
    }
    __syncthreads();
    const int un = s_n;
    if (un > kUnionCap || 2 * un > s_listed) {     // uniform: both are read after the barrier and not written before the next
      if (tid == 0) tiles_left[atomicAdd(&list_counts[kTilesLeftWord], 1)] = s_slot;
      continue;
    }
    // the product: lane -> instance / node l16, features 4 quad .. 4 quad + 3 of every 16, which four instructions take one
    // each; a wavefront takes the 16-node tiles wave, wave + 4, ... in pairs
    const float *w0 = W + (int64_t)s_node[0] * dim;
    const float *x = X + (int64_t)(s_row[l16] < 0 ? s_row[0] : s_row[l16]) * dim;
    for (int u0 = 16 * wave; u0 < un; u0 += 128) {
      const bool two = u0 + 64 < un;               // uniform over the wavefront
      const float *wa = W + (int64_t)s_node[min(u0 + l16, un - 1)] * dim;
      const float *wb = W + (int64_t)s_node[min(u0 + 64 + l16, un - 1)] * dim;
      typedef double f64x4 __attribute__((ext_vector_type(4)));
      f64x4 da = {0.0, 0.0, 0.0, 0.0}, db = {0.0, 0.0, 0.0, 0.0};
      double xs = 0.0, as = 0.0, bs = 0.0;
      f32x4r xv = row_load<kWide>(x, 4 * quad, dim), rv = row_load<kWide>(w0, 4 * quad, dim);
      f32x4r av = row_load<kWide>(wa, 4 * quad, dim), bv = row_load<kWide>(wb, 4 * quad, dim);
      for (int c0 = 0; c0 < dim; c0 += 16) {
        const int c = c0 + 4 * quad;
        f32x4r xc = xv, rc = rv, ac = av, bc = bv;
        if (c0 + 16 < dim) {
          xv = row_load<kWide>(x, c + 16, dim);
          rv = row_load<kWide>(w0, c + 16, dim);
          av = row_load<kWide>(wa, c + 16, dim);
          if (two) bv = row_load<kWide>(wb, c + 16, dim);
        }
        row_tail<kWide>(xc, c, dim);
        row_tail<kWide>(rc, c, dim);
        row_tail<kWide>(ac, c, dim);
        row_tail<kWide>(bc, c, dim);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double r = (double)rc[e], xd = (double)xc[e] - r, ad = (double)ac[e] - r;
          xs = fma(xd, xd, xs);
          as = fma(ad, ad, as);
          da = __builtin_amdgcn_mfma_f64_16x16x4f64(xd, ad, da, 0, 0, 0);
          if (two) {
            const double bd = (double)bc[e] - r;
            bs = fma(bd, bd, bs);
            db = __builtin_amdgcn_mfma_f64_16x16x4f64(xd, bd, db, 0, 0, 0);
          }
        }
      }
      xs += __shfl_xor(xs, 16, 64); xs += __shfl_xor(xs, 32, 64);
      as += __shfl_xor(as, 16, 64); as += __shfl_xor(as, 32, 64);
      bs += __shfl_xor(bs, 16, 64); bs += __shfl_xor(bs, 32, 64);
      if (quad == 0) {
        if (u0 == 0) s_xn[l16] = xs;
        if (u0 + l16 < un) s_wn[u0 + l16] = as;
        if (u0 + 64 + l16 < un) s_wn[u0 + 64 + l16] = bs;
      }
      // column l16 = node, rows quad + 4 v = instances (the products alone: the norms are added when all are there)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (u0 + l16 < un) s_d2[quad + 4 * v][u0 + l16] = da[v];
        if (u0 + 64 + l16 < un) s_d2[quad + 4 * v][u0 + 64 + l16] = db[v];
      }
    }
    __syncthreads();
    for (int r = wave; r < 16; r += 4) {
      if (s_cnt[r] == 0) continue;
      const int64_t j = s_row[r];
      const double xn = s_xn[r];
      double best = INFINITY, wmax = 0.0;
      for (int u = lane; u < un; u += kWave) {
        const double wn = s_wn[u];
        const double d2 = xn + wn - 2.0 * s_d2[r][u];
        best = fmin(best, d2);
        wmax = fmax(wmax, wn);
      }
#pragma unroll
      for (int o = kWave / 2; o > 0; o >>= 1) {
        best = fmin(best, __shfl_xor(best, o, kWave));
        wmax = fmax(wmax, __shfl_xor(wmax, o, kWave));
      }
      const double reach = sqrt(xn) + sqrt(wmax);
      const double limit = best + 2.0 * 8.881784197001252e-16 * (double)(dim + 8) * reach * reach;      // 2^-50, both sides
      int arg = 0x7fffffff;
      if (limit < INFINITY) {                      // (false on NaN)
        double nearest = INFINITY;
        int under = 0;
        for (int u0 = 0; u0 < un; u0 += kWave)     // how many are under the limit, and which is the last of them
          for (unsigned long long m = __ballot(u0 + lane < un && !(xn + s_wn[min(u0 + lane, un - 1)] - 2.0 * s_d2[r][min(u0 + lane, un - 1)] > limit));
               m; m &= m - 1) {
            ++under;
            arg = s_node[u0 + __ffsll((long long)m) - 1];
          }
        if (under != 1) {                          // the plain sums decide, in the place of the products no longer needed
          typedef int __attribute__((may_alias)) word;
          word *open = reinterpret_cast<word *>(s_d2[r]);
          int at = 0;
          for (int u0 = 0; u0 < un; u0 += kWave) {
            const int u = min(u0 + lane, un - 1);
            const bool in = u0 + lane < un && !(xn + s_wn[u] - 2.0 * s_d2[r][u] > limit);
            const unsigned long long m = __ballot(in);
            // (a word of the list lies at or before the product its lane has read, and every product before that has been read)
            if (in) open[at + __popcll(m & ((1ull << lane) - 1))] = s_node[u];
            at += __popcll(m);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // a lane reads what others have written
          __builtin_amdgcn_wave_barrier();
          arg = nearest_listed(X + j * dim, W, dim, k, open, at, lane, nearest);
        }
      } else {
        arg = nearest_listed(X + j * dim, W, dim, k, collect_list + (int64_t)(e0 + r) * kListCap, s_cnt[r], lane, best);
      }
      if (lane == 0) bmus[j] = arg == 0x7fffffff ? 0 : arg;
    }
  }
}

// Exact scan of all nodes for the instances of rescan_list, a workgroup each.
__device__ __forceinline__ void rescan_rows(const float *__restrict__ X, const float *__restrict__ W, int dim, int k,
                                            const int32_t *__restrict__ rescan_list, int count, int32_t *__restrict__ bmus) {
  __shared__ double s_best[4];
  __shared__ int s_arg[4];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  for (int e = blockIdx.x; e < count; e += gridDim.x) {
    const int64_t j = rescan_list[e];
    const float *x = X + j * dim;
    double best = INFINITY;
    int arg = 0x7fffffff;
    for (int i = wave; i < k; i += 4) {           // ascending within a wave: strict < keeps the lowest index
      const double d2 = sqdist_dense_wave(x, W + (int64_t)i * dim, dim, lane);
      if (d2 < best) { best = d2; arg = i; }
    }
    if (lane == 0) { s_best[wave] = best; s_arg[wave] = arg; }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < 4; ++w)
        if (s_best[w] < best || (s_best[w] == best && s_arg[w] < arg)) { best = s_best[w]; arg = s_arg[w]; }
      bmus[j] = arg == 0x7fffffff ? 0 : arg;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_rescan_dense(const float *__restrict__ X, const float *__restrict__ W,
                                                      int dim, int k, const int32_t *__restrict__ rescan_list,
                                                      const int32_t *__restrict__ list_counts,
                                                      int32_t *__restrict__ bmus) {
  rescan_rows(X, W, dim, k, rescan_list, list_counts[2], bmus);
}

// After k_refine_lists_dense: the lists that it left, a wavefront each (the overflowed ones are on rescan_list by then), and the rescan.  Bound by the
// longest list where there are few: two or four wavefronts share each then (3,734 lists of 1,000 features: a search 667 -> 578 us).
__global__ __launch_bounds__(256) void k_lists_left_and_rescan(const float *__restrict__ X, const float *__restrict__ W, int dim, int k,
                                                               const int32_t *__restrict__ collect_rows,
                                                               const int32_t *__restrict__ collect_cnt,
                                                               const int32_t *__restrict__ collect_list,
                                                               const int32_t *__restrict__ tiles_left,
                                                               const int32_t *__restrict__ rescan_list,
                                                               int32_t *__restrict__ list_counts, int32_t *__restrict__ bmus) {
  const int lane = threadIdx.x & (kWave - 1);
  const int lists = list_counts[1], rescans = list_counts[2];
  const bool tiles = lists >= kListTileMin;
  const int count = tiles ? list_counts[kTilesLeftWord] * 16 : lists;
  auto entry = [&](int at) { return tiles ? tiles_left[at >> 4] * 16 + (at & 15) : at; };
  auto length = [&](int e) {
    const int cn = e < lists ? collect_cnt[e] : 0;
    return cn > kListCap ? 0 : cn;
  };
  const int wave = threadIdx.x / kWave, blocks = gridDim.x;
  const int team = count <= blocks ? 4 : count <= 2 * blocks ? 2 : 1;
  if (team > 1) {
    __shared__ double s_near[4];
    __shared__ int s_node[4];
    const int at = (wave / team) * blocks + blockIdx.x, part = wave % team;
    const int e = at < count ? entry(at) : 0, cn = at < count ? length(e) : 0;
    const int per = ((cn + 3) / 4 + team - 1) / team * 4, first = min(part * per, cn);      // whole fours
    const int64_t j = cn ? collect_rows[e] : 0;
    double best;
    int arg = nearest_listed(X + j * dim, W, dim, k, collect_list + (int64_t)e * kListCap + first, min(per, cn - first), lane, best);
    if (lane == 0) { s_near[wave] = best; s_node[wave] = arg; }
    __syncthreads();
    if (cn && part == 0 && lane == 0) {
      for (int w = wave + 1; w < wave + team; ++w)
        if (nearer(s_near[w], s_node[w], best, arg)) { best = s_near[w]; arg = s_node[w]; }
      bmus[j] = arg == 0x7fffffff ? 0 : arg;
    }
  } else {
    for (ListEntries it(list_counts + kListTickets2); it.at < count; it.next(count, lane)) {
      const int e = entry(it.at), cn = length(e);
      if (cn == 0) continue;
      const int64_t j = collect_rows[e];
      double best;
      const int arg = nearest_listed(X + j * dim, W, dim, k, collect_list + (int64_t)e * kListCap, cn, lane, best);
      if (lane == 0) bmus[j] = arg == 0x7fffffff ? 0 : arg;
    }
  }
  rescan_rows(X, W, dim, k, rescan_list, rescans, bmus);
}

__global__ __launch_bounds__(256) void k_refine_csr(const int64_t *__restrict__ indptr,
                                                    const int32_t *__restrict__ indices,
                                                    const float *__restrict__ values,
                                                    const float *__restrict__ W, const double *__restrict__ wn64,
                                                    int dim, int k, const int32_t *__restrict__ cand_idx,
                                                    const int32_t *__restrict__ cand_n,
                                                    const int32_t *__restrict__ refine_list,
                                                    const int32_t *__restrict__ list_counts,
                                                    int32_t *__restrict__ bmus) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int nwaves = gridDim.x * (blockDim.x / kWave);
  const int count = list_counts[0];
  for (int e = wave; e < count; e += nwaves) {
    const int64_t j = refine_list[e];
    const int64_t s = indptr[j];
    const int len = (int)(indptr[j + 1] - s);
    const int cn = cand_n[j];
    const int arg = nearest_csr(indices + s, values + s, len, W, cand_idx + j * kCand, cn, wn64, dim, k, lane);
    if (lane == 0) bmus[j] = arg == 0x7fffffff ? 0 : arg;      // no finite distance (non-finite input): node 0, as a plain scan gives
  }
}

__global__ __launch_bounds__(256) void k_refine_lists_csr(const int64_t *__restrict__ indptr,
                                                          const int32_t *__restrict__ indices,
                                                          const float *__restrict__ values,
                                                          const float *__restrict__ W,
                                                          const double *__restrict__ wn64, int dim, int k,
                                                          const int32_t *__restrict__ collect_rows,
                                                          const int32_t *__restrict__ collect_cnt,
                                                          const int32_t *__restrict__ collect_list,
                                                          int32_t *__restrict__ rescan_list,
                                                          int32_t *__restrict__ list_counts, int scan_above,
                                                          int32_t *__restrict__ bmus) {
  const int lane = threadIdx.x & (kWave - 1);
  const int count = list_counts[1];
  for (int e = next_entry(list_counts, lane); e < count; e = next_entry(list_counts, lane)) {
    const int64_t j = collect_rows[e];
    const int64_t s = indptr[j];
    const int len = (int)(indptr[j + 1] - s);
    // overflowed (or empty) list: exact scan of all nodes; so is a list longer than scan_above, for which that scan
    // is the cheaper of the two
    if (collect_cnt[e] > min(kListCap, scan_above) || collect_cnt[e] < 1) {
      if (lane == 0) rescan_list[atomicAdd(&list_counts[2], 1)] = (int32_t)j;
      continue;
    }
    const int cn = min(collect_cnt[e], kListCap);
    const int arg = nearest_csr(indices + s, values + s, len, W, collect_list + (int64_t)e * kListCap, cn, wn64, dim, k, lane);
    if (lane == 0) bmus[j] = arg == 0x7fffffff ? 0 : arg;
  }
}

// Exact scan of all nodes for one sparse row from the row-major code book: wavefront w takes the nodes
// w, w + 4, ...; (best, arg) of this wavefront, ties to the lowest index.
__device__ __forceinline__ void rescan_row_major(const int32_t *__restrict__ idx, const float *__restrict__ val,
                                                 int len, const float *__restrict__ W,
                                                 const double *__restrict__ wn64, double xn, int dim, int k,
                                                 int lane, int wave, double &best, int &arg) {
  best = INFINITY;
  arg = 0x7fffffff;
  for (int i = wave; i < k; i += 4) {             // ascending within a wave: strict < keeps the lowest index
    const int node[1] = {i};
    double d2[1];
    sqdist_csr_wave<1>(idx, val, len, W, node, wn64, xn, dim, lane, d2);
    if (d2[0] < best) { best = d2[0]; arg = i; }
  }
}

__global__ __launch_bounds__(256) void k_rescan_csr(const int64_t *__restrict__ indptr,
                                                    const int32_t *__restrict__ indices,
                                                    const float *__restrict__ values,
                                                    const float *__restrict__ W, const double *__restrict__ wn64,
                                                    int dim, int k, const int32_t *__restrict__ rescan_list,
                                                    const int32_t *__restrict__ list_counts,
                                                    int32_t *__restrict__ bmus) {
  __shared__ double s_best[4];
  __shared__ int s_arg[4];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int count = list_counts[2];
  for (int e = blockIdx.x; e < count; e += gridDim.x) {
    const int64_t j = rescan_list[e];
    const int64_t s = indptr[j];
    const int len = (int)(indptr[j + 1] - s);
    const double xn = csr_row_sqnorm_wave(values + s, len, lane);
    double best;
    int arg;
    rescan_row_major(indices + s, values + s, len, W, wn64, xn, dim, k, lane, wave, best, arg);
    if (lane == 0) { s_best[wave] = best; s_arg[wave] = arg; }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < 4; ++w)
        if (s_best[w] < best || (s_best[w] == best && s_arg[w] < arg)) { best = s_best[w]; arg = s_arg[w]; }
      bmus[j] = arg == 0x7fffffff ? 0 : arg;
    }
    __syncthreads();
  }
}

// The same scan from a transposed fp32 copy of the code book, Wt[c][i] with row stride kt.  A scan from the
// row-major code book reads one 4-byte weight per node and nonzero, each from a row of its own: a memory
// transaction per weight.  From the transposed copy the weights of one column and 64 consecutive nodes are
// one 256-byte read, and a thread adds up one node's terms over the row's nonzeros:
//     d2_i = |w_i|^2 + sum_nz ((v - w_ic)^2 - w_ic^2)
// (the regrouped sum of sqdist_csr_regrouped_wave, its terms added in the order of the row instead of
// across a wavefront).  A node for which that sum is all rounding noise needs the plain sum over every
// coordinate, which has to walk the node's row of W: if any node of the scan is that close to the instance,
// the whole scan is done again from the row-major code book, as k_rescan_csr does it (an instance that
// coincides with a weight vector: rare).
// The copy is written by k_transpose_for_rescan, and only when the list of instances to scan is not empty.
constexpr int kRescanChunk = 512;        // nonzeros staged in LDS at a time
constexpr int kRescanNodes = 2;          // nodes per thread and round

__global__ __launch_bounds__(256) void k_transpose_for_rescan(const float *__restrict__ W, int k, int dim, int64_t kt,
                                                              const int32_t *__restrict__ list_counts,
                                                              float *__restrict__ Wt) {
  if (list_counts[2] == 0) return;
  __shared__ float tile[64][65];
  const int tc = (dim + 63) / 64, ti = (k + 63) / 64;
  const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
  for (int64_t t = blockIdx.x; t < (int64_t)tc * ti; t += gridDim.x) {
    const int i0 = (int)(t / tc) * 64, c0 = (int)(t % tc) * 64;
    for (int r = y; r < 64; r += 4) {
      const int i = i0 + r, c = c0 + x;
      tile[r][x] = (i < k && c < dim) ? W[(int64_t)i * dim + c] : 0.f;
    }
    __syncthreads();
    for (int r = y; r < 64; r += 4) {
      const int c = c0 + r, i = i0 + x;
      if (c < dim && i < kt) Wt[(int64_t)c * kt + i] = tile[x][r];
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_rescan_csr_t(const int64_t *__restrict__ indptr,
                                                      const int32_t *__restrict__ indices,
                                                      const float *__restrict__ values,
                                                      const float *__restrict__ W, const float *__restrict__ Wt,
                                                      int64_t kt, const double *__restrict__ wn64, int dim, int k,
                                                      const int32_t *__restrict__ rescan_list,
                                                      const int32_t *__restrict__ list_counts,
                                                      int32_t *__restrict__ bmus) {
  __shared__ int32_t s_col[kRescanChunk];
  __shared__ float s_val[kRescanChunk];
  __shared__ double s_best[4];
  __shared__ int s_arg[4];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int count = list_counts[2];
  for (int e = blockIdx.x; e < count; e += gridDim.x) {
    const int64_t j = rescan_list[e];
    const int64_t s = indptr[j];
    const int len = (int)(indptr[j + 1] - s);
    const double xn = csr_row_sqnorm_wave(values + s, len, lane);
    const double noise_scale = ((double)dim + (double)len + 2.0) * 1.862645149230957e-09;      // as in sqdist_csr_wave
    const bool fits = len <= kRescanChunk;
    if (fits) {
      for (int p = tid; p < len; p += 256) {
        s_col[p] = min(max(indices[s + p], 0), dim - 1);
        s_val[p] = values[s + p];
      }
      __syncthreads();
    }
    double best = INFINITY;
    int arg = 0x7fffffff;
    bool in_noise = false;
    for (int i0 = 0; i0 < k; i0 += 256 * kRescanNodes) {
      double acc[kRescanNodes];
      int node[kRescanNodes];
#pragma unroll
      for (int r = 0; r < kRescanNodes; ++r) {
        acc[r] = 0.0;
        node[r] = min(i0 + r * 256 + tid, k - 1);       // a thread beyond the last node reads node k - 1 and drops the result
      }
      for (int p0 = 0; p0 < len; p0 += kRescanChunk) {
        const int cn = min(kRescanChunk, len - p0);
        if (!fits) {
          __syncthreads();
          for (int p = tid; p < cn; p += 256) {
            s_col[p] = min(max(indices[s + p0 + p], 0), dim - 1);
            s_val[p] = values[s + p0 + p];
          }
          __syncthreads();
        }
#pragma unroll 4
        for (int p = 0; p < cn; ++p) {
          const float *row = Wt + (int64_t)s_col[p] * kt;
          const double v = (double)s_val[p];
#pragma unroll
          for (int r = 0; r < kRescanNodes; ++r) {
            const double wc = (double)row[node[r]];
            const double d = v - wc;
            acc[r] += d * d - wc * wc;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < kRescanNodes; ++r) {
        const int i = i0 + r * 256 + tid;
        if (i < k) {                                    // ascending per thread: strict < keeps the lowest index
          const double wn = wn64[i];
          const double d2 = wn + acc[r];
          if (d2 < noise_scale * (wn + xn)) in_noise = true;
          if (d2 < best) { best = d2; arg = i; }
        }
      }
    }
    if (__syncthreads_or(in_noise)) {
      rescan_row_major(indices + s, values + s, len, W, wn64, xn, dim, k, lane, wave, best, arg);
    } else {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best, o, kWave);
        const int oa = __shfl_xor(arg, o, kWave);
        if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
      }
    }
    if (lane == 0) { s_best[wave] = best; s_arg[wave] = arg; }
    __syncthreads();
    if (tid == 0) {
      for (int w = 1; w < 4; ++w)
        if (s_best[w] < best || (s_best[w] == best && s_arg[w] < arg)) { best = s_best[w]; arg = s_arg[w]; }
      bmus[j] = arg == 0x7fffffff ? 0 : arg;
    }
    __syncthreads();
  }
}

static int persistent_blocks(const som_ctx *c, int64_t upper) {
  int64_t b = (int64_t)c->n_cu * 8;
  if (b > upper) b = upper;
  if (b < 1) b = 1;
  return (int)b;
}

// Roundings a product term can suffer in the fp32 MFMA pass: the accumulator is flushed into a
// second one every kDenseAccumBlock features.
static double fp32_pass_roundings(int dim) {
  return (double)kDenseAccumBlock + (double)((dim + kDenseAccumBlock - 1) / kDenseAccumBlock) + 2.0;
}

// The same for the split-fp16 pass, in units of u relative to sum |x_c w'_c|.  Measured
// behaviour of v_mfma_f32_32x32x16_f16 on gfx950 (checked by a test through som_debug_mfma_f16):
// the 16 products are aligned to the largest of them and truncated 25 bits below its leading bit,
// their sum joins the accumulator with an error of at most 2 u of the result.  Priced here at
// 9 u max|product| + 2.5 u (|C| + sum|products|) per instruction: over a flush interval of f chunks
// of 32 features (6 f instructions) that is 2.5 * 6 f + 9; every flush adds one rounding, and a
// wavefront flushes at most ceil(dim / (32 f)) + 1 times per node block.
static double split_pass_roundings(int dim) {
  const int chunks = split_flush_chunks(dim);
  return 2.5 * 6.0 * chunks + 9.0 + (double)((dim + 32 * chunks - 1) / (32 * chunks)) + 2.0;
}

// The rounding model of the filter that produced the scores (mode = kCertify*).
// Roundings of the split-fp16 pass over `dim` features (see split_pass_roundings).
static double split_roundings_for(int dim) {
  const int chunks = split_flush_chunks(dim);
  return 2.5 * 6.0 * chunks + 9.0 + (double)((dim + 32 * chunks - 1) / (32 * chunks)) + 2.0;
}

MarginModel margin_model(const som_ctx *c, int mode, const int64_t *indptr, bool hot) {
  MarginModel mm{2.0 * fp32_pass_roundings(c->dim) + 4.0, 0.0, nullptr, nullptr, 0, nullptr, nullptr, 0.0, nullptr, nullptr, nullptr, nullptr, nullptr,
                 nullptr, nullptr, 0};
  if (mode == kCertifyCsr) {
    mm.indptr = indptr;
    mm.row_q = c->row_q;
    if (hot) {
      // the hot block's dot product: accumulation + 12 u of the split, doubled by the factor -2 of the score;
      // its product then joins the chain of the tail (one more rounding, inside the tail's own + 6)
      mm.coef_hot = 2.0 * split_roundings_for(kHot) + 24.0;
      mm.hot_xn = c->hot_xn;
      mm.hot_xscale = c->hot_xscale;
      mm.hot_wscale = c->hot_wscale;
    }
  }
  if (mode == kCertifyCoarse) {
    // One fp16 product per feature pair on the hi halves alone (coarse pass of the two-level search), whatever the
    // rows are.  An operand element v / scale is rounded to 11 significant bits, |dv| <= 2^-11 |v| + 2^-25 scale, so
    // by Cauchy-Schwarz the dot product of the rounded rows is off by at most
    //   |dx| |w'| + |hi_x| |dw| <= (2 + 2^-11) 2^-11 X Wm + floor terms = (2^14 + 8) u X Wm + ...,
    // doubled by the factor -2 of the score.  Accumulation: one chain of ceil(dim / 16) matrix instructions
    // per score, never flushed, priced per instruction like the split pass (2.5 u of the running sum each,
    // 9 u of the largest product once, + 2).  The stored c_i, the final multiply-add and the roundings of
    // w - mu and x - mu as in the split model.
    const double chain = 2.5 * (double)((c->dim + 15) / 16) + 9.0 + 2.0;
    mm.coef_xw = 2.0 * (16384.0 + 8.0) + 2.0 * chain + 4.0 + 2.0;
    mm.coef_floor = sqrt((double)c->dim);        // 2^-25 per element and operand, doubled = u
    mm.xscale = c->xscale;
    mm.wscale = c->wscale;
    mm.x_centered = 1;
  }
  if (mode == kCertifySelect || mode == kCertifySubspace) {
    // The same pass, with the norms |dx| and |dw| that these rows really have (xlost, wlost_bits) in the place of
    // their worst case: the roundings are spread evenly, so the norms are less than half of it, and the block
    // selection keeps fewer blocks.
    const double chain = 2.5 * (double)((c->dim + 15) / 16) + 9.0 + 2.0;
    mm.coef_xw = 2.0 * chain * (1.0 + 0x1p-9) + 4.0 + 2.0;
    mm.x_centered = 1;
    mm.xlost = c->xlost;
    mm.wlost_bits = c->wlost_bits;
    if (mode == kCertifySubspace) {
      mm.sub = c->sub_state;
      mm.sub_err = c->sub_err;
    }
  }
  if (mode == kCertifySubspaceCsr || mode == kCertifySubspaceCsrSelect) {
    // the sparse rows are not centred: terms in |mu| as in the sweep; everything else is in the coordinates' own bounds
    mm.sub = c->sub_state;
    mm.sub_err = mode == kCertifySubspaceCsr ? c->sub_err2 : c->sub_err;
    mm.sub_fine = mode == kCertifySubspaceCsr;
  }
  if (mode == kCertifySplit || mode == kCertifySubspaceFine) {
    // dot product: accumulation + 3 * 2^-22 of the split (= 12 u) ; both doubled by the factor -2;
    // + 4 for the stored c_i, the final multiply-add and the rounding of w - mu, + 2 for the rounding
    // of x - mu (its part that does not depend on the node cancels in every comparison).  Never
    // below the fp32 coefficient.
    const double split = 2.0 * split_pass_roundings(c->dim) + 24.0 + 4.0 + 2.0;
    if (split > mm.coef_xw) mm.coef_xw = split;
    mm.coef_floor = sqrt((double)c->dim);        // 2 * 2^-25 per element = u, |v|_1 <= sqrt(dim) |v|_2
    mm.xscale = c->xscale;
    mm.wscale = c->wscale;
    mm.x_centered = 1;
    if (mode == kCertifySubspaceFine) {
      mm.sub = c->sub_state;
      mm.sub_err = c->sub_err2;
      mm.sub_fine = 1;
    }
  }
  return mm;
}

hipError_t launch_certify(som_ctx *c, int64_t n, int groups, int mode, const int64_t *indptr, int32_t *bmus, bool hot,
                          const int32_t *order, const SubspaceState *state) {
  CandView cand{c->cand_val, c->cand_idx, c->cand_over};
  const MarginModel mm = margin_model(c, mode, indptr, hot);
  UnitWork work{0, 0, nullptr, nullptr, nullptr};
  if (mode == kCertifyCsr)
    work = UnitWork{c->csr_sweeps, c->unit_cap, c->unit_work, c->list_counts + kUnitCounts, c->collect_list};
  hipLaunchKernelGGL(k_certify, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, cand, groups, c->xn32,
                     c->wmax_bits, c->mu_norm2, mm, n, c->k, bmus, c->cand_n, c->refine_list, c->collect_rows,
                     c->collect_thr, c->collect_cnt, c->list_counts, work, order, state, mode == kCertifySubspaceCsr);
  return hipGetLastError();
}

// Test hook: the margin k_certify applies to every instance (the same function, the same inputs).
__global__ __launch_bounds__(256) void k_margins(const float *__restrict__ xn32, const unsigned *__restrict__ wmax_bits,
                                                 const float *__restrict__ mu_norm2, MarginModel mm, int64_t n,
                                                 double *__restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) out[j] = score_margin(mm, j, (double)xn32[j], (double)__uint_as_float(*wmax_bits), (double)*mu_norm2);
}

hipError_t launch_margins(som_ctx *c, int64_t n, int mode, const int64_t *indptr, double *out, bool hot) {
  hipLaunchKernelGGL(k_margins, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->xn32, c->wmax_bits,
                     c->mu_norm2, margin_model(c, mode, indptr, hot), n, out);
  return hipGetLastError();
}

hipError_t launch_refine_lists_dense(som_ctx *c, const float *X, const float *W, int32_t *bmus, bool ordered) {
  const int blocks = 3 * c->n_cu;          // of the union's kernel: what their LDS leaves room for
  if (!ordered)
    hipLaunchKernelGGL(k_refine_lists_each, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, X, W,
                       c->dim, c->k, c->collect_rows, c->collect_cnt, c->collect_list, c->rescan_list, c->list_counts, bmus);
  else if (c->dim >= 4)
    hipLaunchKernelGGL(k_refine_lists_dense<true>, dim3(blocks), dim3(256), 0, c->stream, X, W,
                       c->dim, c->k, c->collect_rows, c->collect_cnt, c->collect_list, c->rescan_list, c->list_counts, c->refine_list, bmus);
  else
    hipLaunchKernelGGL(k_refine_lists_dense<false>, dim3(blocks), dim3(256), 0, c->stream, X, W,
                       c->dim, c->k, c->collect_rows, c->collect_cnt, c->collect_list, c->rescan_list, c->list_counts, c->refine_list, bmus);
  return hipGetLastError();
}

hipError_t launch_refine_dense(som_ctx *c, const float *X, const float *W, int32_t *bmus) {
  hipLaunchKernelGGL(k_refine_dense, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, X, W, c->dim,
                     c->cand_idx, c->cand_n, c->refine_list, c->list_counts, bmus);
  return hipGetLastError();
}

// ordered: as of launch_refine_lists_dense, which has left some of its lists (in tiles: refine_list, whose own entries are done).
hipError_t launch_rescan_dense(som_ctx *c, const float *X, const float *W, int32_t *bmus, bool ordered) {
  if (ordered) {
    hipLaunchKernelGGL(k_lists_left_and_rescan, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, X, W, c->dim,
                       c->k, c->collect_rows, c->collect_cnt, c->collect_list, c->refine_list, c->rescan_list, c->list_counts, bmus);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_rescan_dense, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, X, W, c->dim,
                     c->k, c->rescan_list, c->list_counts, bmus);
  return hipGetLastError();
}

hipError_t launch_refine_csr(som_ctx *c, const int64_t *indptr, const int32_t *indices, const float *values,
                             const float *W, int32_t *bmus) {
  hipLaunchKernelGGL(k_refine_csr, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, indptr, indices,
                     values, W, c->wn64, c->dim, c->k, c->cand_idx, c->cand_n, c->refine_list, c->list_counts, bmus);
  return hipGetLastError();
}

hipError_t launch_refine_lists_csr(som_ctx *c, const int64_t *indptr, const int32_t *indices, const float *values,
                                   const float *W, int32_t *bmus) {
  // A listed node costs a memory transaction per nonzero (its weights lie in a row of their own); the scan of all
  // nodes from the transposed copy reads the same weights 16 to a transaction, and measured 24 times cheaper per
  // (instance, node) pair on a 50 x 50 map: beyond k / 24 listed nodes the scan of everything wins.
  const int scan_above = c->Wt32 ? (c->k / 24 > 16 ? c->k / 24 : 16) : kListCap;
  hipLaunchKernelGGL(k_refine_lists_csr, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, indptr,
                     indices, values, W, c->wn64, c->dim, c->k, c->collect_rows, c->collect_cnt, c->collect_list,
                     c->rescan_list, c->list_counts, scan_above, bmus);
  return hipGetLastError();
}

// ---------------------------------------------------------------- distances to the BMUs
// Post-training output: Euclidean distance between every instance and the weight vector of
// the node it is mapped to, in fp64, and the mean of those distances (quantisation error).
// A workgroup owns a contiguous block of instances and leaves one
// partial sum, the partial sums are added in index order by k_mean_of_partials: the result
// does not depend on the schedule.  A node index outside [0, k) yields NaN.

// Dense rows: memory-bound, one read of the instances (the nodes' rows come out of L2); kLanes lanes share a row (16 up
// to 64 features, 32 up to 128, else the wavefront) and take 4 kAhead features each of instance and node before they use
// the first (100,000 x 1,000: 208 -> 82 us; 91,834 x 30: 25 -> 9).
// Sparse rows need |w|^2 of their nodes.  The nodes met are marked first (k_mark_nodes) and their norms taken once,
// by a workgroup each (k_marked_norms): an instance's own wavefront reading its node's whole row took 321 us for 1,000
// instances of a 50,000-column set on 321 nodes, the three launches take 35.
constexpr int kDistThreads = 512;

template <bool kCsr, bool kWide, int kLanes, int kAhead>
__global__ __launch_bounds__(kDistThreads) void k_bmu_distances(const float *__restrict__ X,
                                                                const int64_t *__restrict__ indptr,
                                                                const int32_t *__restrict__ indices,
                                                                const float *__restrict__ values,
                                                                const float *__restrict__ W, const double *__restrict__ wn64,
                                                                int64_t n, int k, int dim,
                                                                const int32_t *__restrict__ bmus, float *__restrict__ dist,
                                                                double *__restrict__ partial) {
  constexpr int kTeams = kDistThreads / kLanes;
  __shared__ double team_total[kTeams];
  const int lane = threadIdx.x % kLanes;
  const int team = threadIdx.x / kLanes;
  const int64_t per_block = (n + gridDim.x - 1) / gridDim.x;
  const int64_t j0 = (int64_t)blockIdx.x * per_block;
  const int64_t j1 = j0 + per_block < n ? j0 + per_block : n;
  double total = 0.0;
  for (int64_t j = j0 + team; j < j1; j += kTeams) {
    const int b = bmus[j];
    double d = NAN;
    if ((unsigned)b < (unsigned)k) {
      const float *w = W + (int64_t)b * dim;
      double d2;
      if (kCsr) {
        const int64_t rs = indptr[j];
        const int len = (int)(indptr[j + 1] - rs);
        const int node[1] = {b};
        double one[1];
        sqdist_csr_wave<1>(indices + rs, values + rs, len, W, node, wn64, csr_row_sqnorm_wave(values + rs, len, lane), dim, lane, one);
        d2 = one[0];
      } else {
        const float *x = X + j * dim;
        double s = 0.0;
        for (int c0 = 0; c0 < dim; c0 += 4 * kAhead * kLanes) {
          f32x4r xv[kAhead], wv[kAhead];
#pragma unroll
          for (int u = 0; u < kAhead; ++u) {
            xv[u] = row_load<kWide>(x, c0 + 4 * (lane + kLanes * u), dim);
            wv[u] = row_load<kWide>(w, c0 + 4 * (lane + kLanes * u), dim);
          }
#pragma unroll
          for (int u = 0; u < kAhead; ++u) {
            const int c = c0 + 4 * (lane + kLanes * u);
            if (c0 + 4 * kLanes * (u + 1) > dim) {      // uniform
              row_tail<kWide>(xv[u], c, dim);
              row_tail<kWide>(wv[u], c, dim);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double t = (double)xv[u][e] - (double)wv[u][e];
              s += t * t;
            }
          }
        }
        d2 = team_sum<kLanes>(s);
      }
      d = sqrt(d2);
    }
    if (dist && lane == 0) dist[j] = (float)d;
    total += d;
  }
  if (lane == 0) team_total[team] = total;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = team_total[0];
    for (int w = 1; w < kTeams; ++w) t += team_total[w];
    partial[blockIdx.x] = t;
  }
}

// owner[i] = one of the instances of node i, counted from one; which one does not matter.  Zero at all others: every entry
// is cleared by the kernel below as it takes it.
__global__ __launch_bounds__(256) void k_mark_nodes(const int32_t *__restrict__ bmus, int64_t n, int k, int32_t *__restrict__ owner) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < n && (unsigned)bmus[j] < (unsigned)k) owner[bmus[j]] = (int32_t)j + 1;
}

// Looks through the instances or through the nodes, whichever are fewer, for the owners or the owned.  A workgroup looks at a stretch of them at once, then
// takes the norms of those found one after the other.  (A walk over all nodes whatever n, a flag at a time: 10 rows on
// 4,000,000 nodes 529 us for the distances instead of 17.)
__global__ __launch_bounds__(256) void k_marked_norms(const float *__restrict__ W, int64_t n, int k, int dim,
                                                      const int32_t *__restrict__ bmus, int32_t *__restrict__ owner,
                                                      double *__restrict__ wn64) {
  __shared__ double s_part[4];
  __shared__ int s_node[256], s_found;
  const int tid = threadIdx.x;
  const bool by_instance = n < k;
  const int64_t items = by_instance ? n : k;
  const int64_t per = (items + gridDim.x - 1) / gridDim.x, first = blockIdx.x * per;
  const int64_t last = first + per < items ? first + per : items;
  for (int64_t t0 = first; t0 < last; t0 += 256) {
    if (tid == 0) s_found = 0;
    __syncthreads();
    const int64_t t = t0 + tid;
    int i = -1;
    if (t < last) {
      if (by_instance) {
        i = bmus[t];
        if ((unsigned)i >= (unsigned)k || owner[i] != (int32_t)t + 1) i = -1;
      } else if (owner[t] != 0) {
        i = (int)t;
      }
    }
    if (i >= 0) {
      owner[i] = 0;
      s_node[atomicAdd(&s_found, 1)] = i;
    }
    __syncthreads();
    const int found = s_found;
    for (int f = 0; f < found; ++f) {
      const float *w = W + (int64_t)s_node[f] * dim;
      double s[4] = {0, 0, 0, 0};
      for (int c0 = 0; c0 < dim; c0 += 8 * 256) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = w[min(c0 + 256 * u + tid, dim - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u & 3] += c0 + 256 * u + tid < dim ? (double)v[u] * (double)v[u] : 0.0;
      }
      const double sum = wave_sum((s[0] + s[1]) + (s[2] + s[3]));
      if ((tid & 63) == 0) s_part[tid >> 6] = sum;
      __syncthreads();
      if (tid == 0) wn64[s_node[f]] = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
      __syncthreads();
    }
    __syncthreads();                             // (nobody still reads s_found when it is cleared again)
  }
}

__global__ __launch_bounds__(64) void k_mean_of_partials(const double *__restrict__ partial, int count, int64_t n,
                                                         double *__restrict__ out) {
  double s = 0.0;
  for (int i = threadIdx.x; i < count; i += kWave) s += partial[i];
  s = wave_sum(s);
  if (threadIdx.x == 0) *out = n > 0 ? s / (double)n : 0.0;
}

static int distance_blocks(int64_t n, int lanes) {
  const int teams = kDistThreads / lanes;
  int64_t blocks = (n + teams - 1) / teams;
  if (blocks > kDistBlocks) blocks = kDistBlocks;
  return blocks < 1 ? 1 : (int)blocks;
}

// Dense rows (no context needed).
hipError_t launch_bmu_distances_on(hipStream_t stream, const float *X, int64_t n, const float *W, int k, int dim,
                                   const int32_t *bmus, float *dist, double *qerror, double *partial) {
  const int blocks = distance_blocks(n, dim <= 64 ? 16 : dim <= 128 ? 32 : kWave);
#define SOM_DISTANCES(WIDE, L, AHEAD)                                                                                  \
  hipLaunchKernelGGL((k_bmu_distances<false, WIDE, L, AHEAD>), dim3(blocks), dim3(kDistThreads), 0, stream, X, nullptr, \
                     nullptr, nullptr, W, nullptr, n, k, dim, bmus, dist, partial)
  if (dim < 4) SOM_DISTANCES(false, 16, 1);
  else if (dim <= 64) SOM_DISTANCES(true, 16, 1);
  else if (dim <= 128) SOM_DISTANCES(true, 32, 1);
  else if (dim <= 256) SOM_DISTANCES(true, 64, 1);
  else if (dim <= 512) SOM_DISTANCES(true, 64, 2);
  else SOM_DISTANCES(true, 64, 4);
#undef SOM_DISTANCES
  if (qerror) hipLaunchKernelGGL(k_mean_of_partials, dim3(1), dim3(64), 0, stream, partial, blocks, n, qerror);
  return hipGetLastError();
}

hipError_t launch_bmu_distances(som_ctx *c, const float *X, const int64_t *indptr, const int32_t *indices,
                                const float *values, int64_t n, const float *W, const int32_t *bmus, float *dist,
                                double *qerror) {
  if (X) return launch_bmu_distances_on(c->stream, X, n, W, c->k, c->dim, bmus, dist, qerror, c->dist_partial);
  const int64_t items = n < c->k ? n : c->k;
  hipLaunchKernelGGL(k_mark_nodes, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, bmus, n, c->k, c->dist_owner);
  hipLaunchKernelGGL(k_marked_norms, dim3((unsigned)(items < c->n_cu * 16 ? items : c->n_cu * 16)), dim3(256), 0, c->stream, W,
                     n, c->k, c->dim, bmus, c->dist_owner, c->wn64);
  const int blocks = distance_blocks(n, kWave);
  hipLaunchKernelGGL((k_bmu_distances<true, false, kWave, 1>), dim3(blocks), dim3(kDistThreads), 0, c->stream, nullptr, indptr, indices,
                     values, W, c->wn64, n, c->k, c->dim, bmus, dist, c->dist_partial);
  if (qerror) hipLaunchKernelGGL(k_mean_of_partials, dim3(1), dim3(64), 0, c->stream, c->dist_partial, blocks, n, qerror);
  return hipGetLastError();
}

hipError_t launch_rescan_csr(som_ctx *c, const int64_t *indptr, const int32_t *indices, const float *values,
                             const float *W, int32_t *bmus) {
  if (c->Wt32) {
    hipLaunchKernelGGL(k_transpose_for_rescan, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, W, c->k,
                       c->dim, c->kt32, c->list_counts, c->Wt32);
    hipLaunchKernelGGL(k_rescan_csr_t, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, indptr, indices,
                       values, W, c->Wt32, c->kt32, c->wn64, c->dim, c->k, c->rescan_list, c->list_counts, bmus);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_rescan_csr, dim3(persistent_blocks(c, 1 << 20)), dim3(256), 0, c->stream, indptr, indices,
                     values, W, c->wn64, c->dim, c->k, c->rescan_list, c->list_counts, bmus);
  return hipGetLastError();
}

}  // namespace som
