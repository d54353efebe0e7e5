// Per-node sums of the batch update (paper: batch equation; "Parallelism": the accumulation of
// local weights used to be the bottleneck when done by one process).
//
// The neighbourhood weight of an instance depends on it only through its BMU, so the update
// needs S_b = sum of the instances whose BMU is b and C_b = their number.  Dense data:
//   1. stable counting sort of the instance ids by BMU (counters of all nodes in LDS, ballot-based ranking),
//      so every segment lists its instances in ascending order; C_b and the segment offsets fall out of it
//      (maps whose counters do not fit LDS, or whose table would be too large: LSD radix sort, offsets by binary search
//      in the sorted keys);
//   2. small sets skip the sort: a workgroup per node picks its instances out of the list of BMUs;
//   3. every segment is cut into chunks of kChunkRows instances; one workgroup sums one chunk
//      (fp64 registers, instances read as whole rows through the permutation);
//   4. chunks of a node are added in order.
// No floating-point atomics: the result is bit-reproducible.  Sparse data uses the same sort and
// chunking, with a column tile in LDS per chunk and atomic adds (k_accumulate_csr below): the order of
// the additions is not fixed there, so two sparse runs agree to rounding only.
#include "epoch_tables.hpp"

namespace som {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int clamp_node(int b, int k) { return b < 0 ? 0 : (b >= k ? k - 1 : b); }

// Segment offsets of the sorted keys: seg_off[b] = first position whose key is >= b.
__global__ __launch_bounds__(256) void k_segment_bounds(const int32_t *__restrict__ sorted_keys, int64_t n, int k,
                                                        int32_t *__restrict__ seg_off,
                                                        int32_t *__restrict__ counts) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= k) return;
  int bound[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (sorted_keys[mid] < b + e) lo = mid + 1; else hi = mid;
    }
    bound[e] = (int)lo;
  }
  seg_off[b] = bound[0];
  counts[b] = bound[1] - bound[0];
  if (b == k - 1) seg_off[k] = (int32_t)n;
}

// Exclusive scan of in[0..len) into out[0..len], out[len] = total.  One workgroup of 1024 walks the
// array in steps of 4096: a thread takes four consecutive elements (one 16-byte access when the
// arrays allow it), the wavefronts scan the thread sums with shuffles and the sixteen wavefront
// totals are combined through LDS.
// `transform` > 0: scan ceil(in / transform) instead of in (chunks per node).
// in and out may be the same array (a thread reads its elements before it writes them).
__global__ __launch_bounds__(1024) void k_scan_exclusive(const int32_t *in, int32_t *out, int len, int transform) {
  __shared__ int s_wave[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool vec = (len & 3) == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  int carry = 0;
  int phase = 0;
  for (int base = 0; base < len; base += 4096, phase ^= 1) {
    const int i = base + 4 * tid;
    int v[4] = {0, 0, 0, 0};
    if (vec) {
      if (i < len) {
        const int4 q = *reinterpret_cast<const int4 *>(in + i);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i + e < len) v[e] = in[i + e];
    }
    if (transform > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (v[e] + transform - 1) / transform;
    }
    const int sum = (v[0] + v[1]) + (v[2] + v[3]);
    int inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    if (lane == 63) s_wave[phase][wave] = inc;
    __syncthreads();                       // one barrier per step: the totals alternate between two rows
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int t = s_wave[phase][w];
      before += w < wave ? t : 0;
      all += t;
    }
    int run = carry + before + inc - sum;
    if (vec) {
      if (i < len) {
        int4 q;
        q.x = run; q.y = run + v[0]; q.z = q.y + v[1]; q.w = q.z + v[2];
        *reinterpret_cast<int4 *>(out + i) = q;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (i + e < len) out[i + e] = run;
        run += v[e];
      }
    }
    carry += all;
  }
  if (tid == 0) out[len] = carry;
}

// ---------------------------------------------------------------- stable radix sort
// Digits of `bits` bits (at most 8) at `shift`; hist[digit][tile].
__global__ __launch_bounds__(256) void k_radix_hist(const int32_t *__restrict__ keys, int64_t n, int shift, int bits,
                                                    int nblk, int tile, int k, int32_t *__restrict__ hist) {
  __shared__ int s_hist[256];
  const int mask = (1 << bits) - 1;
  s_hist[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * tile;
  for (int e = threadIdx.x; e < tile; e += 256) {
    const int64_t j = base + e;
    if (j < n) atomicAdd(&s_hist[(clamp_node(keys[j], k) >> shift) & mask], 1);
  }
  __syncthreads();
  if ((int)threadIdx.x <= mask) hist[(int64_t)threadIdx.x * nblk + blockIdx.x] = s_hist[threadIdx.x];
}

// One wavefront ranks its tile 64 keys at a time, in order: a key's position is the running
// count of its digit plus the number of lower lanes holding the same digit (a ballot per digit bit).
__global__ __launch_bounds__(64) void k_radix_scatter(const int32_t *__restrict__ keys_in,
                                                      const int32_t *__restrict__ vals_in,
                                                      int32_t *__restrict__ keys_out,
                                                      int32_t *__restrict__ vals_out, int64_t n, int shift, int bits,
                                                      int nblk, int tile, int k,
                                                      const int32_t *__restrict__ hist_scanned) {
  __shared__ int s_cnt[256];
  const int lane = threadIdx.x;
  const int mask = (1 << bits) - 1;
  for (int d = lane; d <= mask; d += 64) s_cnt[d] = hist_scanned[(int64_t)d * nblk + blockIdx.x];
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * tile;
  for (int step = 0; step < tile / 64; ++step) {
    const int64_t j = base + step * 64 + lane;
    const bool valid = j < n;
    const int key = valid ? clamp_node(keys_in[j], k) : 0;
    const int val = valid ? (vals_in ? vals_in[j] : (int32_t)j) : 0;
    const int d = (key >> shift) & mask;
    unsigned long long same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (b < bits) {                              // uniform
        const bool bit = (d >> b) & 1;
        const unsigned long long bal = __ballot(bit);
        same &= bit ? bal : ~bal;
      }
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    const int before = valid ? s_cnt[d] : 0;
    __syncthreads();
    if (valid && rank == 0) s_cnt[d] = before + __popcll(same);
    __syncthreads();
    if (valid) {
      keys_out[before + rank] = key;
      vals_out[before + rank] = val;
    }
  }
}

// ---------------------------------------------------------------- counting sort by node
// The radix sort above needs three launches per digit and four more for the segments and chunks; with one counter
// per node in LDS a single digit does.  A wavefront ranks its own consecutive keys, 64 at a time, in order, with
// counters of its own (16 bits, so that several wavefronts' sets fit); the sets are then turned into exclusive
// prefixes over the wavefronts.  Up to 2,048 keys per wavefront of one workgroup the rest is done there too
// (k_group_one); beyond, a workgroup counts one tile of the keys (k_group_tiles), the tables are
// summed over the tiles and scanned within blocks of 64 nodes (k_group_prefix), and k_group_place puts the ids in place.  Measured, everything up to the chunk table (us):
// 20,011 keys, 2,700 nodes 37 -> 15; 100,000 keys, 2,500 nodes 71 -> 17; 1,000,000 keys, 10,000 nodes 144 -> 46.
constexpr size_t kGroupLds = 160 * 1024 - 1024;      // the rest is for the scan's own words
constexpr int kGroupKeysMax = 2048;                  // keys per wavefront, at most
constexpr int kGroupOneKeys = 16384;                 // keys that one workgroup sorts faster than three launches do

// Lanes whose key equals this lane's, among the valid ones: the ballots of all key bits are independent of each
// other, and a lane collects the lanes that differ from it in any of them.
__device__ __forceinline__ unsigned long long same_key_lanes(int key, bool valid, int bits) {
  unsigned long long differ = 0;
#pragma unroll
  for (int b0 = 0; b0 < 20; b0 += 4) {
    if (b0 >= bits) break;                            // uniform; the bits past the key's are equal everywhere
#pragma unroll
    for (int b = b0; b < b0 + 4; ++b) {
      const unsigned bit = ((unsigned)key >> b) & 1u;
      const unsigned long long bal = __ballot(bit);
      const unsigned long long mine = 0ull - (unsigned long long)bit;
      differ |= bal ^ mine;
    }
  }
  return ~differ & __ballot(valid);
}

// Ranks the keys lo .. hi - 1 of this wavefront against its own counters; rank_out[j] = number of earlier keys of the
// wavefront with the same value.
__device__ __forceinline__ void group_rank_wave(const int32_t *__restrict__ keys, int64_t lo, int64_t hi, int k, int bits,
                                                volatile uint16_t *cnt, int32_t *__restrict__ rank_out, int lane) {
  const unsigned long long below = (1ull << lane) - 1ull;
  int next = lo + lane < hi ? keys[lo + lane] : 0;
  for (int64_t j0 = lo; j0 < hi; j0 += 64) {
    const bool valid = j0 + lane < hi;
    const int key = valid ? clamp_node(next, k) : 0;
    if (j0 + 64 + lane < hi) next = keys[j0 + 64 + lane];
    const unsigned long long same = same_key_lanes(key, valid, bits);
    const int rank = __popcll(same & below);
    const int before = valid ? cnt[key] : 0;
    if (valid && rank == 0) cnt[key] = (uint16_t)(before + __popcll(same));
    if (valid) rank_out[j0 + lane] = before + rank;
  }
}

// Exclusive scans over the nodes of their counts and of their chunk counts by a workgroup of kThreads, into LDS (seg,
// chk: k + 1 entries each).  count(b) and chunks_of(b, count(b)) must be readable by every thread.
template <int kThreads, typename Count, typename Chunks>
__device__ __forceinline__ void group_scan(Count count, Chunks chunks_of, int k, int *seg, int *chk, int (*s_wave)[2]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (k + kThreads - 1) / kThreads;
  const int b0 = min(tid * per, k), b1 = min(b0 + per, k);
  int sum = 0, chunks = 0;
  for (int b = b0; b < b1; ++b) {
    const int v = count(b);
    sum += v;
    chunks += chunks_of(b, v);
  }
  int inc = sum, cinc = chunks;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, 64), u = __shfl_up(cinc, o, 64);
    if (lane >= o) { inc += t; cinc += u; }
  }
  if (lane == 63) { s_wave[wave][0] = inc; s_wave[wave][1] = cinc; }
  __syncthreads();
  int run = inc - sum, crun = cinc - chunks;
  for (int w = 0; w < wave; ++w) { run += s_wave[w][0]; crun += s_wave[w][1]; }
  for (int b = b0; b < b1; ++b) {
    const int v = count(b);
    seg[b] = run;
    chk[b] = crun;
    run += v;
    crun += chunks_of(b, v);
  }
  if (tid == kThreads - 1) { seg[k] = run; chk[k] = crun; }
  __syncthreads();
}

// Writes the node of every chunk of 64 nodes b0 .. b0 + 63, a lane per node: the first chunks of a node by its lane,
// the rest of a node with many by the whole wavefront.
__device__ __forceinline__ void fill_chunk_nodes(int b, int first, int chunks, int32_t *__restrict__ chunk_node, int lane) {
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (u < chunks) chunk_node[first + u] = b;
  unsigned long long more = __ballot(chunks > 4);
  for (; more; more &= more - 1) {
    const int q = __ffsll((long long)more) - 1;
    const int f = __shfl(first, q, 64), n = __shfl(chunks, q, 64), bq = __shfl(b, q, 64);
    for (int t = 4 + lane; t < n; t += 64) chunk_node[f + t] = bq;
  }
}

template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void k_group_one(const int32_t *__restrict__ keys, int n, int k, int bits,
                                                           int chunk_rows, int32_t *__restrict__ perm,
                                                           int32_t *__restrict__ rank, int32_t *__restrict__ counts,
                                                           int32_t *__restrict__ seg_off, int32_t *__restrict__ chunk_off,
                                                           int32_t *__restrict__ chunk_node) {
  extern __shared__ int s_dyn[];                      // seg [k + 1], chk [k + 1], counters [kWaves][k2]
  __shared__ int s_wave[kWaves][2];
  const int k2 = (k + 1) & ~1;
  int *seg = s_dyn, *chk = seg + k + 1;
  uint16_t *cnt = reinterpret_cast<uint16_t *>(chk + k + 1);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int kThreads = 64 * kWaves;
  for (int i = tid; i < kWaves * k2 / 2; i += kThreads) reinterpret_cast<uint32_t *>(cnt)[i] = 0u;
  __syncthreads();
  const int per = ((n + kWaves - 1) / kWaves + 63) / 64 * 64;
  const int lo = min(wave * per, n), hi = min(lo + per, n);
  group_rank_wave(keys, lo, hi, k, bits, cnt + wave * k2, rank, lane);
  __syncthreads();
  for (int b = tid; b < k; b += kThreads) {
    int t[kWaves], run = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t[w] = cnt[w * k2 + b];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      cnt[w * k2 + b] = (uint16_t)run;
      run += t[w];
    }
    counts[b] = run;
  }
  __syncthreads();                                    // (also makes counts visible to the workgroup)
  group_scan<kThreads>([&](int b) { return counts[b]; }, [&](int, int v) { return (v + chunk_rows - 1) / chunk_rows; }, k, seg, chk, s_wave);
  for (int b = tid; b <= k; b += kThreads) { seg_off[b] = seg[b]; chunk_off[b] = chk[b]; }
  for (int b0 = 64 * wave; b0 < k; b0 += kThreads) {
    const int b = b0 + lane;
    fill_chunk_nodes(b, b < k ? chk[b] : 0, b < k ? chk[b + 1] - chk[b] : 0, chunk_node, lane);
  }
  for (int j = lo + lane; j < hi; j += 64) {
    const int key = clamp_node(keys[j], k);
    perm[seg[key] + cnt[wave * k2 + key] + rank[j]] = j;
  }
}

// table[tile][node] = keys of the tile, rank[j] = position of key j among the equal ones of its tile.  kWaves of the
// wavefronts rank; all of them clear and sum the counters.  Few workgroups at work, so the chain of one is what it takes: where a wavefront has
// four steps of keys only (kSteps 4; 0: any number) it keeps them and their ranks in registers from the first
// load to the last store, and a node's counters are read together before they are written (100,000 keys on 2,500 nodes 10.4 -> 9.0 us).
constexpr int kTileThreads = 1024;

template <int kWaves, int kSteps>
__global__ __launch_bounds__(kTileThreads) void k_group_tiles(const int32_t *__restrict__ keys, int64_t n, int k, int bits,
                                                              int keys_per_wave, int32_t *__restrict__ table,
                                                              int32_t *__restrict__ rank) {
  extern __shared__ int s_dyn[];                      // counters [kWaves][k2]
  const int k2 = (k + 1) & ~1;
  uint16_t *cnt = reinterpret_cast<uint16_t *>(s_dyn);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t tile0 = (int64_t)blockIdx.x * kWaves * keys_per_wave;
  const int64_t tile1 = tile0 + kWaves * keys_per_wave < n ? tile0 + kWaves * keys_per_wave : n;
  const int64_t lo = tile0 + wave * keys_per_wave;
  int key[kSteps ? kSteps : 1], pos[kSteps ? kSteps : 1];
  if (kSteps && wave < kWaves) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s) key[s] = lo + 64 * s + lane < n ? clamp_node(keys[lo + 64 * s + lane], k) : -1;
  }
  for (int i = tid; i < kWaves * k2 / 2; i += kTileThreads) reinterpret_cast<uint32_t *>(cnt)[i] = 0u;
  __syncthreads();
  if (wave < kWaves && lo < n) {
    if (kSteps) {
      volatile uint16_t *own = cnt + wave * k2;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const bool valid = key[s] >= 0;
        const unsigned long long same = same_key_lanes(valid ? key[s] : 0, valid, bits);
        const int earlier = __popcll(same & ((1ull << lane) - 1ull));
        const int before = valid ? own[key[s]] : 0;
        if (valid && earlier == 0) own[key[s]] = (uint16_t)(before + __popcll(same));
        pos[s] = before + earlier;
      }
    } else {
      group_rank_wave(keys, lo, lo + keys_per_wave < n ? lo + keys_per_wave : n, k, bits, cnt + wave * k2, rank, lane);
    }
  }
  __syncthreads();
  for (int b = tid; b < k; b += kTileThreads) {
    int t[kWaves], run = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t[w] = cnt[w * k2 + b];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      cnt[w * k2 + b] = (uint16_t)run;
      run += t[w];
    }
    table[(int64_t)blockIdx.x * k + b] = run;
  }
  if (kSteps) {
    if (kWaves > 1) __syncthreads();
    if (wave < kWaves) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
        if (key[s] >= 0) rank[lo + 64 * s + lane] = pos[s] + (kWaves > 1 ? cnt[wave * k2 + key[s]] : 0);
    }
    return;
  }
  if (kWaves == 1) return;
  __syncthreads();
  for (int64_t j = tile0 + tid; j < tile1; j += kTileThreads)
    rank[j] += cnt[(int)(j - tile0) / keys_per_wave * k2 + clamp_node(keys[j], k)];
}

// Exclusive prefixes of the table over the tiles, in place, and the totals; besides, the exclusive scans of the totals
// and of the chunk counts within the workgroup's 64 nodes (local [2][k]) and their sums (sums [2][blocks]).  The
// wavefronts of a workgroup share the tiles (244 tiles of 10,000 nodes: 15.5 us with four).
constexpr int kPrefixWaves = 16;

__global__ __launch_bounds__(64 * kPrefixWaves) void k_group_prefix(int32_t *__restrict__ table, int tiles, int k, int chunk_rows,
                                                      int32_t *__restrict__ counts, int32_t *__restrict__ local,
                                                      int32_t *__restrict__ sums) {
  __shared__ int s_sum[kPrefixWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.x * 64 + lane;
  const bool live = b < k;
  const int per = (tiles + kPrefixWaves - 1) / kPrefixWaves;
  const int t0 = min(wave * per, tiles), t1 = min(t0 + per, tiles);
  int32_t *col = table + (live ? b : 0);
  int sum = 0;
#pragma unroll 8
  for (int t = t0; t < t1; ++t) sum += col[(int64_t)t * k];
  s_sum[wave][lane] = sum;
  __syncthreads();
  int run = 0;
  for (int w = 0; w < wave; ++w) run += s_sum[w][lane];
  if (wave == kPrefixWaves - 1) {
    const int total = live ? run + sum : 0, chunks = (total + chunk_rows - 1) / chunk_rows;
    int inc = total, cinc = chunks;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64), u = __shfl_up(cinc, o, 64);
      if (lane >= o) { inc += t; cinc += u; }
    }
    if (live) {
      counts[b] = total;
      local[b] = inc - total;
      local[k + b] = cinc - chunks;
    }
    if (lane == 63) { sums[blockIdx.x] = inc; sums[gridDim.x + blockIdx.x] = cinc; }
  }
#pragma unroll 8
  for (int t = t0; t < t1; ++t) {
    const int v = col[(int64_t)t * k];
    if (live) col[(int64_t)t * k] = run;
    run += v;
  }
}

// Every workgroup scans the sums of the 64-node blocks (at most kGroupMaxBlocks of them) for itself.
constexpr int kGroupMaxBlocks = 1280;

__global__ __launch_bounds__(1024) void k_group_place(const int32_t *__restrict__ keys, int64_t n, int k, int tile,
                                                      int chunk_rows, const int32_t *__restrict__ table,
                                                      const int32_t *__restrict__ rank, const int32_t *__restrict__ counts,
                                                      const int32_t *__restrict__ local, const int32_t *__restrict__ sums,
                                                      int32_t *__restrict__ perm, int32_t *__restrict__ seg_off,
                                                      int32_t *__restrict__ chunk_off, int32_t *__restrict__ chunk_node) {
  __shared__ int s_wave[16][2];
  __shared__ int s_seg[kGroupMaxBlocks + 1], s_chk[kGroupMaxBlocks + 1];
  const int blocks = (k + 63) / 64;
  group_scan<1024>([&](int b) { return sums[b]; }, [&](int b, int) { return sums[blocks + b]; }, blocks, s_seg, s_chk, s_wave);
  const int64_t at = (int64_t)blockIdx.x * 1024 + threadIdx.x, stride = (int64_t)gridDim.x * 1024;
  const int lane = threadIdx.x & 63;
  for (int64_t b0 = at - lane; b0 < k; b0 += stride) {
    const int b = (int)b0 + lane;
    int first = 0, chunks = 0;
    if (b < k) {
      first = local[k + b] + s_chk[b >> 6];
      chunks = (counts[b] + chunk_rows - 1) / chunk_rows;
      seg_off[b] = local[b] + s_seg[b >> 6];
      chunk_off[b] = first;
    }
    fill_chunk_nodes(b, first, chunks, chunk_node, lane);
  }
  if (at == 0) { seg_off[k] = s_seg[blocks]; chunk_off[k] = s_chk[blocks]; }
  for (int64_t j = at; j < n; j += stride) {
    const int key = clamp_node(keys[j], k);
    perm[local[key] + s_seg[key >> 6] + table[j / tile * k + key] + rank[j]] = (int32_t)j;
  }
}

// Wavefronts whose counters fit LDS beside `extra` bytes per node; 0: not even one's.
static int group_waves(int k, int extra) {
  for (int w = 16; w >= 1; w /= 2)
    if ((size_t)w * (size_t)((k + 1) & ~1) * 2 + (size_t)extra * ((size_t)k + 1) <= kGroupLds) return w;
  return 0;
}

// Keys per wavefront of the tiled form: workgroups enough to spread over the chip, as long as the table that they write and the next launch adds up stays
// at a few million entries (1,000,000 keys on 10,000 nodes, limit of half a million -> 2.5: tiles 42 -> 18.5 us, prefixes 7 -> 8.2; 50,000 on
// 40,000: 28 -> 14, 5 -> 7.4).
constexpr int64_t kGroupTableFine = 2500000;
static int group_keys_per_wave(int k, int64_t n, int waves) {
  int per = 256;
  while (per < kGroupKeysMax && (n + (int64_t)per * waves - 1) / ((int64_t)per * waves) * k > kGroupTableFine) per *= 2;
  return per;
}

// Wavefronts of a tile: ranking costs some 130 vector instructions per 64 keys, so four that have a SIMD each are done sooner than sixteen, as long
// as the tiles leave CUs idle (100,000 keys on 2,500 nodes: 9.0 -> 5.6 us, their prefixes 5.0 -> 5.6).
static int group_tile_waves(int k, int64_t n) {
  int w = group_waves(k, 0);
  while (w > 4 && n <= (int64_t)w * 256 * 128 && (n + 128 * w - 1) / (128 * w) * k <= kGroupTableFine) w /= 2;
  return w;
}

// The tiled form reads and writes its table three times, and from some 30 million entries on (128 MB: most of the
// memory-side cache) that costs more than the radix sort's passes over the keys.  Counting / radix, update of four
// columns in us: 20,164 nodes, 8,000,000 keys (20 million entries) 824 / 983; 57,600 nodes, 1,000,000 keys (28 million)
// 356 / 403; 81,225 nodes, 1,000,000 keys (40 million) 582 / 572; 25,600 nodes, 8,000,000 keys (50 million) 1,119 / 1,004;
// 81,225 nodes, 8,000,000 keys (317 million) 2,496 / 1,257.
constexpr int64_t kGroupTableMax = 32 << 20;

// Entries of the tiled form's table; 0: its counters do not fit LDS, or the table would be too large.
static int64_t group_tiled_entries(int k, int64_t n) {
  const int waves = group_tile_waves(k, n);
  if (!waves || k > 64 * kGroupMaxBlocks) return 0;
  const int64_t tile = (int64_t)waves * group_keys_per_wave(k, n, waves);
  const int64_t entries = (n + tile - 1) / tile * k;
  return entries <= kGroupTableMax ? entries : 0;
}

int64_t group_table_entries(int k, int64_t n) {
  if (!group_waves(k, 0) || k > 64 * kGroupMaxBlocks) return 1;
  // (a shorter list may be cut finer, but then its table has no more entries than the finest cut of this one and at most
  // kGroupTableFine; where this one is too long for the tiled form a shorter one need not be)
  const int64_t own = group_tiled_entries(k, n), least = group_waves(k, 0) < 4 ? group_waves(k, 0) : 4;
  const int64_t finest = (n / (256 * least) + 2) * k;
  const int64_t fine = finest < kGroupTableFine ? finest : kGroupTableFine, most = own > fine ? own : fine;
  return own ? most : kGroupTableMax;
}

// ---------------------------------------------------------------- small sets: a workgroup per node
// With few instances on few nodes the sort costs more than every node's looking through all BMUs: workgroup b
// compacts the ids of its instances, in ascending order, and adds them up: kRowLanes rows at a time over the
// columns of its column block, the row lanes' sums combined in order.  Bound by latency: 1,000 x 10 on 400 nodes
// 5 us instead of 45 for sort, chunks and sums.
constexpr int kGatherThreads = 512;
constexpr int kGatherMax = 8192;          // instances (their ids fit 16 bits of LDS each; 16 per thread)

__global__ __launch_bounds__(kGatherThreads) void k_gather_sums(const float *__restrict__ X, const int32_t *__restrict__ bmus,
                                                                int n, int k, int dim, int col_lanes,
                                                                int32_t *__restrict__ counts, float *__restrict__ S,
                                                                EpochTables tables, EpochSchedule schedule) {
  constexpr int kWaves = kGatherThreads / 64, kPer = kGatherMax / kGatherThreads;
  __shared__ uint16_t s_list[kGatherMax];
  __shared__ int s_cnt[kWaves];
  __shared__ double s_part[kGatherThreads];
  const int b = blockIdx.x;
  if (b >= k) {                               // what the smoothing needs of the epoch's radius (params null: it is there)
    if (blockIdx.y == 0 && tables.params)
      write_epoch_tables(tables, schedule, (int64_t)(b - k) * kGatherThreads + threadIdx.x, (int64_t)(gridDim.x - k) * kGatherThreads);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // wavefront w looks through the w-th stretch of the list, 64 instances at a time; all its loads are in flight at once
  const int steps = (n + kGatherThreads - 1) / kGatherThreads;
  const int lo = wave * steps * 64;
  int key[kPer];
#pragma unroll
  for (int s = 0; s < kPer; ++s)
    if (s < steps) {                          // uniform
      const int j = lo + 64 * s + lane;
      key[s] = j < n ? clamp_node(bmus[j], k) : -1;
    }
  unsigned mine = 0;                          // bit s: this lane's instance of step s belongs to the node
  int found = 0;
#pragma unroll
  for (int s = 0; s < kPer; ++s)
    if (s < steps) {
      if (key[s] == b) mine |= 1u << s;
      found += __popcll(__ballot(key[s] == b));
    }
  if (lane == 0) s_cnt[wave] = found;
  __syncthreads();
  int at = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int t = s_cnt[w];
    if (w < wave) at += t;
    total += t;
  }
  if (found)
    for (int s = 0; s < steps; ++s) {
      const unsigned long long bal = __ballot((mine >> s) & 1u);
      if ((mine >> s) & 1u) s_list[at + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(lo + 64 * s + lane);
      at += __popcll(bal);
    }
  __syncthreads();
  const int row_lanes = kGatherThreads / col_lanes;
  const int cl = tid % col_lanes, rl = tid / col_lanes;
  const int c = blockIdx.y * col_lanes + cl;
  const bool live = c < dim;
  const float *col = X + (live ? c : 0);
  double sum = 0.0;
  for (int r = rl; r < total; r += 8 * row_lanes) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = col[(int64_t)s_list[min(r + u * row_lanes, total - 1)] * dim];      // (no branch: all in flight)
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += r + u * row_lanes < total ? (double)v[u] : 0.0;
  }
  s_part[tid] = sum;
  __syncthreads();
  if (rl == 0) {
    double s = s_part[cl];
    for (int r = 1; r < row_lanes; ++r) s += s_part[r * col_lanes + cl];
    if (live) S[(int64_t)b * dim + c] = (float)s;
  }
  if (tid == 0 && blockIdx.y == 0) counts[b] = total;
}

// The nodes' looking through the list (8e6 comparisons take about as long as a launch) and the worst case, all rows
// on one node (2^18 values: 20 us), draw the line.
bool gather_pays(const som_ctx *c, int64_t n) {
  return n <= kGatherMax && n * (int64_t)c->k * ((c->dim + 255) / 256) <= 8000000 && n * (int64_t)c->dim <= 262144;
}

// ---------------------------------------------------------------- chunks
__global__ __launch_bounds__(256) void k_fill_chunk_nodes(const int32_t *__restrict__ chunk_off, int k,
                                                          int32_t *__restrict__ chunk_node) {
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int nwaves = gridDim.x * 4;
  for (int b = wave; b < k; b += nwaves)
    for (int t = chunk_off[b] + lane; t < chunk_off[b + 1]; t += 64) chunk_node[t] = b;
}

template <bool kVec4>
__global__ __launch_bounds__(256) void k_accumulate_dense(const float *__restrict__ X, int dim,
                                                          const int32_t *__restrict__ perm,
                                                          const int32_t *__restrict__ seg_off,
                                                          const int32_t *__restrict__ chunk_off,
                                                          const int32_t *__restrict__ chunk_node, int k,
                                                          float *__restrict__ S, float *__restrict__ partial) {
  __shared__ int s_rows[kChunkRows];
  const int chunk = blockIdx.x;
  if (chunk >= chunk_off[k]) return;
  const int b = chunk_node[chunk];
  const int first_chunk = chunk_off[b];
  const int lo = seg_off[b] + (chunk - first_chunk) * kChunkRows;
  const int hi = min(lo + kChunkRows, seg_off[b + 1]);
  const int nrows = hi - lo;
  if (threadIdx.x < nrows) s_rows[threadIdx.x] = perm[lo + threadIdx.x];
  __syncthreads();
  const bool single = (chunk_off[b + 1] - first_chunk) == 1;
  float *dst = single ? S + (int64_t)b * dim : partial + (int64_t)chunk * dim;
  if (kVec4) {
    for (int q = threadIdx.x; q < dim / 4; q += blockDim.x) {
      double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
      for (int r = 0; r < nrows; ++r) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(X + (int64_t)s_rows[r] * dim + 4 * q);
        a0 += (double)v[0]; a1 += (double)v[1]; a2 += (double)v[2]; a3 += (double)v[3];
      }
      f32x4 o = {(float)a0, (float)a1, (float)a2, (float)a3};
      *reinterpret_cast<f32x4 *>(dst + 4 * q) = o;
    }
  } else {
    for (int c = threadIdx.x; c < dim; c += blockDim.x) {
      double a = 0;
      for (int r = 0; r < nrows; ++r) a += (double)X[(int64_t)s_rows[r] * dim + c];
      dst[c] = (float)a;
    }
  }
}

// Nodes with many chunks (early in training a few nodes hold most of the instances, thousands of chunks
// each; one workgroup adding them one after the other took three times as long as computing them): every
// group of kCombineGroup consecutive chunks of such a node is first added up, in place, into the group's
// first chunk.  One workgroup per chunk slot; only the group leaders of large nodes do anything.
constexpr int kCombineGroup = 32;

__global__ __launch_bounds__(256) void k_combine_groups(const int32_t *__restrict__ chunk_off,
                                                        const int32_t *__restrict__ chunk_node, int k, int dim,
                                                        float *__restrict__ partial) {
  const int chunk = blockIdx.x;
  if (chunk >= chunk_off[k]) return;
  const int b = chunk_node[chunk];
  const int c0 = chunk_off[b], nc = chunk_off[b + 1] - c0;
  const int at = chunk - c0;
  if (nc <= kCombineGroup || at % kCombineGroup != 0) return;
  const int len = min(kCombineGroup, nc - at);
  float *dst = partial + (int64_t)chunk * dim;
  for (int c = blockIdx.y * blockDim.x + threadIdx.x; c < dim; c += gridDim.y * blockDim.x) {
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int t = 0;
    for (; t + 8 <= len; t += 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] += (double)dst[(int64_t)(t + u) * dim + c];
    for (int u = 0; t < len; ++t, ++u) a[u] += (double)dst[(int64_t)t * dim + c];
    dst[c] = (float)(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
  }
}

// Empty node: zero row.  One chunk: already written.  Several: add the partial rows (of a node with more
// than kCombineGroup chunks: the group sums k_combine_groups left in every kCombineGroup-th row), eight
// interleaved running sums (term t goes to sum t mod 8) combined pairwise at the end: a fixed order, with
// eight loads in flight instead of one.
__global__ __launch_bounds__(256) void k_combine_chunks(const int32_t *__restrict__ chunk_off, int dim,
                                                        const float *__restrict__ partial, float *__restrict__ S) {
  const int b = blockIdx.x;
  const int c0 = chunk_off[b], nc = chunk_off[b + 1] - c0;
  if (nc == 1) return;
  float *dst = S + (int64_t)b * dim;
  const bool grouped = nc > kCombineGroup;
  const int terms = grouped ? (nc + kCombineGroup - 1) / kCombineGroup : nc;
  const int64_t step = (int64_t)(grouped ? kCombineGroup : 1) * dim;
  const float *src = partial + (int64_t)c0 * dim;
  // grid.y splits the columns: late in training a few dozen nodes hold all the chunks
  for (int c = blockIdx.y * blockDim.x + threadIdx.x; c < dim; c += gridDim.y * blockDim.x) {
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int t = 0;
    for (; t + 8 <= terms; t += 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] += (double)src[(t + u) * step + c];
    for (int u = 0; t < terms; ++t, ++u) a[u] += (double)src[t * step + c];
    dst[c] = (float)(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
  }
}

// ---------------------------------------------------------------- sparse rows
// S_b for CSR data.
//
// The instances are sorted by BMU as in the dense path and cut into chunks of kCsrChunkRows; a workgroup adds the nonzeros of its
// chunk into a copy of the node's row in LDS (LDS atomics: the rows of a node share their frequent columns), one tile of columns
// after the other.  A node with a single chunk is then written with plain stores, zeros included, so its row needs no clearing
// beforehand; the chunks of a larger node add their nonzero entries to a row cleared by k_zero_rows_if.
//
// Bound by the chain of loads that leads to a chunk's entries (chunk, node, ids, row bounds, entries) and, with long rows, by writing
// S.  So the chain is walked once per chunk: it has as many rows as eight wavefronts keep in registers, eight each, and
// the tiles take their entries from there (a tile as a workgroup of its own, chunks of 256 rows: 302 us on 100,000 rows of 50,000 columns
// and 100 nonzeros, 2,500 nodes; chunks of 256 / 128 / 64 rows with the first ones kept: 223 / 208 / 192, 1.0 GB moved; clearing S and
// one global atomic for each nonzero outside the 256 most frequent columns: 451; what is beyond 128 entries dealt out: 177).  5e6 nonzeros in
// rows of 1,000 columns: 82 -> 42 us.  Few chunks of many tiles leave the chip idle, so their tiles are shared out until there are kCsrFill workgroups per CU
// (whole update, us, atomics / a chunk's tiles by one workgroup / shared out: 16 nodes of 200,000 columns, 32 instances of 100 nonzeros
// 59 / 76 / 53, 3,200 of 2,000 355 / 1,359 / 185; 100 nodes of 50,000, 4,000 of 4,000 534 / 721 / 246).
//
// Everything goes straight into S instead, the chosen rows cleared and a global atomic for every nonzero in instance order, where that is less:
// long rows with fewer than kTileFrom instances per node, where the sort costs more (the whole update, atomics / tiles, us: 2,500 nodes of
// 20,000 columns, one instance per node 241 / 248, two 266 / 273 evenly spread and 265 / 255 skewed, eight 334 / 303 and 400 / 293; two of
// 13,100 columns 214 / 208, of 16,000 242 / 226); and rows of more than kTilesMax tiles, where going through the tiles costs more than
// the atomics save (100 nodes, 10,000 instances of 20 / 500 / 2,000 nonzeros: 300,000 columns 218 / 242, 449 / 410, 1,127 / 795; 400,000 274 /
// 310, 506 / 539, 1,192 / 1,061; 600,000 402 / 451, 621 / 727, 1,319 / 1,486; 1,000,000 637 / 719, 857 / 1,164, 1,556 / 2,263).
//
// Where a node has few entries most of eight wavefronts have nothing to do and take their time to start: four then, four rows each at a time
// (whole update, us, eight wavefronts / four / two: 10,000 nodes, rows of 200 columns and 20 nonzeros, 1 / 4 / 10 evenly spread instances per node
// 101 / 88 / 83, 118 / 96 / 90, 123 / 100 / 100; 1,000 and 100 122 / 110 / 107, 144 / 130 / 131, 164 / 159 / 163; 40,000 nodes, 2,000 and 100, 2 per node
// 785 / 721 / 697; 2,500 nodes, 1,000 and 100, 10 per node 73 / 76 / 76, 20 86 / 90 / 89; but instances as an epoch's search leaves them, in
// epochs, four / two: 14,733 instances of 12,857 columns and 100 nonzeros on 8,816 nodes 3,141 / 3,160, 2,592 of 392 and 25 on 800 127 / 133).
// Not with fewer nodes than CUs, where the chain of a chunk's batches is what it takes (1,270 instances of 307 and 12 on 108 nodes 87 / 89 / 92).
//
// Up to about a hundred instances of short rows per node: chunks of 128, which most nodes fit, so that a node is still written once. Each half
// of the wavefronts adds its 64 rows to a copy of its own, so no sum is longer than in a chunk of 64 (whole update, us, chunks of 64 / of
// 128: 900 nodes of 4,000 columns, 100 nonzeros, 60 instances per node 107 / 103, 90 138 / 118, 104 129 / 128; 256 of 1,000, 40 57 / 58, 64 78 / 69,
// 90 66 / 63, 104 74 / 77; with 100 nodes, which don't fill the chip, 100 per node 54 / 59; beyond, the second chunk of a node is nearly empty:
// 130 145 / 153).
constexpr int kCsrChunkRows = 64;         // (or twice as many, in two copies of the row)
constexpr int kCsrTile = 13056;           // columns of a row copy in LDS (51 KB: three workgroups per CU)
constexpr int64_t kTileFrom = 2, kTilesMax = 32, kCsrFill = 6, kCsrFewEntries = 768;
static_assert(kCsrChunkRows % kChunkRows == 0, "the chunk tables are sized for kChunkRows");

// Clears the rows of S whose node has more than `lo` instances.
__global__ __launch_bounds__(256) void k_zero_rows_if(const int32_t *__restrict__ counts, int lo, int dim,
                                                      float *__restrict__ S) {
  const int b = blockIdx.x;
  if (counts[b] <= lo) return;
  float *dst = S + (int64_t)b * dim;
  for (int c = blockIdx.y * 256 + threadIdx.x; c < dim; c += gridDim.y * 256) dst[c] = 0.f;
}

// A lane holds the bounds of one row of the batch at hand, kEach rows to a wavefront, which keeps entries lane and lane + 64 of its own; what lies
// beyond is dealt to the wavefronts in pieces of 256 entries and read again for every tile.  With more than one batch to a chunk there
// is one tile.  grid.y: the tiles of a chunk are shared out.  kCopies = 2: the wavefronts' halves have a copy of the row each.
template <int kWaves, int kEach, int kCopies>
__global__ __launch_bounds__(64 * kWaves) void k_accumulate_csr(const int64_t *__restrict__ indptr,
                                                                const int32_t *__restrict__ indices,
                                                                const float *__restrict__ values, int dim, int tile,
                                                                const int32_t *__restrict__ perm,
                                                                const int32_t *__restrict__ seg_off,
                                                                const int32_t *__restrict__ chunk_off,
                                                                const int32_t *__restrict__ chunk_node, int k,
                                                                float *__restrict__ S) {
  constexpr int kThreads = 64 * kWaves, kBatch = kWaves * kEach, kRows = kCsrChunkRows * kCopies;
  static_assert(kBatch <= kWave && kRows % kBatch == 0, "a lane for every row of a batch");
  extern __shared__ float4 s_row4[];          // kCopies x tile floats
  float *s_row = reinterpret_cast<float *>(s_row4);
  const int chunk = blockIdx.x;
  if (chunk >= chunk_off[k]) return;          // uniform over the workgroup
  const int b = chunk_node[chunk];
  const int first_chunk = chunk_off[b];
  int lo = seg_off[b] + (chunk - first_chunk) * kRows;
  const int hi = min(lo + kRows, seg_off[b + 1]);
  const bool single = (chunk_off[b + 1] - first_chunk) == 1;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float *own = kCopies > 1 ? s_row + (2 * wave / kWaves) * tile : s_row;
  int64_t from;
  int length;
  int ec[kEach][2];
  float ev[kEach][2];
  auto start = [&](int r) {                   // scalars: the address of a load is one pair of them and the lane
    return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)from, r) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)from >> 32), r) << 32);
  };
  auto load = [&] {
    from = 0;
    length = 0;
    if (lane < kBatch && lo + lane < hi) {
      const int64_t j = perm[lo + lane];
      from = indptr[j];
      length = (int)(indptr[j + 1] - from);
    }
#pragma unroll
    for (int t = 0; t < kEach; ++t) {
      const int r = wave + kWaves * t, len = __builtin_amdgcn_readlane(length, r);
      const int32_t *ip = indices + start(r);
      const float *vp = values + start(r);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (lane + 64 * u < len) {
          ec[t][u] = ip[lane + 64 * u];
          ev[t][u] = vp[lane + 64 * u];
        }
    }
  };
  const int tiles = (dim + tile - 1) / tile, per = (tiles + (int)gridDim.y - 1) / (int)gridDim.y;
  const int c_end = min(((int)blockIdx.y + 1) * per * tile, dim);      // (few tiles: no overflow)
  load();
  for (int c0 = (int)blockIdx.y * per * tile; c0 < c_end; c0 += tile) {
    const int width = min(tile, dim - c0);
    for (int c = threadIdx.x; 4 * c < kCopies * tile; c += kThreads) s_row4[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    auto add = [&](int c, float v) {
      const unsigned at = (unsigned)(min(max(c, 0), dim - 1) - c0);
      if (at < (unsigned)width) atomicAdd(&own[at], v);
    };
    for (;;) {
#pragma unroll
      for (int t = 0; t < kEach; ++t) {
        const int len = __builtin_amdgcn_readlane(length, wave + kWaves * t);
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (lane + 64 * u < len) add(ec[t][u], ev[t][u]);
      }
      int before = 0;                         // pieces of the long rows before this one
      for (unsigned long long m = __ballot(length > 128); m; m &= m - 1) {
        const int r = __ffsll((long long)m) - 1, len = __builtin_amdgcn_readlane(length, r), pieces = (len - 128 + 255) / 256;
        const int32_t *ip = indices + start(r);
        const float *vp = values + start(r);
        for (int q = (wave - before) & (kWaves - 1); q < pieces; q += kWaves) {
          const int x = 128 + 256 * q + lane;
          int xc[4];
          float xv[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {       // (no branch: all in flight)
            xc[u] = ip[min(x + 64 * u, len - 1)];
            xv[u] = vp[min(x + 64 * u, len - 1)];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (x + 64 * u < len) add(xc[u], xv[u]);
        }
        before += pieces;
      }
      if (lo + kBatch >= hi) break;           // uniform over the workgroup
      lo += kBatch;
      load();
    }
    __syncthreads();
    float *dst = S + (int64_t)b * dim + c0;
    if (single && (dim & 3) == 0) {           // tiles are whole fours, so are the rows: 16 bytes a lane
      for (int c = threadIdx.x; 4 * c < width; c += kThreads) {
        float4 v = s_row4[c];
        if (kCopies > 1) {
          const float4 w = s_row4[tile / 4 + c];
          v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
        }
        reinterpret_cast<float4 *>(dst)[c] = v;
      }
    } else {
      for (int c = threadIdx.x; c < width; c += kThreads) {
        const float v = kCopies > 1 ? s_row[c] + s_row[tile + c] : s_row[c];
        if (single) dst[c] = v;
        else if (v != 0.f) unsafeAtomicAdd(dst + c, v);
      }
    }
    if (c0 + tile < c_end) __syncthreads();      // other threads clear the tile for the next one
  }
}

// C_b for the sparse path.  Trained maps send most instances to few nodes, so the lanes of a
// wavefront that hold the same node are merged into one atomic add.
__global__ __launch_bounds__(256) void k_count_bmus(const int32_t *__restrict__ bmus, int64_t n, int k,
                                                    int32_t *__restrict__ counts) {
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t rounds = (n + stride - 1) / stride;
  for (int64_t r = 0; r < rounds; ++r) {
    const int64_t j = r * stride + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool pending = j < n;
    const int b = pending ? clamp_node(bmus[j], k) : 0;
    unsigned long long todo = __ballot(pending);
    while (todo) {
      const int leader = __ffsll((long long)todo) - 1;
      const int lb = __shfl(b, leader, 64);
      const unsigned long long same = __ballot(pending && b == lb);
      if (lane == leader) atomicAdd(&counts[lb], __popcll(same));
      if (pending && b == lb) pending = false;
      todo &= ~same;
    }
  }
}

__global__ __launch_bounds__(256) void k_scatter_csr(const int64_t *__restrict__ indptr,
                                                     const int32_t *__restrict__ indices,
                                                     const float *__restrict__ values, int64_t n, int dim, int k,
                                                     const int32_t *__restrict__ bmus, float *__restrict__ S) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  for (int64_t j = wave; j < n; j += nwaves) {
    float *dst = S + (int64_t)clamp_node(bmus[j], k) * dim;
    for (int64_t p = indptr[j] + lane; p < indptr[j + 1]; p += 64) {
      int c = indices[p];
      c = c < 0 ? 0 : (c >= dim ? dim - 1 : c);
      unsafeAtomicAdd(dst + c, values[p]);
    }
  }
}

// Stable permutation of the ids 0 .. n - 1 by integer keys in [0, key_range) (larger keys are clamped).
// On return c->sort_val[0] holds the permutation, c->sort_key[0] the sorted keys.
static hipError_t launch_sort_keys(som_ctx *c, const int32_t *bmus, int64_t n, int key_range) {
  const RadixPlan plan = radix_plan(n, key_range);
  const int bins = 1 << plan.digit_bits;
  const int32_t *kin = bmus;
  const int32_t *vin = nullptr;
  // an even number of hops ends in buffer 0: start in buffer 1 when the pass count is even
  int dst = (plan.passes % 2 == 0) ? 1 : 0;
  for (int p = 0; p < plan.passes; ++p) {
    hipLaunchKernelGGL(k_radix_hist, dim3(plan.nblk), dim3(256), 0, c->stream, kin, n, plan.digit_bits * p,
                       plan.digit_bits, plan.nblk, plan.tile, key_range, c->radix_hist);
    hipLaunchKernelGGL(k_scan_exclusive, dim3(1), dim3(1024), 0, c->stream, c->radix_hist, c->radix_hist,
                       bins * plan.nblk, 0);
    hipLaunchKernelGGL(k_radix_scatter, dim3(plan.nblk), dim3(64), 0, c->stream, kin, vin, c->sort_key[dst],
                       c->sort_val[dst], n, plan.digit_bits * p, plan.digit_bits, plan.nblk, plan.tile, key_range,
                       c->radix_hist);
    kin = c->sort_key[dst];
    vin = c->sort_val[dst];
    dst ^= 1;
  }
  return hipGetLastError();
}

template <int kWaves>
static void launch_group_one(som_ctx *c, const int32_t *bmus, int64_t n, int bits, int chunk_rows) {
  const size_t lds = (size_t)kWaves * ((c->k + 1) & ~1) * 2 + 8 * ((size_t)c->k + 1);
  hipLaunchKernelGGL(k_group_one<kWaves>, dim3(1), dim3(64 * kWaves), lds, c->stream, bmus, (int)n, c->k, bits, chunk_rows,
                     c->sort_val[0], c->sort_key[1], c->counts, c->seg_off, c->chunk_off, c->chunk_node);
}

template <int kWaves>
static void launch_group_tiles(som_ctx *c, const int32_t *bmus, int64_t n, int bits, int per, unsigned tiles) {
  const size_t lds = (size_t)kWaves * ((c->k + 1) & ~1) * 2;
  if (per == 256)
    hipLaunchKernelGGL((k_group_tiles<kWaves, 4>), dim3(tiles), dim3(kTileThreads), lds, c->stream, bmus, n, c->k, bits, per,
                       c->group_table, c->sort_key[1]);
  else
    hipLaunchKernelGGL((k_group_tiles<kWaves, 0>), dim3(tiles), dim3(kTileThreads), lds, c->stream, bmus, n, c->k, bits, per,
                       c->group_table, c->sort_key[1]);
}

// Stable permutation of the instance ids by BMU (c->sort_val[0]), counts, segment offsets, chunk offsets and the
// node of every chunk, for chunks of chunk_rows instances.
static hipError_t launch_group_by_bmu(som_ctx *c, const int32_t *bmus, int64_t n, int chunk_rows) {
  int bits = 1;
  while ((1ll << bits) < (long long)c->k) ++bits;
  const int one = group_waves(c->k, 8), many = group_tile_waves(c->k, n);
  if (one && n <= kGroupOneKeys && n <= (int64_t)one * kGroupKeysMax) {
    switch (one) {
      case 16: launch_group_one<16>(c, bmus, n, bits, chunk_rows); break;
      case 8: launch_group_one<8>(c, bmus, n, bits, chunk_rows); break;
      case 4: launch_group_one<4>(c, bmus, n, bits, chunk_rows); break;
      case 2: launch_group_one<2>(c, bmus, n, bits, chunk_rows); break;
      default: launch_group_one<1>(c, bmus, n, bits, chunk_rows);
    }
    return hipGetLastError();
  }
  if (group_tiled_entries(c->k, n) > 0) {
    const int per = group_keys_per_wave(c->k, n, many);
    const int tile = many * per;
    const unsigned tiles = (unsigned)((n + tile - 1) / tile);
    switch (many) {
      case 16: launch_group_tiles<16>(c, bmus, n, bits, per, tiles); break;
      case 8: launch_group_tiles<8>(c, bmus, n, bits, per, tiles); break;
      case 4: launch_group_tiles<4>(c, bmus, n, bits, per, tiles); break;
      case 2: launch_group_tiles<2>(c, bmus, n, bits, per, tiles); break;
      default: launch_group_tiles<1>(c, bmus, n, bits, per, tiles);
    }
    const int nodeblocks = (c->k + 63) / 64;
    int32_t *local = c->group_local, *sums = c->group_local + 2 * (size_t)c->k;
    hipLaunchKernelGGL(k_group_prefix, dim3(nodeblocks), dim3(64 * kPrefixWaves), 0, c->stream, c->group_table, (int)tiles, c->k, chunk_rows,
                       c->counts, local, sums);
    int64_t blocks = ((n > c->k ? n : c->k) + 1023) / 1024;
    if (blocks > 2 * (int64_t)c->n_cu) blocks = 2 * (int64_t)c->n_cu;
    hipLaunchKernelGGL(k_group_place, dim3((unsigned)blocks), dim3(1024), 0, c->stream, bmus, n, c->k, tile, chunk_rows,
                       c->group_table, c->sort_key[1], c->counts, local, sums, c->sort_val[0], c->seg_off, c->chunk_off,
                       c->chunk_node);
    return hipGetLastError();
  }
  hipError_t e = launch_sort_keys(c, bmus, n, c->k);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_segment_bounds, dim3((c->k + 255) / 256), dim3(256), 0, c->stream, c->sort_key[0], n, c->k,
                     c->seg_off, c->counts);
  hipLaunchKernelGGL(k_scan_exclusive, dim3(1), dim3(1024), 0, c->stream, c->counts, c->chunk_off, c->k, chunk_rows);
  hipLaunchKernelGGL(k_fill_chunk_nodes, dim3(c->n_cu * 2), dim3(256), 0, c->stream, c->chunk_off, c->k, c->chunk_node);
  return hipGetLastError();
}

// Order of the instances by a key below k: the permutation alone (c->sort_val[0]; the tables of the grouping are scratch).
hipError_t launch_order_by_key(som_ctx *c, const int32_t *keys, int64_t n) {
  return launch_group_by_bmu(c, keys, n, 1 << 20);
}

hipError_t launch_scan_exclusive_i32(som_ctx *c, const int32_t *in, int32_t *out, int len) {
  hipLaunchKernelGGL(k_scan_exclusive, dim3(1), dim3(1024), 0, c->stream, in, out, len, 0);
  return hipGetLastError();
}

// tables: where the epoch is in its schedule, if its tables are still to be written (then gather_pays(c, n) holds).
hipError_t launch_accumulate_dense(som_ctx *c, const float *X, int64_t n, const int32_t *bmus, const EpochSchedule *tables) {
  if (gather_pays(c, n)) {
    int col_lanes = 16;
    while (col_lanes < c->dim && col_lanes < 256) col_lanes *= 2;
    EpochTables t{};
    int64_t work = 0;
    if (tables) t = epoch_tables(c, false, &work);
    const int64_t more = (work + kGatherThreads - 1) / kGatherThreads;
    const int blocks = c->k + (int)(more < 4 * c->n_cu ? more : 4 * c->n_cu);
    hipLaunchKernelGGL(k_gather_sums, dim3(blocks, (c->dim + col_lanes - 1) / col_lanes), dim3(kGatherThreads), 0, c->stream, X,
                       bmus, (int)n, c->k, c->dim, col_lanes, c->counts, c->S, t, tables ? *tables : EpochSchedule{});
    return hipGetLastError();
  }
  const hipError_t e = launch_group_by_bmu(c, bmus, n, kChunkRows);
  if (e != hipSuccess) return e;
  int64_t max_chunks = n / kChunkRows + (n < c->k ? n : c->k);
  if (max_chunks < 1) max_chunks = 1;
  const bool vec4 = (c->dim % 4 == 0) && ((uintptr_t)X % 16 == 0);
  int threads = vec4 ? c->dim / 4 : c->dim;
  threads = ((threads + 63) / 64) * 64;
  if (threads > 256) threads = 256;
  if (threads < 64) threads = 64;
  if (vec4)
    hipLaunchKernelGGL(k_accumulate_dense<true>, dim3((unsigned)max_chunks), dim3(threads), 0, c->stream, X,
                       c->dim, c->sort_val[0], c->seg_off, c->chunk_off, c->chunk_node, c->k, c->S, c->partial);
  else
    hipLaunchKernelGGL(k_accumulate_dense<false>, dim3((unsigned)max_chunks), dim3(threads), 0, c->stream, X,
                       c->dim, c->sort_val[0], c->seg_off, c->chunk_off, c->chunk_node, c->k, c->S, c->partial);
  int ysplit = (c->dim + 255) / 256;
  if (ysplit > 16) ysplit = 16;
  const int cthreads = c->dim >= 256 ? 256 : (c->dim + 63) / 64 * 64;
  if (max_chunks > kCombineGroup)
    hipLaunchKernelGGL(k_combine_groups, dim3((unsigned)max_chunks, ysplit), dim3(cthreads), 0, c->stream, c->chunk_off,
                       c->chunk_node, c->k, c->dim, c->partial);
  hipLaunchKernelGGL(k_combine_chunks, dim3(c->k, ysplit), dim3(256), 0, c->stream, c->chunk_off, c->dim, c->partial,
                     c->S);
  return hipGetLastError();
}

hipError_t launch_accumulate_csr(som_ctx *c, const int64_t *indptr, const int32_t *indices,
                                 const float *values, int64_t n, int64_t nnz, const int32_t *bmus) {
  int ysplit = (c->dim + 4095) / 4096;
  if (ysplit > 64) ysplit = 64;
  const int64_t k = c->k, tiles = ((int64_t)c->dim + kCsrTile - 1) / kCsrTile;
  if (tiles == 1 || (tiles <= kTilesMax && n >= kTileFrom * k)) {
    const int tile = (int)((c->dim + tiles - 1) / tiles + 3) & ~3;
    const bool few = tiles == 1 && k >= c->n_cu && nnz < kCsrFewEntries * k;
    const bool twice = !few && tiles == 1 && 2 * tile <= kCsrTile && k >= c->n_cu && n >= 48 * k && n <= 100 * k;
    const int rows = twice ? 2 * kCsrChunkRows : kCsrChunkRows;
    hipError_t e = launch_group_by_bmu(c, bmus, n, rows);
    if (e != hipSuccess) return e;
    if (c->GxT) {          // matrix smoothing only reads the rows of chosen nodes
      hipLaunchKernelGGL(k_zero_rows_if, dim3(c->k, ysplit), dim3(256), 0, c->stream, c->counts, rows, c->dim, c->S);
    } else {               // the stencil smoothing reads every row: those of nodes nobody chose must be zero
      e = launch_fill_zero_u32(c->stream, c->S, k * c->dim);
      if (e != hipSuccess) return e;
    }
    const int64_t max_chunks = n / rows + (n < k ? n : k);
    int64_t ways = (kCsrFill * (int64_t)c->n_cu + max_chunks - 1) / max_chunks;
    if (ways > tiles) ways = tiles;
    const dim3 grid((unsigned)max_chunks, (unsigned)ways);
    const size_t lds = (size_t)tile * sizeof(float);
    if (few)
      hipLaunchKernelGGL((k_accumulate_csr<4, 4, 1>), grid, dim3(256), lds, c->stream, indptr, indices, values, c->dim, tile,
                         c->sort_val[0], c->seg_off, c->chunk_off, c->chunk_node, c->k, c->S);
    else if (twice)
      hipLaunchKernelGGL((k_accumulate_csr<8, 8, 2>), grid, dim3(512), 2 * lds, c->stream, indptr, indices, values, c->dim, tile,
                         c->sort_val[0], c->seg_off, c->chunk_off, c->chunk_node, c->k, c->S);
    else
      hipLaunchKernelGGL((k_accumulate_csr<8, 8, 1>), grid, dim3(512), lds, c->stream, indptr, indices, values, c->dim, tile,
                         c->sort_val[0], c->seg_off, c->chunk_off, c->chunk_node, c->k, c->S);
    return hipGetLastError();
  }
  hipError_t e = launch_fill_zero_u32(c->stream, c->counts, c->k);
  if (e != hipSuccess) return e;
  int64_t cb = (n + 255) / 256;
  if (cb > (int64_t)c->n_cu * 16) cb = (int64_t)c->n_cu * 16;
  hipLaunchKernelGGL(k_count_bmus, dim3((unsigned)cb), dim3(256), 0, c->stream, bmus, n, c->k, c->counts);
  if (c->GxT) {
    hipLaunchKernelGGL(k_zero_rows_if, dim3(c->k, ysplit), dim3(256), 0, c->stream, c->counts, 0, c->dim, c->S);
  } else {
    e = launch_fill_zero_u32(c->stream, c->S, (int64_t)c->k * c->dim);
    if (e != hipSuccess) return e;
  }
  int64_t sb = (n + 3) / 4;
  if (sb > (int64_t)c->n_cu * 32) sb = (int64_t)c->n_cu * 32;
  hipLaunchKernelGGL(k_scatter_csr, dim3((unsigned)sb), dim3(256), 0, c->stream, indptr, indices, values, n,
                     c->dim, c->k, bmus, c->S);
  return hipGetLastError();
}

}  // namespace som
