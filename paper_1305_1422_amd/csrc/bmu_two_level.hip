// Dense best-matching-unit search in two levels (paper: BMU equation; "Parallelism": distances
// through linear algebra).
//
// The split-fp16 filter (bmu_dense_h.hip) spends three matrix products per feature on EVERY
// (instance, node) pair to get fp32-grade scores, although all it needs of most pairs is the
// knowledge that the node is not the best one.  One product on the hi halves alone gives scores with
// 11-bit operands at a third of the work, and a proven bound e_j on their error (margin.hpp).  So:
//   1. coarse pass (k_bmu_dense_h, block-minimum mode): m[b][j] = the smallest coarse score of instance
//      j among the 128 nodes of block b;
//   2. k_select_blocks: with m_j = min_b m[b][j], the BMU of j lies in a block with
//      m[b][j] <= m_j + 2 e_j - a node of any other block has an exact score above that of the node
//      that gave m_j, strictly, so it is not the BMU and does not tie with it.  The kernel writes that
//      block set as a bit mask, and a sort key made of the size class of the set (1, 2, 3-4, 5-8, ...
//      blocks; the widest class first), its lowest block and the distance from there to its highest;
//   3. the instances are put in the order of their keys (segsum.hip's grouping).  A fine-pass tile
//      works on the union of its 128 instances' sets, so one instance with a wide set (one that lies
//      between clusters, say) makes its whole tile expensive: the size class keeps such instances among
//      themselves, and within a class the lowest and the highest block put instances with the same sets
//      side by side (listed blocks per tile, lowest alone / both: sparse uniform rows on 50 x 50 nodes
//      3.0 / 1.7, uniform noise on 74 x 95 7.3 / 6.0, a mixture on 100 x 100 2.1 / 1.9);
//   4. k_tile_lists: the union of the masks over every 128 consecutive instances of that order, as an
//      ascending list of blocks;
//   5. fine pass (k_bmu_dense_h, fine mode): the split-fp16 filter over those (tile, block) pairs only.
// Its candidates go through the exact stage like those of the one-level filter: the nodes it never saw
// are out by the argument of step 2, whatever the exact stage decides about the others.
// A block is a patch of the map, not 128 nodes of consecutive index: the planes hold the nodes in bands of about
// kPatchRows rows, column by column within a band, so that a block is about 12 rows of 10 or 11 columns.  The
// candidates of an instance lie in a neighbourhood of its BMU, which such patches cover with far fewer blocks than
// strips of one or two map rows do (listed blocks per tile, strips / patches, both with the bound on e_j that the
// residuals give: 1,000,000 x 128 on 100 x 100 nodes 5.3 / 2.1, 50,000 x 256 on 200 x 200 12.1 / 4.4; fine pass
// there 950 -> 300 and 250 -> 90 us).
// The price is steps 2-4 and the table m (4 bytes per instance and node block, written once and read
// twice); when every block of every tile is listed (a code book of equal rows) the fine pass is the
// whole one-level filter and the coarse pass is lost: a third more work in that worst case.
#include "margin.hpp"

namespace som {

// kParts threads per instance (one per wavefront of the workgroup, so that a wavefront reads 64 consecutive
// instances of a table row); thread p of an instance takes the blocks p, p + kParts, ... and keeps the first
// 32 of them in registers, so that the table is read once for maps of up to 32 kParts blocks (beyond that the
// rest is read again for the comparison); minima, mask words and the key are combined through LDS.
// Bound by the read of the table, provided that the vector units keep out of its way: the block number is a scalar, so that rows are
// addressed and left out without vector instructions, and one wavefront takes the fp64 margins for all (another one in every
// workgroup, as wavefronts of a number share a SIMD).  1,000,000 instances x 79 blocks 132 -> 74 us (4.3 TB/s; 168 -> 60 registers), 50,000 x 313
// 28.9 -> 23.0, 100,000 x 20 16 -> 5.9.
template <int kParts>
__global__ __launch_bounds__(64 * kParts) void k_select_blocks(const float *__restrict__ m, int64_t n, int blocks,
                                                              const float *__restrict__ xn32,
                                                              const unsigned *__restrict__ wmax_bits,
                                                              const float *__restrict__ mu_norm2, MarginModel mm,
                                                              int classes, int spans, int only, int32_t *__restrict__ key,
                                                              uint32_t *__restrict__ mask) {
  constexpr int kHold = 32;
  constexpr int kWordsAtOnce = kHold * kParts / 32;      // mask words combined per round: the first are those held
  constexpr int kRun = 4;                       // loads between two looks at the number of blocks
  __shared__ float s_best[kParts][64];
  __shared__ double s_margin[64];
  __shared__ uint32_t s_bits[kParts][kWordsAtOnce][64];
  const int lane = threadIdx.x & 63;
  const int part = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + (int)blockIdx.x) & (kParts - 1);
  const int64_t j0 = (int64_t)blockIdx.x * 64, j = j0 + lane;
  const bool live = j < n;
  const unsigned at = (unsigned)(live ? lane : (int)(n - 1 - j0));      // lanes past the end repeat the last instance
  if (only && !mm.sub->use) {                   // no scores: no blocks (the passes behind this one find nothing to do)
    if (part == 0 && live) {
      for (int w = 0; 32 * w < blocks; ++w) mask[(int64_t)w * n + j] = 0;
      key[j] = 0;
    }
    return;
  }
  float held[kHold];
  float best = INFINITY;
#pragma unroll
  for (int i = 0; i < kHold; ++i) {
    held[i] = INFINITY;
  }
#pragma unroll
  for (int i0 = 0; i0 < kHold; i0 += kRun)
    if (part + i0 * kParts < blocks) {          // (blocks past the last repeat it)
#pragma unroll
      for (int i = i0; i < i0 + kRun; ++i) held[i] = (m + (int64_t)min(part + i * kParts, blocks - 1) * n + j0)[at];
    }
  // score_margin is the bound for a PAIR of scores (2 e_j and slack): exactly the window of step 2
  if (part == 0)
    s_margin[lane] = score_margin(mm, j0 + at, (double)xn32[j0 + at], (double)__uint_as_float(*wmax_bits), (double)*mu_norm2);
#pragma unroll
  for (int i = 0; i < kHold; ++i) best = fminf(best, held[i]);
  for (int b = part + kHold * kParts; b < blocks; b += kParts) best = fminf(best, (m + (int64_t)b * n + j0)[at]);
  s_best[part][lane] = best;
  __syncthreads();
  best = s_best[0][lane];
#pragma unroll
  for (int p = 1; p < kParts; ++p) best = fminf(best, s_best[p][lane]);
  float t32 = INFINITY;                         // no finite score at all: every block stays in
  if (best < INFINITY) {
    const double thr = (double)best + s_margin[lane];
    t32 = (float)thr;                           // rounded up: no block inside the window is lost
    if ((double)t32 < thr) t32 = nextafterf(t32, INFINITY);
  }
  int listed = 0, lowest = 0x7fffffff, highest = 0;          // kept by part 0
  for (int w0 = 0; w0 < blocks; w0 += 32 * kWordsAtOnce) {
    uint32_t bits[kWordsAtOnce];
#pragma unroll
    for (int w = 0; w < kWordsAtOnce; ++w) bits[w] = 0;
    if (w0 == 0) {                              // the blocks held in registers: 32 kParts <= 256 of them
#pragma unroll
      for (int i = 0; i < kHold; ++i) {
        // compile-time word and bit position up to `part`; a NaN keeps its block in, blocks past the last go below
        bits[(i * kParts) >> 5] |= held[i] > t32 ? 0u : 1u << ((i * kParts) & 31);
      }
    }
    if (kParts > 4 && w0 > 0) {                 // (the launcher gives four parts to maps that fit the registers)
#pragma unroll
      for (int w = 0; w < kWordsAtOnce; ++w)
        if (w0 + 32 * w < blocks) {
          float v[32 / kParts];
#pragma unroll
          for (int t = 0; t < 32 / kParts; ++t) v[t] = (m + (int64_t)min(w0 + 32 * w + part + kParts * t, blocks - 1) * n + j0)[at];
#pragma unroll
          for (int t = 0; t < 32 / kParts; ++t) bits[w] |= v[t] > t32 ? 0u : 1u << (kParts * t);
        }
    }
#pragma unroll
    for (int w = 0; w < kWordsAtOnce; ++w) bits[w] <<= part;
#pragma unroll
    for (int w = 0; w < kWordsAtOnce; ++w) s_bits[part][w][lane] = bits[w];
    __syncthreads();
    if (part == 0 && live) {
#pragma unroll
      for (int w = 0; w < kWordsAtOnce; ++w) {
        if (w0 + 32 * w >= blocks) break;
        uint32_t all = 0;
#pragma unroll
        for (int p = 0; p < kParts; ++p) all |= s_bits[p][w][lane];
        if (blocks - w0 - 32 * w < 32) all &= (1u << (blocks - w0 - 32 * w)) - 1;
        mask[(int64_t)((w0 >> 5) + w) * n + j] = all;
        if (all && lowest == 0x7fffffff) lowest = w0 + 32 * w + __ffs((int)all) - 1;
        if (all) highest = w0 + 32 * w + 31 - __clz((int)all);
        listed += __popc(all);
      }
    }
    __syncthreads();
  }
  if (part == 0 && live) {
    const int size_class = listed <= 1 ? 0 : 32 - __clz(listed - 1);      // ceil(log2(listed))
    // widest sets first: their tiles are the longest workgroups of the fine pass and should not start last
    const int first = lowest == 0x7fffffff ? 0 : lowest;
    key[j] = ((classes - 1 - size_class) * blocks + first) * spans + min(max(highest - first, 0), spans - 1);
  }
}

// Size classes 0 .. ceil(log2(blocks)) of a block set.
static int size_classes(int blocks) {
  int classes = 1;
  while ((1 << (classes - 1)) < blocks) ++classes;
  return classes;
}

// The order of the nodes in the planes (see the head of this file): bands of rows, each column by column.
__global__ __launch_bounds__(256) void k_patch_order(int rows, int cols, int bands, int32_t *__restrict__ node_of,
                                                     int32_t *__restrict__ pos_of) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= rows * cols) return;
  const int band = (int)((((int64_t)p / cols + 1) * bands - 1) / rows);      // the last one that starts at or before that row
  const int r0 = (int)((int64_t)band * rows / bands), r1 = (int)((int64_t)(band + 1) * rows / bands);
  const int in = p - r0 * cols, col = in / (r1 - r0), row = r0 + in % (r1 - r0);
  const int node = row * cols + col;
  node_of[p] = node;
  pos_of[node] = p;
}

hipError_t launch_patch_order(som_ctx *c) {
  int bands = (c->rows + kPatchRows / 2) / kPatchRows;
  if (bands < 1) bands = 1;
  hipLaunchKernelGGL(k_patch_order, dim3((c->k + 255) / 256), dim3(256), 0, c->stream, c->rows, c->cols, bands, c->node_of,
                     c->pos_of);
  return hipGetLastError();
}

// One wavefront per tile of 128 consecutive entries of `rows`: OR of their masks, expanded to a list.
// The masks are stored with stride n; `rows` has n entries, or *n_rows of them if n_rows is given.
__global__ __launch_bounds__(256) void k_tile_lists(const uint32_t *__restrict__ mask, const int32_t *__restrict__ rows,
                                                    int64_t n, const int32_t *__restrict__ n_rows, int blocks,
                                                    int32_t *__restrict__ tile_cnt, int32_t *__restrict__ tile_list) {
  const int lane = threadIdx.x & 63;
  const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t entries = n_rows ? (int64_t)*n_rows : n;
  if (tile * 128 >= entries) return;            // uniform over the wavefront
  const int64_t p0 = tile * 128 + lane, p1 = p0 + 64;
  const int64_t r0 = p0 < entries ? rows[p0] : -1, r1 = p1 < entries ? rows[p1] : -1;
  int32_t *out = tile_list + tile * blocks;
  int count = 0;
  for (int w0 = 0; w0 < blocks; w0 += 32) {
    uint32_t bits = 0;
    if (r0 >= 0) bits |= mask[(int64_t)(w0 >> 5) * n + r0];
    if (r1 >= 0) bits |= mask[(int64_t)(w0 >> 5) * n + r1];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) bits |= __shfl_xor(bits, o, 64);
    const bool set = lane < 32 && w0 + lane < blocks && ((bits >> lane) & 1u);
    const unsigned long long bal = __ballot(set);
    if (set) out[count + __popcll(bal & ((1ull << lane) - 1ull))] = w0 + lane;
    count += __popcll(bal);
  }
  if (lane == 0) tile_cnt[tile] = count;
}

hipError_t launch_select_blocks(som_ctx *c, int64_t n, SubspaceUse sub) {
  const int blocks = (c->k + 127) / 128, classes = size_classes(blocks);
  const int mode = sub == kSubOnly ? kCertifySubspaceCsrSelect : sub == kSubMay ? kCertifySubspace : kCertifySelect;
  // as many steps of the span as keep the keys below k: the grouping by key has room for that many
  const int spans = c->k / (classes * blocks) > blocks ? blocks : c->k / (classes * blocks) > 1 ? c->k / (classes * blocks) : 1;
  if (blocks <= 128)      // 32 blocks held per thread: all of them
    hipLaunchKernelGGL(k_select_blocks<4>, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, c->stream, c->coarse_min, n,
                       blocks, c->xn32, c->wmax_bits, c->mu_norm2, margin_model(c, mode, nullptr),
                       classes, spans, sub == kSubOnly, c->coarse_key, c->coarse_mask);
  else
    hipLaunchKernelGGL(k_select_blocks<8>, dim3((unsigned)((n + 63) / 64)), dim3(512), 0, c->stream, c->coarse_min, n,
                       blocks, c->xn32, c->wmax_bits, c->mu_norm2, margin_model(c, mode, nullptr),
                       classes, spans, sub == kSubOnly, c->coarse_key, c->coarse_mask);
  return hipGetLastError();
}

hipError_t launch_tile_lists(som_ctx *c, int64_t n) {
  const int blocks = (c->k + 127) / 128;
  const int64_t tiles = (n + 127) / 128;
  hipLaunchKernelGGL(k_tile_lists, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, c->stream, c->coarse_mask,
                     c->sort_val[0], n, nullptr, blocks, c->tile_cnt, c->tile_list);
  return hipGetLastError();
}

// The same for the instances the exact stage sweeps again (c->collect_rows, their number on the device).
hipError_t launch_collect_tile_lists(som_ctx *c, int64_t n) {
  const int blocks = (c->k + 127) / 128;
  const int64_t tiles = (n + 127) / 128;
  hipLaunchKernelGGL(k_tile_lists, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, c->stream, c->coarse_mask,
                     c->collect_rows, n, c->list_counts + 1, blocks, c->ctile_cnt, c->ctile_list);
  return hipGetLastError();
}

}  // namespace som
