// Dense best-matching-unit search, coarse pass of the two-level search (paper: BMU equation;
// "Parallelism": distances through linear algebra).  See bmu_two_level.hip for what the pass is for.
//
// Scores s = |w'_i|^2 - 2 x'.w'_i from ONE fp16 product per feature, on the hi halves of the split
// planes alone (split_f16.hip: rows of 64-feature chunks, 128 bytes each), accumulated in fp32 by
// v_mfma_f32_32x32x16_f16 without intermediate flushes; kept is only the smallest score per instance and
// block of 128 nodes.
//
// With one product per operand pair the pass is bound by LDS traffic, not by the matrix pipes: a
// wavefront tile of 64 x 64 outputs (the shape of the three-product pass, bmu_dense_h.hip) reads 1 KB of
// operands per MFMA.  So a wavefront owns 128 nodes x 64 instances here (4 x 2 MFMA blocks, 128
// accumulator registers, 0.75 KB per MFMA), a workgroup has 8 wavefronts on 256 nodes x 256 instances,
// two LDS stages of (256 + 256) rows x 128 bytes (128 KB), one workgroup per CU: measured 1.4 times the
// rate of the 64 x 64 shape at 1,000 features.  The 128 nodes of a wavefront are one block of the table,
// so the minima need no exchange between wavefronts.  Tile loads, swizzle and grid decoding are those of
// bmu_dense_h.hip.
#include "bmu_dense_common.hpp"

namespace som {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void *lptr_c_t;

constexpr int kCRow = 32;                  // floats per tile row (= 64 halves = one chunk of 64 features)
constexpr int kCTN = 256, kCTI = 256;      // nodes / instances per workgroup tile
constexpr int kCThreads = 512;

__device__ __forceinline__ unsigned lds_address_c(const float *p) { return (unsigned)(size_t)(lptr_c_t)p; }

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// Direct-to-LDS load of 16 bytes per lane, "wavefront-uniform base + 32-bit byte offset per lane" form
// (see bmu_dense_dl.hip for why this is inline assembly).
__device__ __forceinline__ void load16_to_lds_c(const void *base, unsigned lane_offset, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(lane_offset), "s"(base), "s"(lds_base)
               : "memory", "m0");
}
// The same for 4 bytes per lane: lane l's word goes to LDS byte address lds_base + 4 l.
__device__ __forceinline__ void load4_to_lds_c(const void *base, unsigned lane_offset, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(lane_offset), "s"(base), "s"(lds_base)
               : "memory", "m0");
}

#pragma clang diagnostic pop

__device__ __forceinline__ f16x8 as_halves_c(f32x4 v) { return __builtin_bit_cast(f16x8, v); }

// kDump = false: block_min[node block of 128][instance] = smallest score of the pair.
// kDump = true (test hook): every score to dump[instance * k + node]; the rows of Wh are nodes node_of[0], node_of[1], ...
// wc: node constants c_i, readable for i < k_const (a multiple of 128 >= k, +inf past k).
struct CoarseOperands {
  const float *Xh, *Wh, *xscale, *wscale;
  int nK;                            // chunks of 64 features
};
// Coordinates in the code book's subspace, and the device's decision to run on them.
struct CoarseSubspace {
  const SubspaceState *state;
  const _Float16 *Y1, *U1;
  const float *yscale;
};
constexpr int kSubRing = 64 << 10;   // bytes

// The pass on the subspace's coordinates (bmu_subspace.hip), 16 kKS of them: the instances' operands stay in registers, the
// nodes' rows go through a ring of LDS stages of 256 rows (32 coordinates: four of 16 KB, loaded three tiles ahead; 64: two of 32 KB).  The
// node constants are among the coordinates (three halves per node), so an accumulator holds the score divided by a negative factor of
// the instance, and the epilogue is a running three-way maximum.  A kernel of its own, because it needs half the registers and LDS of the general
// one: two workgroups per CU, four wavefronts per SIMD, fill each other's barriers.  Bound by the matrix pipes and the maxima beside
// them: 1,000,000 instances x 10,000 nodes 1,754 us (64 coordinates as one chunk of the general loop below) -> 708 (the first 32 in
// a loop like this one inside that kernel) -> 633.
template <int kKS>
__device__ __forceinline__ void coarse_in_subspace(const CoarseSubspace &sub, float *__restrict__ lds, int64_t n, int k,
                                                   int64_t inst0, int nb_first, int nNB, float *__restrict__ out) {
  constexpr int kStages = kKS == 2 ? 4 : 2;
  constexpr int kRowBytes = 32 * kKS, kSlots = 2 * kKS, kTileBytes = kCTN * kRowBytes;
  static_assert(kStages * kTileBytes == kSubRing, "the ring");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wi = wave & 3, l32 = lane & 31, lhi = lane >> 5;
  // 16-byte slot of a row that slot `s` is kept in: any eight consecutive rows read one slot from eight different bank groups
  auto swizzle = [](int row) { return kKS == 4 ? (row & 7) ^ ((row >> 3) & 1) : (row >> 1) & 3; };

  int row[kKS];
  unsigned slot[kKS];
#pragma unroll
  for (int i = 0; i < kKS; ++i) {
    row[i] = (wave * kKS + i) * (64 / kSlots) + lane / kSlots;
    slot[i] = 16u * ((lane % kSlots) ^ swizzle(row[i]));
  }
  const unsigned lds_at = lds_address_c(lds) + wave * kKS * 1024;
  auto issue = [&](int t) {                       // rows past the last node repeat it: they change no maximum
    const char *base = reinterpret_cast<const char *>(sub.U1) + (int64_t)(nb_first + t) * kCTN * (kSub * 2);
    const int last = k - 1 - (nb_first + t) * kCTN;
#pragma unroll
    for (int i = 0; i < kKS; ++i)
      load16_to_lds_c(base, (unsigned)min(row[i], last) * (kSub * 2) + slot[i], lds_at + (t % kStages) * kTileBytes + i * 1024);
  };
  f16x8 h[2][kKS];
  float factor[2];
  int64_t inst[2];
#pragma unroll
  for (int ni = 0; ni < 2; ++ni) {
    inst[ni] = inst0 + wi * 64 + ni * 32 + l32;
    const int64_t j = inst[ni] < n ? inst[ni] : n - 1;
    factor[ni] = -2.f * sub.yscale[j] * sub.state->uscale;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) h[ni][ks] = *reinterpret_cast<const f16x8 *>(sub.Y1 + j * (16 * kKS) + 16 * ks + 8 * lhi);
  }
  for (int t = 0; t < kStages - 1 && t < nNB; ++t) issue(t);
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float best[2] = {INFINITY, INFINITY};
  int best_block = -1;
  auto store = [&]() {                            // of the previous tile: its latency then passes beside a tile's products
    if (best_block < 0 || best_block * 128 >= k || lhi != 0) return;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
      if (inst[ni] < n) out[(int64_t)best_block * n + inst[ni]] = best[ni];
  };
  for (int t = 0; t < nNB; ++t) {
    // the loads of tile t have landed when at most those of the tiles behind it are in flight (loads return in order)
    if (kStages == 4 && t + 2 < nNB) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * kKS));
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    store();
    if (t + kStages - 1 < nNB) issue(t + kStages - 1);      // into the stage that every wavefront has left
    const char *at = reinterpret_cast<const char *>(lds) + (t % kStages) * kTileBytes + (wm * 128 + l32) * kRowBytes;
    float m[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
      f16x8 g[kKS];
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
        g[ks] = *reinterpret_cast<const f16x8 *>(at + mi * 32 * kRowBytes + 16 * ((2 * ks + lhi) ^ swizzle(l32)));
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) {
        f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(g[0], h[ni][0], zero, 0, 0, 0);
#pragma unroll
        for (int ks = 1; ks < kKS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(g[ks], h[ni][ks], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; v += 2) m[ni] = fmaxf(fmaxf(m[ni], acc[v]), acc[v + 1]);
      }
    }
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) best[ni] = factor[ni] * fmaxf(m[ni], __shfl_xor(m[ni], 32, 64));
    best_block = (nb_first + t) * 2 + wm;
  }
  store();
}

__global__ __launch_bounds__(kCThreads, 4) void k_bmu_coarse_subspace(CoarseSubspace sub, int64_t n, int k, int groups,
                                                                      float *__restrict__ out) {
  __shared__ __attribute__((aligned(16))) float s_ring[kSubRing / 4];
  const int use = sub.state->use;
  if (!use) return;                  // the same for every workgroup
  const int64_t slot_id = blockIdx.x >> 3, tile = (slot_id / groups) * 8 + (blockIdx.x & 7);      // as in k_bmu_coarse
  const int group = (int)(slot_id % groups), nNB_all = (k + kCTN - 1) / kCTN, nb_per = (nNB_all + groups - 1) / groups;
  const int nb_first = group * nb_per, nNB = min(nb_per, nNB_all - nb_first);
  if (tile * kCTI >= n || nNB <= 0) return;
  if (use == 1) coarse_in_subspace<2>(sub, s_ring, n, k, tile * kCTI, nb_first, nNB, out);
  else coarse_in_subspace<4>(sub, s_ring, n, k, tile * kCTI, nb_first, nNB, out);
}

template <bool kDump>
__global__ __launch_bounds__(kCThreads, 1) void k_bmu_coarse(CoarseOperands op, const SubspaceState *__restrict__ off,
                                                             const float *__restrict__ wc, int k_const, int64_t n, int k,
                                                             int groups, float *__restrict__ out,
                                                             const int32_t *__restrict__ node_of) {
  if (off && off->use) return;
  const float *__restrict__ Xh = op.Xh, *__restrict__ Wh = op.Wh, *__restrict__ xscale = op.xscale, *__restrict__ wscale = op.wscale;
  const int nK = op.nK;
  __shared__ __attribute__((aligned(16))) float s_stage[2 * (kCTN + kCTI) * kCRow];
  float (*sW)[kCTN * kCRow] = reinterpret_cast<float (*)[kCTN * kCRow]>(s_stage);
  float (*sX)[kCTI * kCRow] = reinterpret_cast<float (*)[kCTI * kCRow]>(s_stage + 2 * kCTN * kCRow);
  __shared__ float sWn[2][kCTN];     // node constants of the node tiles in flight, by parity of the tile's ordinal

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2;          // which 128-node half of the tile
  const int wi = wave & 3;           // which 64-instance quarter of the tile
  const int l32 = lane & 31;
  const int lhi = lane >> 5;

  // workgroup -> (instance tile, node group): the groups of one instance tile are workgroups 8 apart
  const int64_t ntiles = (n + kCTI - 1) / kCTI;
  const int xcd = (int)(blockIdx.x & 7);
  const int64_t slot_id = blockIdx.x >> 3;
  const int group = (int)(slot_id % groups);
  const int64_t tile = (slot_id / groups) * 8 + xcd;
  if (tile >= ntiles) return;        // uniform over the workgroup
  const int64_t inst0 = tile * kCTI;
  const int nNB_all = (k + kCTN - 1) / kCTN;
  const int nb_per = (nNB_all + groups - 1) / groups;
  const int nb_first = group * nb_per;
  const int nNB = min(nb_per, nNB_all - nb_first);
  if (nNB <= 0) return;              // uniform over the workgroup
  const int total = nK * nNB;

  // ---- loader: one instruction fills 8 tile rows; wavefront w issues W slots 4 w .. 4 w + 3 and X slots
  // 4 w .. 4 w + 3.  Rows past the end of an operand are redirected to its last row (their outputs are
  // never used: such nodes get the constant +inf, such instances are not stored).
  const int ld_rloc = lane >> 3;
  const int ld_pos = lane & 7;
  const unsigned row_bytes = (unsigned)nK * (kCRow * 4);
  const char *xbase = reinterpret_cast<const char *>(Xh) + inst0 * (int64_t)row_bytes;
  const int64_t last_inst = n - 1 - inst0;       // >= 0
  unsigned xoff[4], woff[4], wq[4];
  int wrow[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 8 * (4 * wave + i) + ld_rloc;
    const int q = ld_pos ^ ((row & 7) ^ ((row >> 3) & 1));
    const int rclamped = row < last_inst ? row : (int)last_inst;
    xoff[i] = (unsigned)rclamped * row_bytes + 16u * q;
    wrow[i] = row;
    wq[i] = 16u * q;
    woff[i] = 0;
  }
  const unsigned lds_w = lds_address_c(&sW[0][1024 * wave]);     // 4 slots of 256 floats
  const unsigned lds_x = lds_address_c(&sX[0][1024 * wave]);
  const unsigned lds_wn = lds_address_c(&sWn[0][0]);
  // Up to 128 features the whole instance tile fits the two X stages: it is loaded once, with the first node tile,
  // and only the node tiles stream (half the traffic from L2 into LDS, which is what bounds the pass at so few
  // features per tile).
  const bool x_stays = nK <= 2;
  int ld_nb = nb_first, ld_kc = 0;
  auto issue_loads = [&](int buf) {
    const char *wbase = reinterpret_cast<const char *>(Wh) + (int64_t)ld_nb * kCTN * row_bytes;
    if (ld_kc == 0) {                                             // entering a node tile
      const int last_node = k - 1 - ld_nb * kCTN;                 // >= 0
#pragma unroll
      for (int i = 0; i < 4; ++i) woff[i] = (unsigned)(wrow[i] < last_node ? wrow[i] : last_node) * row_bytes + wq[i];
      // node constants of the tile, as the oldest operation of the batch.  Past the padded constants the
      // last one is read again: either +inf, or a block of the table that is not written at all
      if (wave < 4) {
        const int node = min(ld_nb * kCTN + wave * 64 + lane, k_const - 1);
        load4_to_lds_c(wc, (unsigned)node * 4u, lds_wn + ((ld_nb - nb_first) & 1) * (kCTN * 4) + wave * 256);
      }
    }
    const unsigned off = (unsigned)ld_kc * (kCRow * 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) load16_to_lds_c(wbase + off, woff[i], lds_w + buf * (kCTN * kCRow * 4) + i * 1024);
    if (!x_stays) {
#pragma unroll
      for (int i = 0; i < 4; ++i) load16_to_lds_c(xbase + off, xoff[i], lds_x + buf * (kCTI * kCRow * 4) + i * 1024);
    } else if (ld_nb == nb_first) {                               // chunk kc of the instance tile lives in sX[kc]
#pragma unroll
      for (int i = 0; i < 4; ++i) load16_to_lds_c(xbase + off, xoff[i], lds_x + ld_kc * (kCTI * kCRow * 4) + i * 1024);
    }
    if (++ld_kc == nK) { ld_kc = 0; ++ld_nb; }
  };

  // ---- reader: 16-byte slot 2 t + (lane >> 5) of a row holds this lane's 8 features of k-step t
  const int rd_swz = (l32 & 7) ^ ((l32 >> 3) & 1);
  int rd_off[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) rd_off[g] = 4 * ((2 * g + lhi) ^ rd_swz);
  const int a_base = (wm * 128 + l32) * kCRow;
  const int b_base = (wi * 64 + l32) * kCRow;

  const float sw = *wscale;
  float factor[2];
#pragma unroll
  for (int ni = 0; ni < 2; ++ni) {
    const int64_t inst = inst0 + wi * 64 + ni * 32 + l32;
    factor[ni] = inst < n ? -2.f * xscale[inst] * sw : 0.f;
  }

  f32x16 acc[4][2];
  // Operands of two k-steps (ks and ks + 2 of the chunk's four): 12 LDS reads of 16 bytes for 16 MFMAs.
  struct Operands { f16x8 g1[4], g2[4], h1[2], h2[2]; };
  auto read_operands = [&](Operands &o, int st, int xst, int ks) {
    const float *pw = &sW[st][a_base];
    const float *px = &sX[xst][b_base];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      o.g1[b] = as_halves_c(*reinterpret_cast<const f32x4 *>(pw + b * 32 * kCRow + rd_off[ks]));
      o.g2[b] = as_halves_c(*reinterpret_cast<const f32x4 *>(pw + b * 32 * kCRow + rd_off[2 + ks]));
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      o.h1[b] = as_halves_c(*reinterpret_cast<const f32x4 *>(px + b * 32 * kCRow + rd_off[ks]));
      o.h2[b] = as_halves_c(*reinterpret_cast<const f32x4 *>(px + b * 32 * kCRow + rd_off[2 + ks]));
    }
  };
  // `fresh`: the accumulators start from C = 0 as an operand of the instruction itself.
  auto multiply = [&](const Operands &o, bool fresh) {
    __builtin_amdgcn_s_setprio(1);
    if (fresh) {
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.g2[mi], o.h2[ni], zero, 0, 0, 0);
    } else {
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.g2[mi], o.h2[ni], acc[mi][ni], 0, 0, 0);
    }
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.g1[mi], o.h1[ni], acc[mi][ni], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };

  // Two stages: chunk t + 1 is loaded during iteration t, every wavefront waits for its own loads before
  // the barrier that ends the iteration, and every operand is read after that barrier.
  issue_loads(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wavefront's direct-to-LDS loads have landed
  __syncthreads();

  bool fresh = true;
  Operands op0, op1;
  int stage = 0;
  for (int t = 0; t < total; ++t) {
    const int ord = t / nK, kc = t % nK;         // ordinal of the node tile in this workgroup's run
    if (t + 1 < total) issue_loads(stage ^ 1);   // that stage held chunk t - 1, which every wavefront has left
    const int xstage = x_stays ? kc : stage;
    read_operands(op0, stage, xstage, 0);
    read_operands(op1, stage, xstage, 1);
    multiply(op0, fresh);
    multiply(op1, false);
    fresh = (kc == nK - 1);
    if (fresh) {
      const int nb = nb_first + ord;
      const float *swn = &sWn[ord & 1][wm * 128];
      if (kDump) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int nl = mi * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3);
            const int node = nb * kCTN + wm * 128 + nl;
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) {
              const int64_t inst = inst0 + wi * 64 + ni * 32 + l32;
              if (node < k && inst < n) out[inst * k + node_of[node]] = fmaf(factor[ni], acc[mi][ni][v], swn[nl]);
            }
          }
      } else {
        // smallest score per instance over this wavefront's 128 nodes = one block of the table: over the
        // lane's 64 nodes (pairs: one three-way minimum per two scores), then the other lane half
        const int block = nb * 2 + wm;
        if (block * 128 < k) {                   // uniform over the wavefront
#pragma unroll
          for (int ni = 0; ni < 2; ++ni) {
            float m = INFINITY;
#pragma unroll
            for (int mi = 0; mi < 4; ++mi)
#pragma unroll
              for (int v = 0; v < 16; v += 2) {
                const int nl = mi * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3);
                const float s0 = fmaf(factor[ni], acc[mi][ni][v], swn[nl]);
                const float s1 = fmaf(factor[ni], acc[mi][ni][v + 1], swn[nl + 1]);
                m = fminf(fminf(m, s0), s1);
              }
            m = fminf(m, __shfl_xor(m, 32, 64));
            const int64_t inst = inst0 + wi * 64 + ni * 32 + l32;
            if (lhi == 0 && inst < n) out[(int64_t)block * n + inst] = m;
          }
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
    __syncthreads();
    stage ^= 1;
  }
}

// Node groups per instance tile: enough workgroups for several rounds over the CUs (one workgroup each).
static int bmu_coarse_groups(const som_ctx *c, int64_t n) {
  const int64_t tiles = (n + kCTI - 1) / kCTI;
  const int nNB = (c->k + kCTN - 1) / kCTN;
  int64_t want = (8 * (int64_t)c->n_cu + tiles - 1) / tiles;
  if (want > nNB) want = nNB;
  if (want > 64) want = 64;
  if (want < 1) want = 1;
  const int nb_per = (int)((nNB + want - 1) / want);
  return (nNB + nb_per - 1) / nb_per;
}

// c->Xh1, c->Wh1 -> c->coarse_min [ceil(k/128)][n], or with `dump` every score [n][k] (test hook).
hipError_t launch_bmu_coarse(som_ctx *c, int64_t n, float *dump, SubspaceUse sub) {
  const int groups = bmu_coarse_groups(c, n);
  const int64_t tiles = (n + kCTI - 1) / kCTI;
  const int64_t blocks = (tiles + 7) / 8 * 8 * groups;
  const int k_const = (c->k + kTN - 1) / kTN * kTN;      // the node constants are padded to whole blocks of 128
  const CoarseOperands op{reinterpret_cast<const float *>(c->Xh1), reinterpret_cast<const float *>(c->Wh1), c->xscale, c->wscale,
                          (c->dim + 63) / 64};
  if (sub) {
    const CoarseSubspace cs{c->sub_state, c->sub_Y1, c->sub_U1, c->sub_yscale};
    hipLaunchKernelGGL(k_bmu_coarse_subspace, dim3((unsigned)blocks), dim3(kCThreads), 0, c->stream, cs, n, c->k, groups, c->coarse_min);
    if (sub == kSubOnly) return hipGetLastError();
  }
  if (dump)
    hipLaunchKernelGGL((k_bmu_coarse<true>), dim3((unsigned)blocks), dim3(kCThreads), 0, c->stream, op, nullptr, c->wn32,
                       k_const, n, c->k, groups, dump, c->node_of);
  else
    hipLaunchKernelGGL((k_bmu_coarse<false>), dim3((unsigned)blocks), dim3(kCThreads), 0, c->stream, op, sub ? c->sub_state : nullptr,
                       c->wn32, k_const, n, c->k, groups, c->coarse_min, c->node_of);
  return hipGetLastError();
}

}  // namespace som
