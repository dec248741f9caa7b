// Observation-window scoring for SGD-KV token selection (gfx950).
//
// Token selection keeps, inside each KV head's budget, the keys with the
// largest cumulative attention of a final observation window (SGD-KV
// Sec. 3.3, last paragraph, SnapKV-style; Sec. 5 window placements). Window
// row i of query head q sits at prompt position P0+i (P0 = C-w for the
// Query-Aware window) and attends causally to keys 0..P0+i. For each KV head
// the G*w rows of its query group are one dense block R x d, so the logits of
// a key tile are an R x 16 MFMA product.
//
//   pass 1 (lse_kernel + lse_merge_kernel, lse_pass.h): base-2 log-sum-exp of every
//     window row over its causal keys. Each workgroup covers one chunk of
//     keys (about one workgroup per CU per launch) and leaves per-row partials
//     (m, s); the merge combines the chunks in a fixed order, in fp64.
//   pass 2 (colsum_keys_kernel, colsum_kernel): for every scored key j < P0,
//     a_j = (1/G) sum_rows exp2(l_rj*log2(e) - lse2_r) (group mean; the Ipt.
//     aggregations below weight or pick rows), a fixed-order reduction with
//     no float atomics.
//
// Work split: workgroup = 8 waves; wave v holds row blocks v, v+8, v+16, ...
// (16 rows each) as MFMA A-fragments in registers, so a SIMD (waves v and
// v+4) covers a quarter of the rows. A workgroup holds at most 512 rows; a
// KV head with more window rows (G*w > 512, e.g. the 128-token window of the
// paper's main setting with GQA groups of 7 or 8) splits them over several
// workgroups per key chunk (pass 2: grid z; pass 1: grid x, with the segments). Pass 1 partials are per row
// anyway; pass 2 then leaves one column-sum partial per split, which the
// pooling pass adds (or, for Ipt. max, maximises) in split order. Each key tile (128 keys; 64 in pass 2
// for fp32 keys) is staged once in LDS and read by all eight waves as B-fragments;
// blocks past the last row are skipped. MFMA 16x16x32 bf16 (or 8 x 16x16x4
// f32 for fp32 inputs) accumulates in fp32.
// Output layout of a 16x16 MFMA: lane l holds rows 4*(l/16)+0..3 of key
// column l%16.
#include "score_common.h"
#include "segment_init.h"

namespace sgdkv {

// Pass 2: window-summed probabilities of every scored key --------------------
//
// Group aggregation. Row r of a KV head's window block belongs to query head
// g = r / w of the group. The group mean, Ipt. mean and Ipt. only sum every
// row with a weight (1, sigma_g, or 1 for the top-scored head and 0 for the
// others), folded into the exp2 argument as log2 of the weight, so they cost
// nothing extra. Ipt. max (MAXG) needs each query head's own column sum. With
// head waves (HW: a wave's row blocks are consecutive and lie in one query
// head, which needs w to be a multiple of 16*RBW) the waves sum their rows as
// for the group mean and the reduction adds the partials of each head's
// waves, weights them and takes the maximum. Otherwise the waves keep one
// partial per row block (16 rows of a single head when w is a multiple of
// 16), and the reduction adds each head's blocks the same way.
template <bool MAXG, bool HW>
constexpr bool block_partials() {
  return MAXG && !HW;
}
// Balanced head waves: the last wave keeps four lane-group partials for each of its three blocks,
// 12 rows instead of 4.
template <bool MAXG, bool HW, int RBW>
constexpr int bal_extra_rows() {
  return MAXG && HW && RBW == 4 ? 8 : 0;
}

// LDS layout of pass 2's column partials: three tiles in flight, each with RW partial rows of
// TILE columns per wave. A partial row is 16 banks further than the one before it and a wave's
// rows 16 banks further again, so that neither the four lane groups of a wave storing a subtile
// nor the four waves whose partials the reduction reads together meet in one bank.
template <typename T, int RW, int EXTRA = 0>
struct ColPartials {
  static constexpr int TILE = col_tile<T>();
  static constexpr int SL = TILE + 16;         // floats per partial row
  static constexpr int SW = RW * SL + 16;      // floats per wave
  static constexpr int ST = kScoreWaves * SW + EXTRA * SL;  // floats per tile (EXTRA more rows for the last wave)
  static constexpr int WORDS = 3 * ST;
  __device__ static constexpr int at(int t3, int wave, int r, int col) { return t3 * ST + wave * SW + r * SL + col; }
};

// MIXED: the wave's blocks belong to different heads (the last wave of the balanced head-wave
// layout): it leaves four lane-group partials per block, in rows 4j .. 4j+3 of its region.
template <typename T, int D, int NB, int RBW, bool MAXG, bool HW, bool MIXED = false>
__device__ void colsum_chunk(const CompressArgs& a, char* kbuf, float* red, float* qws, int seg, int r0, int nrows,
                             int wid, int lane,
                             const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32], const rsrc_t& kr, int64_t key0,
                             int64_t key_end, bool bal = false) {
  constexpr int NBX = NB > 0 ? NB : 1;
  constexpr int TILE = col_tile<T>();
  const int lr = lane & 15, lg = lane >> 4;
  const int h = seg % a.Hkv;
  // -lse2 (+ log2 of the row weight) of this lane's row slots; rows past R get -inf so they add 0
  const uint64_t nl = (uint64_t)a.B * a.Hkv * a.R;
  const bool natural = a.window_lse != nullptr;
  const bool weighted = !MAXG && a.agg != 0;
  const rsrc_t lr2 = make_rsrc(natural ? (const void*)a.window_lse : (const void*)a.lse2, nl * sizeof(float));
  float nlse[NBX][4];
#pragma unroll
  for (int j = 0; j < NBX; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row_block<RBW, HW>(wid, j, bal) * 16 + 4 * lg + i;  // within the split
      float l = ldf(lr2, (uint32_t)(((int64_t)seg * a.R + r0 + row) * 4));
      if (natural) l *= 1.44269504088896340736f;
      const float lw = weighted && row < nrows ? a.qweight[h * a.G + (r0 + row) / a.w] : 0.f;
      nlse[j][i] = row < nrows ? lw - l : -INFINITY;
    }
  const float c2 = a.c2;
  const int nseg = a.B * a.Hkv;
  const rsrc_t cr = make_rsrc(a.colsum + ((int64_t)blockIdx.z * nseg + seg) * a.n_scored, (uint64_t)a.n_scored * 4);
  // The chunk's tiles go last to first: pass 1 streams about the same chunks first to last, so
  // the keys it read last, the ends of the chunks, are partly still in the last-level cache.
  // Each key's sum does not depend on the order, so neither does the result.
  const int64_t ntiles = (key_end - key0 + TILE - 1) / TILE;
  // Partials of tile t sit in red[t % 3]: written during tile t, complete at the barrier of
  // tile t+1, summed right after it, rewritten only after the barrier of tile t+2. Each
  // wave sums CPW columns: the LPC lanes of a column read the partials of PPL waves each
  // (one per lane group of the wave for the group mean), shuffles add them, and the first
  // CPW lanes store. Branch-free: a store that must not happen gets an
  // offset past the buffer, which the hardware drops.
  constexpr int CPW = TILE / kScoreWaves, LPC = 64 / CPW, PPL = kScoreWaves / LPC;
  static_assert(CPW <= 16 && 64 % CPW == 0 && PPL >= 1 && PPL * LPC == kScoreWaves, "reduction layout");
  const int rcol = CPW * wid + lane % CPW, rgrp = lane / CPW;
  constexpr bool BP = block_partials<MAXG, HW>();
  using CP = ColPartials<T, BP ? RBW : 4, bal_extra_rows<MAXG, HW, RBW>()>;
  // Ipt. max: the split's head weights go to LDS once (a global load in the per-tile reduction
  // would wait behind the key tiles in flight)
  if constexpr (MAXG) {
    const int g0 = r0 / a.w, ng = nrows / a.w;  // at most kMaxSplitRows / 16 heads
    if (wid == 0 && lane < ng) qws[lane] = a.qweight[h * a.G + g0 + lane];
    __syncthreads();
  }
  auto reduce = [&](int64_t t) {  // t may be -1: nothing is stored
    const float* r = red + CP::at((int)((uint32_t)(t + 3) % 3u), 0, 0, 0);
    float v = 0.f;
    if constexpr (MAXG && HW) {
      // the LPC lanes of a column take the split's heads in turn: add the four lane-group
      // partials of each of a head's w/(16*RBW) waves in wave order, weight, keep the maximum
      // (balanced layout: heads 4-6 then add the four lane-group partials of the block they lent
      // to the last wave)
      const int wph = a.w / (16 * RBW), ng = nrows / a.w;
      for (int g = rgrp; g < ng; g += LPC) {
        float sum = 0.f;
        for (int wv = g * wph; wv < (g + 1) * wph; ++wv)
#pragma unroll
          for (int q = 0; q < 4; ++q) sum += r[wv * CP::SW + q * CP::SL + rcol];
        if (bal && g >= kBalFirstWave) {
          const float* lent = r + (kScoreWaves - 1) * CP::SW + 4 * (g - kBalFirstWave) * CP::SL + rcol;
#pragma unroll
          for (int q = 0; q < 4; ++q) sum += lent[q * CP::SL];
        }
        v = fmaxf(v, qws[g] * sum);
      }
#pragma unroll
      for (int o = CPW; o < 16; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
      v = max_lane_groups(v);
    } else if constexpr (MAXG) {
      // the LPC lanes of a column take the split's heads in turn: sum a head's w/16 blocks
      // (block b sits with wave b % 8, slot b / 8), weight it, keep the maximum
      const int bph = a.w / 16, ng = nrows / a.w;
      for (int g = rgrp; g < ng; g += LPC) {
        float sum = 0.f;
        for (int bb = g * bph; bb < (g + 1) * bph; ++bb)
          sum += r[(bb % kScoreWaves) * CP::SW + (bb / kScoreWaves) * CP::SL + rcol];
        v = fmaxf(v, qws[g] * sum);
      }
#pragma unroll
      for (int o = CPW; o < 16; o <<= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
      v = max_lane_groups(v);
    } else {
      // the partials of every wave and lane group of the column, in a fixed order
#pragma unroll
      for (int k = 0; k < PPL; ++k)
#pragma unroll
        for (int g = 0; g < 4; ++g) v += r[(rgrp + LPC * k) * CP::SW + g * CP::SL + rcol];
#pragma unroll
      for (int o = CPW; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
      v = sum_lane_groups(v);
    }
    const int64_t key = key0 + (ntiles - 1 - t) * TILE + rcol;  // step t holds tile ntiles-1-t
    const bool store = t >= 0 && lane < CPW && key < key_end;
    stf(cr, store ? (uint32_t)(key * 4) : (uint32_t)(a.n_scored * 4), v * a.out_scale);
  };
  chunk_pipeline<T, D, NB, TILE, true, false>(
      kbuf, kr, key0, a.C, ntiles, lr, lg, qa, [](const f32x4(&)[NBX]) {},
      [&](int64_t t, int sub, const f32x4(&acc)[NBX]) {
        const int t3 = (int)((uint32_t)t % 3u);  // tiles of a chunk: far fewer than 2^32
        if constexpr (BP) {
          // one column partial per row block (a single query head's rows)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const float p = (fast_exp2(fmaf(acc[j][0], c2, nlse[j][0])) + fast_exp2(fmaf(acc[j][1], c2, nlse[j][1]))) +
                            (fast_exp2(fmaf(acc[j][2], c2, nlse[j][2])) + fast_exp2(fmaf(acc[j][3], c2, nlse[j][3])));
            red[CP::at(t3, wid, j, 16 * sub + lr)] = sum_lane_groups(p);
          }
        } else if constexpr (MIXED) {
          // four lane-group partials per block (each block a different head's rows)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const float p = (fast_exp2(fmaf(acc[j][0], c2, nlse[j][0])) + fast_exp2(fmaf(acc[j][1], c2, nlse[j][1]))) +
                            (fast_exp2(fmaf(acc[j][2], c2, nlse[j][2])) + fast_exp2(fmaf(acc[j][3], c2, nlse[j][3])));
            red[CP::at(t3, wid, 4 * j + lg, 16 * sub + lr)] = p;
          }
        } else {
          float p = 0.f;
          if constexpr (NB > 0) {
            // four independent partial sums (one per row slot) keep the add chains short
            float pp[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pp[i] = fast_exp2(fmaf(acc[0][i], c2, nlse[0][i]));
#pragma unroll
            for (int j = 1; j < NB; ++j)
#pragma unroll
              for (int i = 0; i < 4; ++i) pp[i] += fast_exp2(fmaf(acc[j][i], c2, nlse[j][i]));
            p = (pp[0] + pp[1]) + (pp[2] + pp[3]);
          }
          red[CP::at(t3, wid, lg, 16 * sub + lr)] = p;  // one partial per lane group; the reduction adds them
        }
      },
      [&](int64_t t) { reduce(t - 1); });
  __syncthreads();
  reduce(ntiles - 1);
}

template <typename T, int D, int RBW, bool MAXG, bool HW>
__global__ __launch_bounds__(kScoreBlock, 1) void colsum_kernel(CompressArgs a) {
  using G = TileGeom<T, D>;
  __shared__ __attribute__((aligned(16))) char ktile[2 * col_tile<T>() * G::LDS_STRIDE];
  __shared__ __attribute__((aligned(16)))
  float red[ColPartials<T, block_partials<MAXG, HW>() ? RBW : 4, bal_extra_rows<MAXG, HW, RBW>()>::WORDS];
  __shared__ float qws[MAXG ? kMaxSplitRows / 16 : 1];  // Ipt. max: the row split's head weights
  const int seg = blockIdx.y;
  const int b = seg / a.Hkv, h = seg % a.Hkv;
  if (blockIdx.x == 0 && blockIdx.z == 0) init_segment(a, seg);  // histograms, offsets for the selection
  const int64_t key0 = (int64_t)blockIdx.x * a.score_chunk;
  if (key0 >= a.n_scored) return;
  const int64_t key_end = key0 + a.score_chunk < a.n_scored ? key0 + a.score_chunk : a.n_scored;
  const int tid = threadIdx.x, wid = tid >> 6, lane = tid & 63;
  const int r0 = (int)blockIdx.z * a.rs_rows;
  const int nrows = a.R - r0 < a.rs_rows ? a.R - r0 : a.rs_rows;
  const rsrc_t kr = make_rsrc(static_cast<const T*>(a.k) + (int64_t)seg * a.C * D, (uint64_t)a.C * G::RB);
  // balanced head waves: a split of seven heads of one wave each, four blocks per head (with
  // three blocks per head the busiest SIMD would carry six blocks either way)
  constexpr bool can_bal = MAXG && HW && RBW == 4;
  const bool bal = can_bal && nrows == 7 * a.w && a.w == 16 * RBW;
  Frag<T> qa[RBW][G::NC];
  load_group_queries<T, D, RBW, HW>(a, b, h, r0, nrows, wid, lane, qa, bal);
  const int nrb = (nrows + 15) / 16;
  if constexpr (HW) {
    // a row split holds whole heads of w/16 blocks, a multiple of RBW: each wave has all
    // RBW of its blocks or none (a wave without rows still stages keys and meets every barrier)
    if constexpr (can_bal) {
      if (bal && wid >= kBalFirstWave) {
        Frag<T> qb[3][G::NC];  // waves 4-6: their first three blocks; wave 7: the three lent blocks
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
          for (int c = 0; c < G::NC; ++c) qb[j][c] = qa[j][c];
        if (wid == kScoreWaves - 1)
          colsum_chunk<T, D, 3, RBW, MAXG, HW, true>(a, ktile, red, qws, seg, r0, nrows, wid, lane, qb, kr, key0,
                                                     key_end, bal);
        else
          colsum_chunk<T, D, 3, RBW, MAXG, HW>(a, ktile, red, qws, seg, r0, nrows, wid, lane, qb, kr, key0, key_end,
                                               bal);
        return;
      }
    }
    // (every wave reduces some columns, so each needs to know the layout: bal goes to all)
    if (row_block<RBW, HW>(wid, 0) < nrb) {
      colsum_chunk<T, D, RBW, RBW, MAXG, HW>(a, ktile, red, qws, seg, r0, nrows, wid, lane, qa, kr, key0, key_end, bal);
    } else {
      Frag<T> qz[1][G::NC];  // never read: the wave has no row blocks
#pragma unroll
      for (int c = 0; c < G::NC; ++c) qz[0][c] = qa[0][c];
      colsum_chunk<T, D, 0, RBW, MAXG, HW>(a, ktile, red, qws, seg, r0, nrows, wid, lane, qz, kr, key0, key_end, bal);
    }
  } else if (wid + kScoreWaves * (RBW - 1) < nrb) {
    colsum_chunk<T, D, RBW, RBW, MAXG, HW>(a, ktile, red, qws, seg, r0, nrows, wid, lane, qa, kr, key0, key_end);
  } else {
    Frag<T> qb[RBW > 1 ? RBW - 1 : 1][G::NC];
#pragma unroll
    for (int j = 0; j < RBW - 1; ++j)
#pragma unroll
      for (int c = 0; c < G::NC; ++c) qb[j][c] = qa[j][c];
    colsum_chunk<T, D, RBW - 1, RBW, MAXG, HW>(a, ktile, red, qws, seg, r0, nrows, wid, lane, qb, kr, key0, key_end);
  }
}

// Pass 2 with the keys in registers -------------------------------------------
//
// For bf16 keys and workgroups that give every wave seven turns or more (all aggregations but Ipt. max): the
// window rows of the split sit in LDS, and each wave takes 64 keys at a time into registers, straight
// from global memory (the next 64 in flight), and walks over all row blocks. A key's sum then stays in
// its lanes until the end: no column partials in LDS, no barrier after the start, every wave all of
// the rows (28 blocks over 8 waves left one wave of a SIMD 4 and the other 3). The waves of a SIMD run
// freely, and the older one gets most of the issue slots, so the turns are handed out by an LDS
// counter, last keys of the chunk first (pass 1 left those in the last-level cache).
//   The step's order, each logit's fma, exp2 and add one MFMA apart from the next one's, is pinned:
// what one wave's MFMAs leave of the vector port is what bounds it (before the order was
// pinned 29.2 cycles per MFMA and its vector work against 31.3 with the key tiles in LDS, counters at 128K
// x 8; a register-only probe of the same instructions: 26.8, and 25.2 with one wave of a SIMD on
// each kind of work). Per launch, tiles / this: 1M x 4 x 4 heads 1954 -> 1738 us, 256K
// x 4 x 8 heads of d 64 238 -> 207, 256K x 2 with a 32-token window 142 -> 121, 64K x 8 heads of d 64
// with 128 rows 40 -> 32.
constexpr int kKeyTurn = 64;  // keys of a wave's turn
// keys of a workgroup from which the turns are worth it: up to sixteen row blocks; with up to 24 twice,
// with more three times as many
constexpr int kKeyChunkMin = 3584;

template <typename T, int D>
__global__ __launch_bounds__(kScoreBlock, 1) void colsum_keys_kernel(CompressArgs a) {
  using G = TileGeom<T, D>;
  constexpr int KS = kKeyTurn / 16;
  __shared__ __attribute__((aligned(16))) char qt[kMaxSplitRows * G::LDS_STRIDE];  // the split's window rows
  __shared__ __attribute__((aligned(16))) float nl[kMaxSplitRows];                 // -lse2 + log2 weight of each
  __shared__ int next_turn;
  const int seg = blockIdx.y;
  const int b = seg / a.Hkv, h = seg % a.Hkv;
  if (blockIdx.x == 0 && blockIdx.z == 0) init_segment(a, seg);  // histograms, offsets for the selection
  const int64_t key0 = (int64_t)blockIdx.x * a.score_chunk;
  if (key0 >= a.n_scored) return;
  const int64_t key_end = key0 + a.score_chunk < a.n_scored ? key0 + a.score_chunk : a.n_scored;
  const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lr = lane & 15, lg = lane >> 4;
  const int r0 = (int)blockIdx.z * a.rs_rows;
  const int nrows = a.R - r0 < a.rs_rows ? a.R - r0 : a.rs_rows;
  const int nrb = (nrows + 15) / 16;
  const rsrc_t kr = make_rsrc(static_cast<const T*>(a.k) + (int64_t)seg * a.C * D, (uint64_t)a.C * G::RB);
  const int turns = (int)((key_end - key0 + kKeyTurn - 1) / kKeyTurn);
  // turn t takes keys [key0 + (turns-1-t)*64, +64); past the last turn the keys read as zeros (the
  // clamp keeps byte offsets below 4 GiB)
  auto load_keys = [&](int t, Frag<T>(&f)[KS][G::NC]) {
    const int64_t k = t < turns ? key0 + (int64_t)(turns - 1 - t) * kKeyTurn : a.C;
    const int64_t key = k < a.C ? k : a.C;
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
      for (int c = 0; c < G::NC; ++c)
        f[u][c] = gload_frag<T>(kr, (uint32_t)((key + 16 * u + lr) * G::RB + (32 * c + 8 * lg) * G::EB));
  };
  Frag<T> kb[2][KS][G::NC];
  load_keys(wid, kb[0]);
  if (tid == 0) next_turn = kScoreWaves;
  {
    const T* qbase = static_cast<const T*>(a.q_win) + ((int64_t)(b * a.Hq + h * a.G) * a.w + r0) * D;
    const rsrc_t qr = make_rsrc(qbase, (uint64_t)nrows * G::RB);  // rows >= nrows read as zeros
    for (int v = tid; v < nrb * 16 * G::V16; v += kScoreBlock) {
      const int row = v / G::V16, c16 = v % G::V16;
      *reinterpret_cast<u32x4*>(qt + row * G::LDS_STRIDE + c16 * 16) = ld128(qr, (uint32_t)(row * G::RB + c16 * 16));
    }
    const bool natural = a.window_lse != nullptr;
    const rsrc_t lr2 = make_rsrc(natural ? (const void*)a.window_lse : (const void*)a.lse2,
                                 (uint64_t)a.B * a.Hkv * a.R * sizeof(float));
    for (int row = tid; row < nrb * 16; row += kScoreBlock) {
      float l = ldf(lr2, (uint32_t)(((int64_t)seg * a.R + r0 + row) * 4));
      if (natural) l *= 1.44269504088896340736f;
      const float lw = a.agg != 0 && row < nrows ? a.qweight[h * a.G + (r0 + row) / a.w] : 0.f;
      nl[row] = row < nrows ? lw - l : -INFINITY;  // rows past R add 0
    }
  }
  __syncthreads();
  const float c2 = a.c2;
  const int nseg = a.B * a.Hkv;
  const rsrc_t cr = make_rsrc(a.colsum + ((int64_t)blockIdx.z * nseg + seg) * a.n_scored, (uint64_t)a.n_scored * 4);
  const char* qlane = qt + lr * G::LDS_STRIDE + 8 * lg * G::EB;
  auto row_frags = [&](int rb, Frag<T>(&f)[G::NC]) {
#pragma unroll
    for (int c = 0; c < G::NC; ++c) f[c] = lds_frag<T>(qlane, (uint32_t)(rb * 16 * G::LDS_STRIDE + 32 * c * G::EB));
  };
  auto turn = [&](int t, const Frag<T>(&k)[KS][G::NC]) {
    float p[KS][4];  // the lane's sums, by key subtile and row slot
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) p[u][i] = 0.f;
    Frag<T> qf[2][G::NC];
    f32x4 acc[2][KS], n4[2];
    auto row_consts = [&](int rb) { return *reinterpret_cast<const f32x4*>(nl + 16 * rb + 4 * lg); };
    row_frags(0, qf[0]);
    row_frags(1 < nrb ? 1 : 0, qf[1]);
    n4[0] = row_consts(0);
#pragma unroll
    for (int c = 0; c < G::NC; ++c)
#pragma unroll
      for (int u = 0; u < KS; ++u) acc[0][u] = mma(qf[0][c], k[u][c], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[0][u]);
    // the vector work of row block rb and, with `more`, the products of block rb + 1
    auto step = [&](int rb, int par, bool more) {
      if (more) {
        row_frags(rb + 2 < nrb ? rb + 2 : nrb - 1, qf[par]);
        n4[par ^ 1] = row_consts(rb + 1);
      }
      constexpr int N = 4 * KS, NM = G::NC * KS;
      float f[N], e[N];
#pragma unroll
      for (int x = 0; x < N + 2; ++x) {
        if (more)
#pragma unroll
          for (int q = 0; q < NM; ++q)
            if (q >= x * NM / N && q < (x + 1) * NM / N) {
              const int c = q / KS, u = q % KS;
              acc[par ^ 1][u] = mma(qf[par ^ 1][c], k[u][c], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[par ^ 1][u]);
            }
        if (x < N) f[x] = fmaf(acc[par][x / 4][x % 4], c2, n4[par][x % 4]);
        if (x >= 1 && x - 1 < N) e[x - 1] = fast_exp2(f[x - 1]);
        if (x >= 2) p[(x - 2) / 4][(x - 2) % 4] += e[x - 2];
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int rb = 0;
    for (; rb + 2 < nrb; rb += 2) {
      step(rb, 0, true);
      step(rb + 1, 1, true);
    }
    if (rb + 1 < nrb) {
      step(rb, 0, true);
      step(rb + 1, 1, false);
    } else {
      step(rb, 0, false);
    }
    // every lane has its column's total of each subtile; lane group lg stores subtile lg
    float x = 0.f;
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      const float v = sum_lane_groups((p[u][0] + p[u][1]) + (p[u][2] + p[u][3]));
      x = lg == u ? v : x;
    }
    const int64_t key = key0 + (int64_t)(turns - 1 - t) * kKeyTurn + lane;
    stf(cr, key < key_end ? (uint32_t)(key * 4) : (uint32_t)(a.n_scored * 4), x * a.out_scale);
  };
  static_assert(KS == 4, "one subtile per lane group");
  auto take = [&]() {
    int t = 0;
    if (lane == 0) t = __hip_atomic_fetch_add(&next_turn, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return __builtin_amdgcn_readfirstlane(t);
  };
  int t0 = wid;
  while (t0 < turns) {
    const int t1 = take();
    load_keys(t1, kb[1]);
    turn(t0, kb[0]);
    if (t1 >= turns) break;
    t0 = take();
    load_keys(t0, kb[0]);
    turn(t1, kb[1]);
  }
}

// Host-side dispatch ----------------------------------------------------------
// Pass 2 with RBW row blocks per wave for its row split.
template <typename T, int D, int RBW>
static hipError_t launch_colsum_t(const CompressArgs& a, hipStream_t st) {
  const dim3 sblk(kScoreBlock);
  if (a.n_col_chunks > 0) {
    const dim3 cgrid(a.n_col_chunks, a.B * a.Hkv, a.n_rsplit);
    if constexpr (sizeof(T) == 2) {
      // The keys a workgroup has make the difference: short chunks lose to the last turns' spread and
      // to filling the rows' LDS, the more rows the longer, and the more so where pass 1 has not left the
      // keys in the last-level cache (a given LSE). Whole call over inputs in turn, tiles / this: 128 rows at
      // 2048 keys 88.2 / 90.4 us, 4096 161.7 / 157.4, 8192 294 / 282; 256 rows at 2048 114.0 / 115.2, 4096 212 /
      // 204, 16384 741 / 694; 320 rows at 8192 444 / 426 (LSE given 259 / 250), 384 486 / 473 (275 / 275); 448
      // rows at 4096 279.5 / 280.3, 8192 531 / 529 (298 / 301), 16384 1035 / 1010 (580 / 564); 512 rows at 8192 582 /
      // 585 (325 / 330), 16384 1149 / 1128 (639 / 618). A chunk holds no more keys than its segment: 256 sequences
      // of 1024 keys, 256 rows, 312 / 332, 64 of 3072 161.7 / 157.9. Ipt. max loses to its reduction per head
      // (100K x 1: 98 / 102 for the pass).
      const int nrb = (a.rs_rows + 15) / 16;
      const int64_t keys = a.score_chunk < a.n_scored ? a.score_chunk : a.n_scored;
      if (a.agg != 1 && keys >= (nrb <= 16 ? kKeyChunkMin : nrb <= 24 ? 2 * kKeyChunkMin : 3 * kKeyChunkMin)) {
        SGDKV_LAUNCH("score_colsum", (colsum_keys_kernel<T, D>), cgrid, sblk, st, a);
        return hipGetLastError();
      }
    }
    if (a.agg == 1 && a.w % (16 * RBW) == 0)
      SGDKV_LAUNCH("score_colsum", (colsum_kernel<T, D, RBW, true, true>), cgrid, sblk, st, a);
    else if (a.agg == 1)
      SGDKV_LAUNCH("score_colsum", (colsum_kernel<T, D, RBW, true, false>), cgrid, sblk, st, a);
    else
      SGDKV_LAUNCH("score_colsum", (colsum_kernel<T, D, RBW, false, false>), cgrid, sblk, st, a);
  }
  return hipGetLastError();
}

template <typename T, int D, int RBW>
struct ColsumLaunch {
  static hipError_t run(const CompressArgs& a, hipStream_t st) { return launch_colsum_t<T, D, RBW>(a, st); }
};

hipError_t launch_scores(const CompressArgs& a, hipStream_t st) {
  if (a.window_lse == nullptr) {
    const hipError_t e = launch_lse(a, st);
    if (e != hipSuccess) return e;
  }
  if (a.dtype == 1) {
    if (a.D == 128) return dispatch_rbw<__bf16, 128, ColsumLaunch>(a.rs_rows, a, st);
    if (a.D == 64) return dispatch_rbw<__bf16, 64, ColsumLaunch>(a.rs_rows, a, st);
  } else {
    if (a.D == 128) return dispatch_rbw<float, 128, ColsumLaunch>(a.rs_rows, a, st);
    if (a.D == 64) return dispatch_rbw<float, 64, ColsumLaunch>(a.rs_rows, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace sgdkv
