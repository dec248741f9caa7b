// Pass 2 of the observation-window scoring, the kernel with the key tiles in LDS (score_kernels.hip has
// the overview of both passes). Its instances are compiled in two files, score_kernels.hip and, with
// another instruction scheduler, score_kernels_ilp.hip.
#pragma once

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

// Instances compiled with the scheduler that puts instruction parallelism first: bf16 keys at d = 64
// with sums over all rows and one, two or four row blocks per wave, with Ipt. max one or four; at d = 128 Ipt. max
// with three. Pass 2 with it / without, four heads: d 64, 13601 x 5 of 8 heads, 32 rows 23.8 / 24.7 us, 32K x 2,
// 256 rows 18.8 / 19.4, 448 26.3 / 27.1, 384 24.6 / 24.2; Ipt. max, 32K x 8, 32 rows 35.0 / 36.9, 128 47.7 / 49.0, 192 60.2 /
// 58.6, 384 110.8 / 110.5, 512 101.3 / 102.7; d 128 Ipt. max 128 rows 70.9 / 68.1, 256 90.0 / 86.9, 384 135.5 / 139.0,
// 448 124.7 / 127.2 (but 100K x 1 of 896 rows 96.8 / 95.6), sums over all rows 448 rows 35.7 / 35.2 (128K x 8 435 /
// 428). fp32 keys within 1 % either way.
template <typename T>
constexpr bool colsum_sched_ilp(int d, int rbw, bool maxg) {
  if (sizeof(T) != 2) return false;
  if (d == 64) return maxg ? rbw == 1 || rbw == 4 : rbw != 3;
  return maxg && rbw == 3;
}

// Launches the tile kernel's instances of this file (ILP: score_kernels_ilp.hip).
template <bool ILP>
struct ColsumTiles {
  template <typename T, int D, int RBW>
  struct Launch {
    template <bool MAXG, bool HW>
    static hipError_t tiles(const CompressArgs& a, hipStream_t st) {
      if constexpr (colsum_sched_ilp<T>(D, RBW, MAXG) == ILP) {
        SGDKV_LAUNCH("score_colsum", (colsum_kernel<T, D, RBW, MAXG, HW>), dim3(a.n_col_chunks, a.B * a.Hkv, a.n_rsplit),
                     dim3(kScoreBlock), st, a);
        return hipGetLastError();
      } else {
        return hipErrorInvalidValue;
      }
    }
    static hipError_t run(const CompressArgs& a, hipStream_t st) {
      if (a.agg != 1) return tiles<false, false>(a, st);
      return a.w % (16 * RBW) == 0 ? tiles<true, true>(a, st) : tiles<true, false>(a, st);
    }
  };
  static hipError_t launch(const CompressArgs& a, hipStream_t st) {
    if (a.dtype == 1) {
      if (a.D == 128) return dispatch_rbw<__bf16, 128, Launch>(a.rs_rows, a, st);
      if (a.D == 64) return dispatch_rbw<__bf16, 64, Launch>(a.rs_rows, a, st);
    } else if constexpr (!ILP) {
      if (a.D == 128) return dispatch_rbw<float, 128, Launch>(a.rs_rows, a, st);
      if (a.D == 64) return dispatch_rbw<float, 64, Launch>(a.rs_rows, a, st);
    }
    return hipErrorInvalidValue;
  }
};

hipError_t launch_colsum_ilp(const CompressArgs& a, hipStream_t st);  // ColsumTiles<true>::launch

}  // namespace sgdkv
