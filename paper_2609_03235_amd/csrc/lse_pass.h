// Pass 1 of the observation-window scoring, the kernel: per-chunk partials of the window rows'
// log-sum-exp (score_kernels.hip has the overview of both passes). Its instances are compiled in two
// files, lse_kernels.hip and, with another instruction scheduler, lse_kernels_ilp.hip.
#pragma once

#include "score_common.h"

namespace sgdkv {

// Pass 1: per-chunk partial log-sum-exp of every window row -------------------
//
// Each lane keeps, for each of its 4*NB row slots, a reference m and a sum
// s = sum 2^(y - m) over the keys it has seen (y = logit * log2 e). The tiles
// of the chunk that every window row sees in full run through the pipeline
// with m fixed at the row's largest logit among the chunk's first 16 keys, so
// each logit costs one fma, one exp2 and one add and the loop has no branch.
// A sum can only overflow if a later logit exceeds that maximum by about 100
// (base 2); the chunk's sums are checked once at its end and, if any left
// [0, 2^122] (inf and NaN included), the whole chunk is recomputed with the
// exact online update (two exp2 per logit, m = running max), reading the keys
// from global memory. The bound leaves room for the 16 lanes of a row, which
// share the reference and are then added as they are: 16 * 2^122 = 2^126 stays
// finite. The keys that reach the window block (causal mask) or the end of the
// head, and those before them that fill no whole tile, are tail chunks of their
// own (lse_tail). Padded rows (past R) keep m = 0.
template <typename T, int D, int NB, int TILE>
__device__ __forceinline__ void lse_exact_tile(const rsrc_t& kr, int lr, int lg, int64_t tile0,
                                               const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32], float c2,
                                               float (&m)[NB > 0 ? NB : 1][4], float (&s)[NB > 0 ? NB : 1][4]) {
  using G = TileGeom<T, D>;
  constexpr int NBX = NB > 0 ? NB : 1;
  auto load = [&](int t, Frag<T>(&kb)[D / 32]) {
#pragma unroll
    for (int c = 0; c < G::NC; ++c)
      kb[c] = gload_frag<T>(kr, (uint32_t)((tile0 + 16 * t + lr) * G::RB + (32 * c + 8 * lg) * G::EB));
  };
  Frag<T> kn[D / 32];
  load(0, kn);
#pragma unroll 1
  for (int t = 0; t < TILE / 16; ++t) {
    Frag<T> kb[D / 32];
#pragma unroll
    for (int c = 0; c < G::NC; ++c) kb[c] = kn[c];
    load(t + 1 < TILE / 16 ? t + 1 : t, kn);  // the next subtile's keys are in flight during this one
    f32x4 acc[NBX];
    subtile_mfma<T, D, NB>(qa, kb, acc);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float y = acc[j][i] * c2;
        const float mn = fmaxf(m[j][i], y);
        if (mn != -INFINITY) {
          s[j][i] = s[j][i] * fast_exp2(m[j][i] - mn) + fast_exp2(y - mn);
          m[j][i] = mn;
        }
      }
  }
}

// Combines the 16 lanes (keys) of each row and stores the row's (m, s) of this chunk.
template <int NB>
__device__ __forceinline__ void lse_store(const CompressArgs& a, int seg, int chunk, int r0, int nrows, int wid,
                                          int lane, const float (&m)[NB > 0 ? NB : 1][4],
                                          const float (&s)[NB > 0 ? NB : 1][4]) {
  const int lr = lane & 15, lg = lane >> 4;
  float* part = a.lse_part + ((int64_t)seg * a.n_lse_chunks + chunk) * a.R * 2;
  const rsrc_t pr = make_rsrc(part, (uint64_t)a.R * 2 * sizeof(float));
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float mx = row16_max(m[j][i]);
      const float ss = row16_sum(m[j][i] == -INFINITY ? 0.f : s[j][i] * fast_exp2(m[j][i] - mx));
      const int row = (wid + kScoreWaves * j) * 16 + 4 * lg + i;
      if (lr == 0 && row < nrows)
        st64(pr, (uint32_t)((r0 + row) * 8), (uint64_t)__float_as_uint(mx) | ((uint64_t)__float_as_uint(ss) << 32));
    }
}

// The keys of a tail chunk (at most kLseTail, from the last whole tile every window row sees to the
// last key some row sees): all products at once, the causal mask, then one exp2 per logit against
// the lane's own maximum. No LDS and no loop; a workgroup is bound by the latency of its queries'
// and keys' loads. (One workgroup per segment walking all of them 16 keys at a time, each load
// waiting for the one before, ended the launch on short prompts: pass 1 at 6K x 1 24 us, now 14.6,
// at 2K fp32 12 us, now 9; event pairs around the launches included.)
template <typename T, int D, int NB>
__device__ __forceinline__ void lse_tail(const CompressArgs& a, int seg, int chunk, int r0, int nrows, int wid, int lane,
                                         const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32], const rsrc_t& kr) {
  using G = TileGeom<T, D>;
  constexpr int NBX = NB > 0 ? NB : 1, S = kLseTail / 16;
  const int64_t key0 = a.lse_tail0 + (int64_t)(chunk - a.n_lse_head) * kLseTail;
  const int lr = lane & 15, lg = lane >> 4;
  Frag<T> kb[S][G::NC];
#pragma unroll
  for (int t = 0; t < S; ++t)
#pragma unroll
    for (int c = 0; c < G::NC; ++c)
      kb[t][c] = gload_frag<T>(kr, (uint32_t)((key0 + 16 * t + lr) * G::RB + (32 * c + 8 * lg) * G::EB));
  f32x4 acc[S][NBX];
#pragma unroll
  for (int t = 0; t < S; ++t) subtile_mfma<T, D, NB>(qa, kb[t], acc[t]);
  int dk[S];  // key - window position; keys past the head are never visible
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int64_t key = key0 + 16 * t + lr;
    dk[t] = key < a.C ? (int)(key - a.win0) : 1 << 30;  // tail keys lie within 2^16 of the window
  }
  float m[NBX][4], s[NBX][4];
  int wj = (r0 + wid * 16 + 4 * lg) % a.w;  // window index of the lane's first row
  const int step = (kScoreWaves * 16) % a.w;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    int wi = wj;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float y[S], mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < S; ++t) {
        y[t] = dk[t] > wi ? -INFINITY : acc[t][j][i] * a.c2;
        mx = fmaxf(mx, y[t]);
      }
      m[j][i] = mx;
      s[j][i] = 0.f;
#pragma unroll
      for (int t = 0; t < S; ++t) s[j][i] += fast_exp2(y[t] - (mx == -INFINITY ? 0.f : mx));
      wi = wi + 1 == a.w ? 0 : wi + 1;
    }
    wj = wj + step >= a.w ? wj + step - a.w : wj + step;
  }
  lse_store<NB>(a, seg, chunk, r0, nrows, wid, lane, m, s);
}

template <typename T, int D, int NB>
__device__ void lse_chunk(const CompressArgs& a, char* kbuf, int seg, int chunk, int r0, int nrows, int wid,
                          int lane, const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32], const rsrc_t& kr, int64_t key0,
                          int64_t key_end) {
  constexpr int NBX = NB > 0 ? NB : 1;
  constexpr int TILE = kLseTile;
  const int lr = lane & 15, lg = lane >> 4;
  const float c2 = a.c2;
  float m[NBX][4], s[NBX][4];
  bool real[NBX][4];
  auto reset = [&]() {
#pragma unroll
    for (int j = 0; j < NBX; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        m[j][i] = real[j][i] ? -INFINITY : 0.f;  // a padded row must not force the exact path
        s[j][i] = 0.f;
      }
  };
#pragma unroll
  for (int j = 0; j < NBX; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) real[j][i] = (wid + kScoreWaves * j) * 16 + 4 * lg + i < nrows;
  reset();
  const int64_t nfast = (key_end - key0) / TILE;  // whole tiles every row sees (>= 1)
  {
    chunk_pipeline<T, D, NB, TILE, false, sizeof(T) == 2>(
        kbuf, kr, key0, a.C, nfast, lr, lg, qa,
        [&](const f32x4(&acc)[NBX]) {
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float mx = row16_max(acc[j][i] * c2);  // every lane of the 16-lane row takes part
              if (real[j][i]) m[j][i] = mx;
            }
        },
        [&](int64_t, int, const f32x4(&acc)[NBX], auto&... next) {
          if constexpr (sizeof...(next) > 0) {
            subtile_step<T, D, NB>(qa, next..., acc, [&](int j, int i, float x) { return fmaf(x, c2, -m[j][i]); },
                                   [&](int j, int i, float e) { s[j][i] += e; });
          } else {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
              for (int i = 0; i < 4; ++i) s[j][i] += fast_exp2(fmaf(acc[j][i], c2, -m[j][i]));
          }
        },
        [&](int64_t) {});
    bool bad = false;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) bad |= !(s[j][i] <= 5.3169119831396635e36f);  // 2^122; catches inf and NaN
    if (__any(bad)) {
      reset();
      for (int64_t t = 0; t < nfast; ++t)
        lse_exact_tile<T, D, NB, TILE>(kr, lr, lg, key0 + t * TILE, qa, c2, m, s);
    }
  }
  lse_store<NB>(a, seg, chunk, r0, nrows, wid, lane, m, s);
}

template <typename T, int D, int RBW>
__global__ __launch_bounds__(kScoreBlock, 1) void lse_kernel(CompressArgs a) {
  using G = TileGeom<T, D>;
  __shared__ __attribute__((aligned(16))) char ktile[2 * kLseTile * G::LDS_STRIDE];
  const int nseg = a.B * a.Hkv;
  const int seg = (int)blockIdx.x % nseg, split = (int)blockIdx.x / nseg;
  const int b = seg / a.Hkv, h = seg % a.Hkv;
  // The uniform chunks of keys every row sees come first in the grid, then the short tail chunks, if
  // those have workgroups of their own (with both mixed segment by segment, some shader engines got
  // more long workgroups than they have compute units: 766 us for 420 at 128K x 8); otherwise the
  // last lse_tailers uniform chunks' workgroups go on to them, in turn. Keys past the last window
  // row's position are seen by no row.
  const int chunk = (int)blockIdx.y;
  const int64_t key0 = (int64_t)chunk * a.lse_chunk;
  const int64_t key_end = key0 + a.lse_chunk < a.lse_tail0 ? key0 + a.lse_chunk : a.lse_tail0;
  // tail chunks of this workgroup: tail0, tail0 + lse_tailers, ..
  const int late = a.n_lse_head - 1 - chunk;  // uniform chunks after this one, or below 0
  const int tail0 = late < 0 ? chunk : late < a.lse_tailers ? a.n_lse_head + late : a.n_lse_chunks;
  const int tstep = late < 0 ? a.n_lse_chunks : a.lse_tailers;
  const int tid = threadIdx.x, wid = tid >> 6, lane = tid & 63;
  const int r0 = split * a.lse_rs_rows;
  const int nrows = a.R - r0 < a.lse_rs_rows ? a.R - r0 : a.lse_rs_rows;
  const rsrc_t kr = make_rsrc(static_cast<const T*>(a.k) + (int64_t)seg * a.C * D, (uint64_t)a.C * G::RB);
  Frag<T> qa[RBW][G::NC];
  load_group_queries<T, D, RBW>(a, b, h, r0, nrows, wid, lane, qa);
  // blocks this wave owns: RBW or RBW-1 (uniform per wave)
  const int nrb = (nrows + 15) / 16;
  if (wid + kScoreWaves * (RBW - 1) < nrb) {
    if (chunk < a.n_lse_head)
      lse_chunk<T, D, RBW>(a, ktile, seg, chunk, r0, nrows, wid, lane, qa, kr, key0, key_end);
    for (int c = tail0; c < a.n_lse_chunks; c += tstep) lse_tail<T, D, RBW>(a, seg, c, r0, nrows, wid, lane, qa, kr);
  } else {
    Frag<T> qb[RBW > 1 ? RBW - 1 : 1][G::NC];
#pragma unroll
    for (int j = 0; j < RBW - 1; ++j)
#pragma unroll
      for (int c = 0; c < G::NC; ++c) qb[j][c] = qa[j][c];
    if (chunk < a.n_lse_head)
      lse_chunk<T, D, RBW - 1>(a, ktile, seg, chunk, r0, nrows, wid, lane, qb, kr, key0, key_end);
    for (int c = tail0; c < a.n_lse_chunks; c += tstep) lse_tail<T, D, RBW - 1>(a, seg, c, r0, nrows, wid, lane, qb, kr);
  }
}

// Instances compiled with the scheduler that puts instruction parallelism first: bf16 keys with one,
// three or four row blocks per wave at d = 128, one at d = 64. Pass 1 with it / without, 64K x 8 x 4
// heads: d 128, 64 rows 89.3 / 89.6 us, 320 rows 172.8 / 176.2, 448 222.5 / 224.3, 512 250.7 / 255.4; d 64, 64
// rows 45.0 / 49.8. The others are faster without: d 128, 256 rows 146.0 / 142.0 (32K x 32 x 8 heads 574 /
// 532), d 64, 256 rows 100.7 / 96.6, 384 138.1 / 134.8, 448 156.8 / 152.8; fp32, 64K x 4 x 4 heads of 448 rows
// 905 / 894.
template <typename T>
constexpr bool lse_sched_ilp(int d, int rbw) {
  return sizeof(T) == 2 && (d == 128 ? rbw != 2 : rbw == 1);
}

// Launches pass 1 where its instance is one of this file's (ILP: lse_kernels_ilp.hip).
template <bool ILP>
struct LsePass {
  template <typename T, int D, int RBW>
  struct Launch {
    static hipError_t run(const CompressArgs& a, hipStream_t st) {
      if constexpr (lse_sched_ilp<T>(D, RBW) == ILP) {
        SGDKV_LAUNCH("score_lse", (lse_kernel<T, D, RBW>), dim3(a.B * a.Hkv * a.lse_n_rsplit, a.n_lse_wgs),
                     dim3(kScoreBlock), st, a);
        return hipGetLastError();
      } else {
        return hipErrorInvalidValue;
      }
    }
  };
  static hipError_t launch(const CompressArgs& a, hipStream_t st) {
    if (a.dtype == 1) {
      if (a.D == 128) return dispatch_rbw<__bf16, 128, Launch>(a.lse_rs_rows, a, st);
      if (a.D == 64) return dispatch_rbw<__bf16, 64, Launch>(a.lse_rs_rows, a, st);
    } else if constexpr (!ILP) {
      if (a.D == 128) return dispatch_rbw<float, 128, Launch>(a.lse_rs_rows, a, st);
      if (a.D == 64) return dispatch_rbw<float, 64, Launch>(a.lse_rs_rows, a, st);
    }
    return hipErrorInvalidValue;
  }
};

hipError_t launch_lse_ilp(const CompressArgs& a, hipStream_t st);  // LsePass<true>::launch

}  // namespace sgdkv
