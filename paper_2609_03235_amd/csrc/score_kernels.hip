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
//   pass 1 (lse_kernel + lse_merge_kernel): base-2 log-sum-exp of every
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
// workgroups per key chunk (grid z = row split). Pass 1 partials are per row
// anyway; pass 2 then leaves one column-sum partial per split, which the
// pooling pass adds (or, for Ipt. max, maximises) in split order. Each key tile (128 keys; 64 in pass 2
// for fp32 keys) is staged once in LDS and read by all eight waves as B-fragments;
// blocks past the last row are skipped. MFMA 16x16x32 bf16 (or 8 x 16x16x4
// f32 for fp32 inputs) accumulates in fp32.
// Output layout of a 16x16 MFMA: lane l holds rows 4*(l/16)+0..3 of key
// column l%16.
#include "device_common.h"
#include "mfma_frag.h"
#include "sgdkv_internal.h"
#include "segment_init.h"

// Row blocks per wave the dispatch instantiates: at most 512 rows (one row split) over all waves.
#define SGDKV_SCORE_WAVES_MAX_RBW (kMaxSplitRowsMacro / (16 * SGDKV_SCORE_WAVES))
#define kMaxSplitRowsMacro 512

namespace sgdkv {

// Shared pieces of both passes ------------------------------------------------
template <typename T>
constexpr int col_tile() {
  return sizeof(T) == 2 ? kColTileBf16 : kColTileF32;
}

template <typename T, int D>
struct TileGeom {
  static constexpr int EB = elt_bytes<T>();
  static constexpr int RB = D * EB;           // bytes per key row
  static constexpr int LDS_STRIDE = RB + 32;  // padded row pitch: 16-B fragment reads free of bank conflicts (measured)
  static constexpr int NC = D / 32;           // 32-wide k chunks
  static constexpr int V16 = RB / 16;         // 16-byte vectors per row
};

// K tile staging: keys [tile0, tile0+TILE) of this head travel global -> registers
// (issued one tile ahead) -> LDS. Keys past the end of the head read as zeros.
template <typename T, int D, int TILE>
struct KeyStage {
  using G = TileGeom<T, D>;
  static constexpr int TOT = TILE * G::V16;                        // 16-byte vectors per tile
  static constexpr int N = (TOT + kScoreBlock - 1) / kScoreBlock;  // per thread
  static constexpr bool ALL = TOT >= kScoreBlock;                  // every thread moves N vectors
  static_assert(TOT % kScoreBlock == 0 || !ALL, "tile must split evenly");
  u32x4 r[N];
  __device__ __forceinline__ void load(rsrc_t kr, int64_t tile0) {
    if (ALL || (int)threadIdx.x < TOT) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int vi = threadIdx.x + u * kScoreBlock;
        const int row = vi / G::V16, c16 = vi % G::V16;
        r[u] = ld128(kr, (uint32_t)((tile0 + row) * G::RB + c16 * 16));
      }
    }
  }
  __device__ __forceinline__ void store(char* ktile) const {
    if (ALL || (int)threadIdx.x < TOT) {
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int vi = threadIdx.x + u * kScoreBlock;
        const int row = vi / G::V16, c16 = vi % G::V16;
        *reinterpret_cast<u32x4*>(ktile + row * G::LDS_STRIDE + c16 * 16) = r[u];
      }
    }
  }
};

// Row block of slot j of wave wid: blocks wid, wid+8, ... (interleaved), or, with HW (head
// waves), blocks wid*RBW .. wid*RBW+RBW-1, so that the rows of a wave belong to one query head
// when w is a multiple of 16*RBW. Balanced head waves (bal: seven heads of one wave each, the
// group size of a 28/4-head model): the last wave, which would hold no rows, takes the last
// block of the heads of waves 4-6 (slots 0-2), so that each SIMD (waves s and s+4) carries
// 2*RBW - 1 blocks instead of 2*RBW on three SIMDs and RBW on the fourth.
constexpr int kBalFirstWave = kScoreWaves / 2;  // heads of waves 4-6 lend their last block
template <int RBW, bool HW>
__device__ __forceinline__ int row_block(int wid, int j, bool bal = false) {
  if (HW && bal && wid == kScoreWaves - 1) return (kBalFirstWave + j) * RBW + RBW - 1;
  return HW ? wid * RBW + j : wid + kScoreWaves * j;
}

// Window rows [r0, r0 + nrows) of KV head h (one row split) as A fragments.
template <typename T, int D, int RBW, bool HW = false>
__device__ __forceinline__ void load_group_queries(const CompressArgs& a, int b, int h, int r0, int nrows, int wid,
                                                   int lane, Frag<T> (&qa)[RBW][D / 32], bool bal = false) {
  using G = TileGeom<T, D>;
  const T* qbase = static_cast<const T*>(a.q_win) + ((int64_t)(b * a.Hq + h * a.G) * a.w + r0) * D;
  const rsrc_t qr = make_rsrc(qbase, (uint64_t)nrows * G::RB);
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int j = 0; j < RBW; ++j) {
    const int row = row_block<RBW, HW>(wid, j, bal) * 16 + lr;  // rows >= nrows read as zeros
#pragma unroll
    for (int c = 0; c < G::NC; ++c)
      qa[j][c] = gload_frag<T>(qr, (uint32_t)(row * G::RB + (32 * c + 8 * lg) * G::EB));
  }
}

// Chunk pipeline --------------------------------------------------------------
//
// A workgroup streams the key tiles of its chunk through two LDS buffers and
// the MFMAs as one rolling pipeline. In step s of tile t a wave issues the
// MFMAs of the next subtile (16 keys), reads the key fragments of the subtile
// after that from LDS, and hands the logits of subtile s to the vector ALU.
// Tile t+1 goes into the other buffer at the start of tile t (its global loads
// were issued one tile earlier), and the tile's single barrier, two subtiles
// before its end, makes that buffer readable; the buffer written at the start
// of tile t was last read before the barrier of tile t-1. The MFMAs of the
// subtile after the chunk's last one run on whatever keys follow (zeros past
// the head) and are discarded. REV streams the chunk's tiles last to first
// (step t covers tile ntiles-1-t; the steps after the last read zeros). On
// gfx950 a wave's own MFMAs and vector instructions issue one after the other,
// and exp2 overlaps little with the MFMAs of the SIMD's other wave; the two
// waves of a SIMD mainly hide each other's latencies.
template <typename T, int D, int NB>
__device__ __forceinline__ void subtile_mfma(const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32],
                                             const Frag<T> (&kb)[D / 32], f32x4 (&acc)[NB > 0 ? NB : 1]) {
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = mma(qa[j][c], kb[c], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[j]);
}

// One step of the pipeline: the MFMAs of the next subtile and, between them, the vector work on the
// logits of the current one, each logit's fma, exp2 and use one MFMA apart so that none waits for
// the one before it.
template <typename T, int D, int NB, typename Arg, typename Use>
__device__ __forceinline__ void subtile_step(const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32], const Frag<T> (&kb)[D / 32],
                                             f32x4 (&nxt)[NB > 0 ? NB : 1], const f32x4 (&cur)[NB > 0 ? NB : 1],
                                             Arg&& arg, Use&& use) {
  constexpr int N = 4 * NB, NM = D / 32 * NB, N1 = N > 0 ? N : 1;
  float f[N1], e[N1];
#pragma unroll
  for (int k = 0; k < N + 2; ++k) {
#pragma unroll
    for (int q = 0; q < NM; ++q)
      if (q >= k * NM / N1 && q < (k + 1) * NM / N1) {
        const int c = q / (NB > 0 ? NB : 1), j = q % (NB > 0 ? NB : 1);
        nxt[j] = mma(qa[j][c], kb[c], c == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : nxt[j]);
      }
    if (k < N) f[k] = arg(k / 4, k % 4, cur[k / 4][k % 4]);
    if (k >= 1 && k - 1 < N) e[k - 1] = fast_exp2(f[k - 1]);
    if (k >= 2) use((k - 2) / 4, (k - 2) % 4, e[k - 2]);
  }
}

template <typename T, int D>
__device__ __forceinline__ void subtile_frags(const char* ktile, int t, int lr, int lg, Frag<T> (&kb)[D / 32]) {
  using G = TileGeom<T, D>;
#pragma unroll
  for (int c = 0; c < G::NC; ++c)
    kb[c] = lds_frag<T>(ktile, (uint32_t)((16 * t + lr) * G::LDS_STRIDE + (32 * c + 8 * lg) * G::EB));
}

// Hooks: begin(acc) once with the logits of the chunk's first subtile (before
// any sub call); sub(t, s, acc) per subtile; at_barrier(t) right after tile t's
// barrier. SKEW: sub(t, s, acc, nxt, kb) issues the next subtile's MFMAs itself,
// between its vector work.
template <typename T, int D, int NB, int TILE, bool REV, bool SKEW, typename Begin, typename Sub, typename AtBarrier>
__device__ __forceinline__ void chunk_pipeline(char* kbuf, const rsrc_t& kr, int64_t key0, int64_t C, int64_t ntiles,
                                               int lr, int lg, const Frag<T> (&qa)[NB > 0 ? NB : 1][D / 32],
                                               Begin&& begin, Sub&& sub, AtBarrier&& at_barrier) {
  using G = TileGeom<T, D>;
  constexpr int NBX = NB > 0 ? NB : 1;
  constexpr int S = TILE / 16;
  constexpr int BUF = TILE * G::LDS_STRIDE;
  static_assert(S >= 4 && S % 2 == 0, "tile geometry");
  // keys past the head read as zeros; the clamp keeps byte offsets below 4 GiB
  auto tile_key = [&](int64_t t) {
    const int64_t k = REV ? (t < ntiles ? key0 + (ntiles - 1 - t) * TILE : C) : key0 + t * TILE;
    return k < C ? k : C;
  };
  KeyStage<T, D, TILE> stage;
  stage.load(kr, tile_key(0));
  stage.store(kbuf);
  stage.load(kr, tile_key(1));
  __syncthreads();
  Frag<T> kb[2][D / 32];
  f32x4 acc[2][NBX];
  subtile_frags<T, D>(kbuf, 0, lr, lg, kb[0]);
  subtile_frags<T, D>(kbuf, 1, lr, lg, kb[1]);
  subtile_mfma<T, D, NB>(qa, kb[0], acc[0]);
  begin(acc[0]);
  for (int64_t t = 0; t < ntiles; ++t) {
    const char* buf = kbuf + (t & 1) * BUF;
    char* nbuf = kbuf + ((t + 1) & 1) * BUF;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (s == 0) {
        stage.store(nbuf);
        stage.load(kr, tile_key(t + 2));
      }
      if (s == S - 2) {
        __syncthreads();
        at_barrier(t);
      }
      if constexpr (!SKEW) subtile_mfma<T, D, NB>(qa, kb[(s + 1) & 1], acc[(s + 1) & 1]);
      if (s + 2 < S)
        subtile_frags<T, D>(buf, s + 2, lr, lg, kb[s & 1]);
      else
        subtile_frags<T, D>(nbuf, s + 2 - S, lr, lg, kb[s & 1]);
      if constexpr (SKEW)
        sub(t, s, acc[s & 1], acc[(s + 1) & 1], kb[(s + 1) & 1]);
      else
        sub(t, s, acc[s & 1]);
    }
  }
}

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
    chunk_pipeline<T, D, NB, TILE, false, true>(
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
        [&](int64_t, int, const f32x4(&acc)[NBX], f32x4(&nxt)[NBX], const Frag<T>(&kb)[D / 32]) {
          subtile_step<T, D, NB>(qa, kb, nxt, acc, [&](int j, int i, float x) { return fmaf(x, c2, -m[j][i]); },
                                 [&](int j, int i, float e) { s[j][i] += e; });
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
  // last uniform chunk's workgroup goes on to them. Keys past the last window row's position are
  // seen by no row.
  const int chunk = (int)blockIdx.y;
  const int64_t key0 = (int64_t)chunk * a.lse_chunk;
  const int64_t key_end = key0 + a.lse_chunk < a.lse_tail0 ? key0 + a.lse_chunk : a.lse_tail0;
  const int tail0 = chunk >= a.n_lse_head ? chunk : a.n_lse_head;  // tail chunks of this workgroup
  const int tail1 = chunk >= a.n_lse_head ? chunk + 1
                    : chunk == a.n_lse_head - 1 && (int)gridDim.y == a.n_lse_head ? a.n_lse_chunks : 0;
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
    for (int c = tail0; c < tail1; ++c) lse_tail<T, D, RBW>(a, seg, c, r0, nrows, wid, lane, qa, kr);
  } else {
    Frag<T> qb[RBW > 1 ? RBW - 1 : 1][G::NC];
#pragma unroll
    for (int j = 0; j < RBW - 1; ++j)
#pragma unroll
      for (int c = 0; c < G::NC; ++c) qb[j][c] = qa[j][c];
    if (chunk < a.n_lse_head)
      lse_chunk<T, D, RBW - 1>(a, ktile, seg, chunk, r0, nrows, wid, lane, qb, kr, key0, key_end);
    for (int c = tail0; c < tail1; ++c) lse_tail<T, D, RBW - 1>(a, seg, c, r0, nrows, wid, lane, qb, kr);
  }
}

// Merge the per-chunk partials of every window row in fp64: 16 lanes per row (16 rows per
// workgroup of segment blockIdx.y), lane l taking chunks l, l+16, ...; the maximum of the chunk
// references over the 16 lanes, then each lane's rescaled sums in chunk order, and the 16 lane
// sums added in a fixed butterfly order. A row's lanes read neighbouring chunks' partials.
constexpr int kMergeLanes = 16;
__global__ __launch_bounds__(kBlock) void lse_merge_kernel(CompressArgs a) {
  const int64_t seg = blockIdx.y;
  const int lane = threadIdx.x % kMergeLanes;
  const int row = blockIdx.x * (kBlock / kMergeLanes) + threadIdx.x / kMergeLanes;
  const bool live = row < a.R;  // every lane takes part in the shuffles
  const int n = a.n_lse_chunks;
  const rsrc_t pr = make_rsrc(a.lse_part + seg * n * a.R * 2, (uint64_t)n * a.R * 2 * sizeof(float));
  auto off = [&](int c) { return (uint32_t)(((int64_t)c * a.R + row) * 8); };
  float mx = -INFINITY;
  if (live)
    for (int c = lane; c < n; c += kMergeLanes) mx = fmaxf(mx, ldf(pr, off(c)));
#pragma unroll
  for (int o = 1; o < kMergeLanes; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  double sum = 0.0;
  if (live && mx != -INFINITY) {
    for (int c = lane; c < n; c += kMergeLanes) {
      const uint64_t ms = ld64(pr, off(c));
      const float mc = __uint_as_float((uint32_t)ms), sc = __uint_as_float((uint32_t)(ms >> 32));
      if (mc != -INFINITY) sum += (double)sc * exp2((double)mc - (double)mx);
    }
  }
#pragma unroll
  for (int o = 1; o < kMergeLanes; o <<= 1) sum += __shfl_xor(sum, o, 64);
  if (!live || lane != 0) return;
  const float lse2 = (mx == -INFINITY || !(sum > 0.0)) ? -INFINITY : (float)((double)mx + log2(sum));
  const rsrc_t lr = make_rsrc(a.lse2 + seg * a.R, (uint64_t)a.R * sizeof(float));
  stf(lr, (uint32_t)row * 4u, lse2);
}

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
// For bf16 keys and chunks that give every wave several turns (all aggregations but Ipt. max): the
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
constexpr int kKeyChunkMin = 4096;       // keys of a chunk from which the turns are worth it
constexpr int kKeyChunkMinTall = 32768;  // the same for more than sixteen row blocks

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
// Pass 1 (and its merge) with RBW row blocks per wave for its row split.
template <typename T, int D, int RBW>
static hipError_t launch_lse_t(const CompressArgs& a, hipStream_t st) {
  const dim3 sblk(kScoreBlock);
  SGDKV_LAUNCH("score_lse", (lse_kernel<T, D, RBW>), dim3(a.B * a.Hkv * a.lse_n_rsplit, a.n_lse_wgs), sblk, st, a);
  constexpr int rows_per_wg = kBlock / kMergeLanes;
  SGDKV_LAUNCH("lse_merge", lse_merge_kernel, dim3((unsigned)((a.R + rows_per_wg - 1) / rows_per_wg), a.B * a.Hkv),
               dim3(kBlock), st, a);
  return hipGetLastError();
}

// Pass 2 with RBW row blocks per wave for its row split.
template <typename T, int D, int RBW>
static hipError_t launch_colsum_t(const CompressArgs& a, hipStream_t st) {
  const dim3 sblk(kScoreBlock);
  if (a.n_col_chunks > 0) {
    const dim3 cgrid(a.n_col_chunks, a.B * a.Hkv, a.n_rsplit);
    if constexpr (sizeof(T) == 2) {
      // at least 8 turns of 64 keys per wave (100K x 2 x 8 heads of d 64, 6400-key chunks: 36 us
      // against 43): shorter chunks lose to the last turns' spread and to filling the rows' LDS (32K x 1:
      // 512-key chunks, 25 us against 22), Ipt. max to its reduction per head (100K x 1: 102 against 98),
      // and three or four whole row blocks on every wave leave the tile kernel nothing uneven (64K x 4
      // with 512 rows: the pass 362 us against 352-377 from box to box; with eight or sixteen blocks in
      // all it reads the LDS too often: 64K x 8 with 128 rows of d 64, 40 us against 32)
      // With more than sixteen row blocks the chip runs at its power limit, and up to 16384-key chunks
      // what pass 2 gains the next pass 1 loses to the clock (128K x 8: pass 2 428-436 -> 407-430 us,
      // pass 1 410 -> 444); at 1M x 4 (65536) the pass gains 4-5 %.
      const int nrb = (a.rs_rows + 15) / 16;
      if (a.agg != 1 && a.score_chunk >= (nrb <= 16 ? kKeyChunkMin : kKeyChunkMinTall) &&
          (nrb <= 16 || nrb % kScoreWaves != 0)) {
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

// Row blocks per wave for a row split of `rows` rows (its largest split), as a template argument.
template <typename T, int D, template <typename, int, int> class L>
static hipError_t dispatch_rbw(int rows, const CompressArgs& a, hipStream_t st) {
  const int nrb = (rows + 15) / 16;
  switch ((nrb + kScoreWaves - 1) / kScoreWaves) {
    case 1: return L<T, D, 1>::run(a, st);
    case 2: return L<T, D, 2>::run(a, st);
    case 3: return L<T, D, 3>::run(a, st);
    case 4: return L<T, D, 4>::run(a, st);
#if SGDKV_SCORE_WAVES_MAX_RBW > 4
    case 5: return L<T, D, 5>::run(a, st);
    case 6: return L<T, D, 6>::run(a, st);
    case 7: return L<T, D, 7>::run(a, st);
    case 8: return L<T, D, 8>::run(a, st);
#endif
    default: return hipErrorInvalidValue;
  }
}
template <typename T, int D, int RBW>
struct LseLaunch {
  static hipError_t run(const CompressArgs& a, hipStream_t st) { return launch_lse_t<T, D, RBW>(a, st); }
};
template <typename T, int D, int RBW>
struct ColsumLaunch {
  static hipError_t run(const CompressArgs& a, hipStream_t st) { return launch_colsum_t<T, D, RBW>(a, st); }
};

template <typename T, int D>
static hipError_t launch_scores_d(const CompressArgs& a, hipStream_t st) {
  if (a.window_lse == nullptr) {
    const hipError_t e = dispatch_rbw<T, D, LseLaunch>(a.lse_rs_rows, a, st);
    if (e != hipSuccess) return e;
  }
  return dispatch_rbw<T, D, ColsumLaunch>(a.rs_rows, a, st);
}

hipError_t launch_scores(const CompressArgs& a, hipStream_t st) {
  if (a.dtype == 1) {
    if (a.D == 128) return launch_scores_d<__bf16, 128>(a, st);
    if (a.D == 64) return launch_scores_d<__bf16, 64>(a, st);
  } else {
    if (a.D == 128) return launch_scores_d<float, 128>(a, st);
    if (a.D == 64) return launch_scores_d<float, 64>(a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace sgdkv
