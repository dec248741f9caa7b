// What the two score passes (lse_kernels.hip, score_kernels.hip) share: the staging of key tiles, the
// window rows as MFMA fragments, the chunk pipeline, the choice of row blocks per wave.
#pragma once

#include "device_common.h"
#include "mfma_frag.h"
#include "sgdkv_internal.h"

// Row blocks per wave the dispatch instantiates: at most 512 rows (one row split) over all waves.
#define SGDKV_SCORE_WAVES_MAX_RBW (kMaxSplitRowsMacro / (16 * SGDKV_SCORE_WAVES))
#define kMaxSplitRowsMacro 512

namespace sgdkv {

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
// barrier. SKEW: sub(t, s, acc, kb, nxt) issues the next subtile's MFMAs itself,
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
        sub(t, s, acc[s & 1], kb[(s + 1) & 1], acc[(s + 1) & 1]);
      else
        sub(t, s, acc[s & 1]);
    }
  }
}

// Row blocks per wave for a row split of `rows` rows (its largest split), and as a template argument.
constexpr int row_blocks_per_wave(int rows) { return ((rows + 15) / 16 + kScoreWaves - 1) / kScoreWaves; }
template <typename T, int D, template <typename, int, int> class L>
static hipError_t dispatch_rbw(int rows, const CompressArgs& a, hipStream_t st) {
  switch (row_blocks_per_wave(rows)) {
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

}  // namespace sgdkv
