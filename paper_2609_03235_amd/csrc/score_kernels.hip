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
//   pass 2 (colsum_keys_kernel, and colsum_kernel in colsum_pass.h): for every scored key j < P0,
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
#include "colsum_pass.h"

namespace sgdkv {

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
constexpr int kKeyChunkMinFlat = 32768;  // with up to four of d 128 and no LSE given

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
// Whether pass 2 takes the keys in registers.
static bool colsum_by_keys(const CompressArgs& a) {
  // The keys a workgroup has make the difference: short chunks lose to the last turns' spread and
  // to filling the rows' LDS, the more rows the longer, and the more so where pass 1 has not left the
  // keys in the last-level cache (a given LSE). Whole call over inputs in turn, tiles / this: 128 rows at
  // 2048 keys 88.2 / 90.4 us, 4096 161.7 / 157.4, 8192 294 / 282; 256 rows at 2048 114.0 / 115.2, 4096 212 /
  // 204, 16384 741 / 694; 320 rows at 8192 444 / 426 (LSE given 259 / 250), 384 486 / 473 (275 / 275); 448
  // rows at 4096 279.5 / 280.3, 8192 531 / 529 (298 / 301), 16384 1035 / 1010 (580 / 564); 512 rows at 8192 582 /
  // 585 (325 / 330), 16384 1149 / 1128 (639 / 618). A chunk holds no more keys than its segment: 256 sequences
  // of 1024 keys, 256 rows, 312 / 332, 64 of 3072 161.7 / 157.9. Up to four row blocks of d 128 leave the pass to
  // the memory, which whole tiles read better, except in the longest chunks (64 rows at 4096 keys 138 / 145,
  // 8192 261 / 269, 16384 521 / 522, 65536 2017 / 2004; LSE given at 8192 241 / 243, 12288 369 / 365; d 64 at
  // 8192 166 / 155). Ipt. max loses to its reduction per
  // head (100K x 1: 98 / 102 for the pass).
  const int nrb = (a.rs_rows + 15) / 16;
  const int64_t keys = a.score_chunk < a.n_scored ? a.score_chunk : a.n_scored;
  if (a.dtype != 1 || a.agg == 1) return false;
  if (a.D == 128 && nrb <= 4) return keys >= (a.window_lse ? 3 * kKeyChunkMin : kKeyChunkMinFlat);
  return keys >= (nrb <= 16 ? kKeyChunkMin : nrb <= 24 ? 2 * kKeyChunkMin : 3 * kKeyChunkMin);
}

hipError_t launch_scores(const CompressArgs& a, hipStream_t st) {
  if (a.window_lse == nullptr) {
    const hipError_t e = launch_lse(a, st);
    if (e != hipSuccess) return e;
  }
  if (a.n_col_chunks == 0) return hipGetLastError();
  if (colsum_by_keys(a)) {
    const dim3 grid(a.n_col_chunks, a.B * a.Hkv, a.n_rsplit), blk(kScoreBlock);
    if (a.D == 128)
      SGDKV_LAUNCH("score_colsum", (colsum_keys_kernel<__bf16, 128>), grid, blk, st, a);
    else if (a.D == 64)
      SGDKV_LAUNCH("score_colsum", (colsum_keys_kernel<__bf16, 64>), grid, blk, st, a);
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  }
  const bool ilp = a.dtype == 1 && colsum_sched_ilp<__bf16>(a.D, row_blocks_per_wave(a.rs_rows), a.agg == 1);
  return ilp ? launch_colsum_ilp(a, st) : ColsumTiles<false>::launch(a, st);
}

}  // namespace sgdkv
