// Rules by which a call's work is cut into workgroups.  Plain C++ without HIP, so that they can be compiled and checked on a
// host on their own.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "hyp_stage.h"

namespace hyp {

constexpr int kCus = 256;  // compute units of the chip

// tiles of 64 bytes that K elements of `esize` bytes take
constexpr int tiles_of_64_bytes(int K, int esize) { return (K * esize + 63) / 64; }

// ----------------------------------------------------------------------------
// Decode attention of generic stages: the workgroups that share the keys of a (request, group of heads).
// ----------------------------------------------------------------------------
constexpr int kPlainMaxSplit = 8;
constexpr size_t kPlainSplitGroups = 512;  // workgroups that a split may make of a decode step

// Waves of a workgroup.  Heads of more than 128 features fill the registers of one wave a SIMD.
constexpr int plain_attn_waves(int d) { return d > 128 ? 4 : 8; }

// pairs: (request, group of four query heads) of the step; longest: keys of the longest context.  A split is taken where the
// rounds of 16-key blocks that it saves its waves pay for the merging launch (5 us).  A round takes its MFMAs (two waves a SIMD,
// 2.4 GHz) and 0.5 us of softmax and latency; wide heads, whose waves wait for each block on their own, 1.5 us and the bytes at
// 64 B a clock and CU more (measured a round of 256 features: bf16 2.9 us, float 4.2; of 128: 0.9 and 1.2).  Workgroups beyond
// what the CUs hold at once - two each up to 64 features, else one - take turns.
// (A block of 4 requests, 500 keys, 256 features in bf16: 1, 2, 4, 8 shares 46.6, 38.1, 33.0, 28.5 us; of 32 requests, 700 keys:
// 60.0, 47.8, 41.1, 45.6.  Float, 128 features, 32 requests, 700 keys: 39.9, 41.0, 42.1, 45.1.)
inline int plain_attn_split(int esize, int d, size_t pairs, int longest) {
  const int nc = tiles_of_64_bytes(d, esize), nf = (d + 15) / 16, kw = plain_attn_waves(d), per_cu = d <= 64 ? 2 : 1;
  double round_us = (nc * (esize == 4 ? 4 : 1) + nf * 4) * 16.0 / 2400.0 + 0.5;
  if (d > 128) round_us += 1.5 + kw * (nc * 1024.0 + nf * 256.0 * esize) / (64.0 * 2400.0);
  const size_t blocks = (size_t)longest / 16 + 1, at_once = (size_t)kCus * per_cu;
  int split = 1;
  double best = 0.0;
  for (int c = 1; c == 1 || (c <= kPlainMaxSplit && pairs * c <= kPlainSplitGroups); c *= 2) {
    const double turns = (double)((pairs * c + at_once - 1) / at_once), rounds = (double)((blocks + kw * c - 1) / (kw * c));
    const double t = turns * rounds * round_us + (c > 1 ? 5.0 : 0.0);
    if (c == 1 || t < best) { best = t; split = c; }
  }
  return split;
}

// Parts of a head's value features that unsplit heads are dealt to, a workgroup each, where every workgroup then still has a CU of
// its own: four of 128 features, two of 64.  Other head sizes: one, since k_plain_dec_attn_parts is built for heads that fill its
// registers, not because those of 80 or 96 features would not gain.
inline int plain_attn_parts(int d, size_t pairs, int split) {
  const int parts = d == 128 ? 4 : d == 64 ? 2 : 1;
  return split == 1 && pairs * parts <= (size_t)kCus ? parts : 1;
}

// ----------------------------------------------------------------------------
// Prefill contractions of generic stages: the form.
// ----------------------------------------------------------------------------
enum { PLAIN_GEMM_REGISTERS = 0, PLAIN_GEMM_SMALL = 1, PLAIN_GEMM_WIDE = 2, PLAIN_GEMM_MANY = 3 };

// out^T[N, rows] = W[N, K] X[rows, K]^T in tiles of 32 x 32 from registers, or of 64 x 64 or 128 x 128 through LDS: microseconds
// by what was measured on 300 contractions of 256 - 5120 wide layers.  A tile costs so many nanoseconds per element of K, on every
// CU at once, and CUs with a tile more than the others are waited for (not so the small float tiles, whose waves fill in for
// each other); what comes before and behind the K loop is paid once.  (Float, 64 x 64: 320 x 584 tiles take as long as 512.)
// MANY: the wide bf16 tiles in four waves, three workgroups to a CU, where there are that many; residual epilogues, which
// those hide less of, only behind a long K loop (1280 tiles: K = 8960 even, K = 3200 7 % slower).
inline int plain_gemm_form(int esize, int rows, int N, int K, bool qkv, bool swiglu) {
  auto tiles = [&](int per) { return (double)((N + per - 1) / per) * ((rows + per - 1) / per); };
  auto rounds = [](double n) { return (double)(int64_t)((n + kCus - 1) / kCus); };
  const double n32 = tiles(32), n64 = tiles(64), n128 = tiles(128), k = K * 1e-3;
  double reg, small, wide;
  if (esize == 4) {
    reg = 4.0 + k * 6.5 * std::max(1.0, n32 / kCus);
    small = 5.0 + k * (n64 <= kCus ? 19.0 : 22.5 * rounds(n64));
    wide = 5.0 + k * 68.0 * rounds(n128);
  } else {
    reg = 3.5 + (qkv || swiglu ? 2.0 : 0.0) + k * 1.9 * rounds(n32);
    small = 6.5 + (qkv ? 1.5 : 0.0) + k * (n64 <= kCus ? 3.2 : 3.9 * rounds(n64));
    wide = 6.0 + (qkv ? 1.5 : 0.0) + k * (n128 <= kCus ? 10.0 : 7.8 * rounds(n128));
  }
  if (reg <= small && reg <= wide) return PLAIN_GEMM_REGISTERS;
  if (small <= wide) return PLAIN_GEMM_SMALL;
  return esize == 2 && n128 >= 3 * kCus && (qkv || swiglu || K >= 6144) ? PLAIN_GEMM_MANY : PLAIN_GEMM_WIDE;
}

// ----------------------------------------------------------------------------
// A decode step's kernels one by one, or a recorded HIP graph of them?  A replay takes the host 25 us + 1.5 us a block, launches
// 14 us a block; but a replay stands apart from what the stream runs before and behind it: one by one, one Phi-3 block takes 121 us
// instead of 126 (batch 8 at 2100 keys 143 instead of 147.5, a Llama3-8B block 88 / 92, a 512-wide one 20 / 25), eight Phi-3 blocks 1005 /
// 1009.  One by one where the host is then no slower, up to two blocks, or where it can't hold up the device: in stages of up to
// eight blocks whose weights take longer to stream than their launches (128 MiB at 6.6 TB/s: 20 us), however many stages
// a thread feeds on the GPU.  (Three stages on three streams fed by one thread, us for a step of each, one by one / replayed: 512 wide, one block 64 /
// 110, two 105 / 114, three 143 / 120, eight 417 / 194; 1024 wide, FFN 4096, two 105 / 112, three 143 / 122, eight 422 / 332.  Two Llama3-8B stages:
// three blocks 439 / 448, eight 1188 / 1192.)
// ----------------------------------------------------------------------------
inline bool decode_step_direct(int blocks, size_t block_weight_bytes) {
  return blocks <= 2 || (blocks <= 8 && block_weight_bytes >= ((size_t)128 << 20));
}

// ----------------------------------------------------------------------------
// How one skinny GEMM of a decode step is cut into workgroups.
//   fbw     32-row blocks per workgroup: 2 where the epilogue pairs rows of two blocks (gate and up) and
//           for long K; 1 for the residual GEMMs at short K, which then run as unsplit 4-wave
//           workgroups with a 10-tile window; QKV below
//   nw      waves per workgroup; they share the k-tiles of the workgroup's K slice.  8 for the
//           64-row workgroups: the same waves in flight with half the K slices of 4-wave workgroups
//   ksplit  K slices across workgroups (partial sums in memory, the last to arrive adds them up):
//           the fewest that put a wave on every slot of the chip (16 per CU), as long as a wave
//           keeps at least 20 k-tiles (four windows of the streaming loop) and the fp32 partial sums
//           (written and read once per slice and token) stay a few percent of the weight bytes.
//           Phi-3-medium shapes: gate/up unsplit (560 workgroups), down 7 slices;
//           measured against every other admissible cut of each GEMM at batch 8 and 32, this rule's
//           choices were the fastest or within 1 % of it.
struct GemvPlan { int fbw = 2, nw = 4, ksplit = 1, tail = 1; };  // tail: how many times finer the row groups of a thin second round are cut

constexpr int kWavesPerCu = 16;  // 4 per SIMD

inline GemvPlan mfma_gemv_plan(int cls, int N, int K, int batch) {
  GemvPlan g;
  const int KT = K / 16;
  // QKV: rotary partners lie in one block of 32 rows, and no slices: no partial sums, counter and gather (Phi-3, batch 1: 16.2 ->
  // 14.7 us).  One block to a workgroup while every workgroup has a CU of its own; beyond, two, which halves what is read of the
  // tokens (8192 x 12288, batch 1 / 32: 40.6 -> 35.7, 57.1 -> 45.2 us; 4096 x 12288: 22.7 -> 21.5, 31.9 -> 26.6) and costs time
  // where CUs would idle (5120 x 7168: 18.3 -> 21.6).  Eight waves share K beyond 5120 (8192 x 1536: 21.2 -> 18.7; 8192 x 6144:
  // 24.1 -> 21.9; 5120 x 7168 even), but not below (4096 x 6144: 14.4 -> 15.8).  Two slices of 64 rows would be 2 % of a block
  // faster for 6144 rows of K = 7168 and 8192 at batch 32 (and 4 - 6 % slower at batch 1 and 8).
  if (cls == HYP_K_GEMV_QKV) {
    g.fbw = N / 32 > kCus ? 2 : 1;
    g.nw = g.fbw == 2 || K > 5120 ? 8 : 4;
    g.ksplit = 1;
    return g;
  }
  if ((cls == HYP_K_GEMV_O || cls == HYP_K_GEMV_DOWN) && KT / 4 <= 112 && KT % 4 == 0) {
    g.fbw = 1; g.nw = 4; g.ksplit = 1;
    return g;
  }
  g.fbw = 2; g.nw = 8; g.ksplit = 1;
  const int groups = N / 64, wave_slots = kWavesPerCu * kCus;
  int cap = (int)(0.025 * K / (batch > 0 ? batch : 1));
  if (cap < 1) cap = 1;
  for (int ks = 1; ks <= 64 && ks <= cap; ++ks) {
    if (KT % (ks * g.nw) != 0 || KT / (ks * g.nw) < 20) continue;
    g.ksplit = ks;
    if (groups * ks * g.nw >= wave_slots) break;
  }
  // More workgroups than fit the chip at once, but fewer than two rounds: the groups beyond the first round
  // are cut finer, for what would otherwise be a thin second round of long workgroups.  A CU serves its waves'
  // loads oldest first, so the late workgroups stream last whatever their size: they should be many (bytes
  // in flight on every CU to the end) and short.  Four times finer where a wave keeps two windows of
  // the streaming loop (gate/up: 62.3 -> 59.6 us), else twice.
  const int units = groups * g.ksplit, slots = wave_slots / g.nw, tpw = KT / (g.ksplit * g.nw);
  if (units > slots && units < 2 * slots) {
    if (tpw % 4 == 0 && tpw / 4 >= 10) g.tail = 4;
    else if (tpw % 2 == 0 && tpw / 2 >= 10) g.tail = 2;
  }
  return g;
}

// k-tiles of a wave that are in flight at once.  One window: with all of a wave's tiles requested at the start, in registers that
// leave room for two or three waves a SIMD instead of four
constexpr int gemv_window(int fbw, bool one_window) { return one_window ? (fbw == 1 ? 16 : 10) : fbw == 1 ? 10 : 5; }

// One window, for unsplit GEMVs of at most that many tiles a wave whose workgroups all fit the chip at two waves a SIMD: eight-wave ones
// up to one a CU, four-wave ones up to two.  Beyond, they take a further round, or wait for registers.  (Steps of one block at batch 8, gate/up in one window
// / in several: 1024 wide, FFN 4096 = 128 workgroups 29.3 / 31.4 us, 8192 = 256 37.5 / 38.7, 8448 = 264 37.3 / 36.8, 16384 = 512
// 44.2 / 42.8; 1280 wide, FFN 28672 59.1 / 56.7.  QKV: the second of two blocks of 512 x 18432 = 288 workgroups 36.6 / 34.9, of
// 1280 x 24576 = 384 47.1 / 48.0, of 768 x 36864 = 576 45.4 / 45.0; the opening one there 47.5 / 46.5 and 45.8 / 44.7.)
inline bool mfma_gemv_one_window(const GemvPlan &g, int N, int K) {
  return g.ksplit == 1 && g.tail == 1 && K / 16 / g.nw <= gemv_window(g.fbw, true) && N / (32 * g.fbw) * g.nw <= 8 * kCus;
}

// Keys per chunk of decode attention (one wave each, at most two waves per SIMD): the largest power-of-two
// multiple of 128 up to 1024 that still gives the longest context about 512 waves over all
// (request, KV head) pairs - chunks of 256 for 8 x 10 pairs in room for 2K keys, 1024 for 8 x 10 pairs at 9K and for 32 x 10
// pairs from 1025 keys on, 512 up to there (asking for 768 or 1024 waves instead costs a step of one block at 4 x 10 pairs of
// 6K keys 146.6 -> 151.7 us, 16 x 8 of 3K 126.0 -> 128.7: fewer, longer waves win until a wave's own serial time shows) -
// doubled until a context has at most 64 chunks.  Between one wave and two per SIMD (1024 .. 2048 waves)
// some SIMDs would hold two and take longer than the others: `even` halves the chunk there (32 x 10 pairs in room for 3073 - 6144
// keys; ragged ones of 1K - 4K in pages: the attention 79.6 -> 69.7 us; within 1 % where the contexts are alike).
inline int mfma_decode_chunk_keys(int max_seq, int heads_in_flight, bool even) {
  int c = 1024;
  auto waves = [&] { return (long)heads_in_flight * ((max_seq + c - 1) / c); };
  while (c > 128 && waves() < 512) c /= 2;
  if (even && waves() > 1024 && waves() < 2048) c /= 2;
  while ((max_seq + c - 1) / c > 64) c *= 2;
  return c;
}

// ----------------------------------------------------------------------------
// Prefill GEMMs: the form, and the slices of the K loop.
// ----------------------------------------------------------------------------
struct GemmShape { int tok_blocks, feat_blocks, lds_stages; };  // 32-row blocks of tokens and features of a tile, stages in LDS
constexpr GemmShape kGemmWide = {8, 8, 4}, kGemm64 = {2, 4, 6}, kGemm128 = {4, 4, 4};
constexpr int kGemmStageTiles = 2;     // k-tiles of 16 in a stage
constexpr int kGemmSplitUnits = 512;   // most (tile, slice) pairs of a split GEMM
constexpr int kGemmShortMaxTiles = 511;  // short forms: tiles that may be split, and counters
// Wide GEMMs of two and a half rounds of 256 tiles or more are never split: a request that fills them alone then has the same
// bits in any batch, and what splitting the last, partial round saves falls with the number of rounds (Phi-3 block: gate/up 210
// -> 155 us at 384 rows = 280 tiles, 325 -> 292 at 1024 = 560).
constexpr int kGemmSplitMaxTiles = 639;

struct GemmCut {
  int form;               // tokens of a tile: 64, 128, 256
  int tiles_t, n_tiles;   // token tiles, tiles
  // tiles from `first` on have their K loop split over `ksplit` workgroups each; finish: a second kernel adds the slices up
  int first, ksplit;
  bool finish;
  int n_static, pool_wgs;     // many rounds: tiles assigned by position, workgroups that draw the rest
  int first_grid, rest_grid;  // workgroups of unsplit tiles, of slices
};

// A K loop in slices costs their partial tiles, written and read at 5 TB/s together, and the launch that adds them up.
inline double gemm_slice_us(int tiles, int c, int tok_blocks, int feat_blocks) {
  return c == 1 ? 0.0 : (double)tiles * c * tok_blocks * feat_blocks * 4096.0 / 2.5e6 + 5.0;
}

// Tiles of 128 features x 64 tokens, several of them along the tokens, their K loop in c slices: a stage takes 0.235 us while every
// workgroup has a CU of its own and 0.325 with two to a CU, which is all that fit; a further round takes 2.5 us to begin and end.
// Slices cost the second launch (1.5 us more with two to a CU), their partial tiles, most of which stay in the caches (10 TB/s
// written and read), and a second round trip of the sums beyond eight.
inline double gemm64_us(int tiles, int stages, int c) {
  const int units = tiles * c, rounds = units / (2 * kCus), rest = units % (2 * kCus);
  const double stage_us = rounds * 0.325 + (rest == 0 ? 0.0 : rest <= kCus ? 0.235 : 0.325);
  double us = 7.8 + 2.5 * (rounds - (rest == 0)) + (stages + c - 1) / c * stage_us;
  if (c > 1) us += 3.0 + (units > kCus ? 1.5 : 0.0) + units * (double)(kGemm64.tok_blocks * kGemm64.feat_blocks) * 4096.0 / 5.0e6 + (c > 8 ? 1.0 : 0.0);
  return us;
}
inline int gemm64_split(int tiles, int stages) {
  int split = 1;
  double best = 0.97 * gemm64_us(tiles, stages, 1);  // a split has to win clearly
  for (int c = 2; c <= 32 && tiles * c <= kGemmSplitUnits && stages / c >= 2 * kGemm64.lds_stages; ++c) {
    const double t = gemm64_us(tiles, stages, c);
    if (t < best) { best = t; split = c; }
  }
  return split;
}

// rows % 32 == 0, N % 256 == 0, K % 32 == 0; swiglu: the gate/up GEMM, whose epilogue stores half as much and reads nothing
inline GemmCut mfma_gemm_cut(int rows, int N, int K, bool swiglu) {
  const int tok_blocks = rows / 32, feat_blocks = N / 32, stages = K / 16 / kGemmStageTiles;
  GemmCut g = {};
  // The wide form: whole rounds of one tile per CU, then the rest, in as many rounds as its slices take.  Slices are whole
  // numbers of stages, at least two rounds through the LDS buffers.
  const GemmShape wide = kGemmWide;
  const int wide_tiles = (tok_blocks + wide.tok_blocks - 1) / wide.tok_blocks * (feat_blocks / wide.feat_blocks), wide_rest = wide_tiles % kCus;
  const double tile_us = K * 0.020, start_us = 4.0;  // a 256 x 256 tile on one CU, whatever the others do (K = 5120: 105 us)
  int wide_split = 1;
  if (wide_tiles <= kGemmSplitMaxTiles) {
    double best = 0.95 * (tile_us + start_us);  // a split has to win clearly
    for (int c = 2; c <= 32 && wide_rest * c <= kGemmSplitUnits && wide_rest > 0 && stages / c >= 2 * wide.lds_stages; ++c) {
      const int rounds = (wide_rest * c + kCus - 1) / kCus;
      const double t = rounds * (tile_us / c + start_us) + gemm_slice_us(wide_rest, c, std::min(tok_blocks, wide.tok_blocks), wide.feat_blocks);
      if (t < best) { best = t; wide_split = c; }
    }
  }
  // Which form?  Up to 128 tokens the weights' streaming time counts, not the products (see GemmForm): one token tile.  Beyond, a
  // GEMM of few tiles is bound by the latency of a stage and by its epilogue, and takes tiles of 128 features x 64 tokens where
  // those, in slices or not, come out ahead of the wide form, whose unsplit tiles end in a long epilogue at one workgroup a CU
  // and whose partial tiles stay in the caches, too (12 TB/s).  (512 wide, 553 rows: QKV 26.7 -> 12.3 us, gate/up 18.8 -> 10.9;
  // 2048 x 2048, 200 rows: O 20.7 -> 16.6 in 4 slices.  576 tiles of gate/up, K = 2048: 47.2 against 42.7 in the wide form.  Of
  // 484 GEMMs of 256 - 5120 wide layers and 160 - 3500 rows this picks one that is more than 3 % from the better form.)
  g.form = 256;
  const int tiles64 = (tok_blocks + kGemm64.tok_blocks - 1) / kGemm64.tok_blocks * (feat_blocks / kGemm64.feat_blocks), split64 = gemm64_split(tiles64, stages);
  if (tok_blocks <= kGemm128.tok_blocks) {
    g.form = tok_blocks <= kGemm64.tok_blocks || 2.0 * N * K <= 16e6 ? 64 : 128;
  } else {
    const int rest_rounds = (wide_rest * wide_split + kCus - 1) / kCus;
    double wide_us = wide_split > 1 && wide_rest == wide_tiles ? 4.0 : swiglu ? 2.0 : 9.0;  // the epilogue
    wide_us += wide_tiles / kCus * (tile_us + start_us) + rest_rounds * (tile_us / wide_split + start_us);
    if (wide_split > 1) wide_us += 5.0 + (double)wide_rest * wide_split * std::min(tok_blocks, wide.tok_blocks) * wide.feat_blocks * 4096.0 / 6.0e6;
    if (gemm64_us(tiles64, stages, split64) < 0.95 * wide_us) g.form = 64;
  }
  const GemmShape shape = g.form == 64 ? kGemm64 : g.form == 128 ? kGemm128 : wide;
  g.tiles_t = (tok_blocks + shape.tok_blocks - 1) / shape.tok_blocks;
  g.n_tiles = g.tiles_t * (feat_blocks / shape.feat_blocks);
  g.first = g.n_tiles; g.ksplit = 1; g.finish = true;
  if (g.form < 256) {
    if (g.tiles_t > 1) {
      g.ksplit = split64;
      if (split64 > 1) g.first = 0;
    } else if (g.n_tiles <= kGemmShortMaxTiles) {
      // One token tile, few tiles: the chip streams as much as its workgroups keep in flight over 1.5 us of latency, 6 TB/s at best,
      // and a CU with one workgroup more than the others is waited for.  (64 rows, slices 10 -> 5: down 51 -> 43 us, O 25 ->
      // 21; QKV 8 -> 4: 30 -> 26.)
      const double in_flight = (shape.lds_stages - 1) * (double)shape.feat_blocks * kGemmStageTiles * 1024, bytes = 2.0 * N * K;
      double best = 1e30;
      for (int c = 1; c == 1 || (c <= 32 && g.n_tiles * c <= kGemmSplitUnits); ++c) {
        if (c > 1 && stages / c < 2 * shape.lds_stages) continue;
        const int units = g.n_tiles * c, per_cu = (units + kCus - 1) / kCus;
        const double even = units <= kCus ? 1.0 : units / ((double)per_cu * kCus);
        const double t = bytes / (std::min(6.0e6, units * in_flight / 1.5) * even) + gemm_slice_us(g.n_tiles, c, tok_blocks, shape.feat_blocks);
        if (t < best) { best = t; g.ksplit = c; g.first = c > 1 ? 0 : g.n_tiles; }
      }
      // More tiles than CUs, unsplit: the ones beyond the first 256 (24 of gate/up's 280) would double a few CUs' work.
      // They are split so that they spread over all CUs beside the others, and added up there.
      const int rest = g.n_tiles - kCus;
      if (g.ksplit == 1 && rest > 0)
        for (int c = 16; c >= 2; --c)
          if (stages / c >= 2 * shape.lds_stages && rest * c <= kCus) {
            g.first = kCus; g.ksplit = c; g.finish = false;
            break;
          }
    }
  } else if (wide_split > 1) {
    g.ksplit = wide_split; g.first = g.n_tiles - wide_rest;
  }
  g.first_grid = (g.first + 7) / 8 * 8;
  g.rest_grid = ((g.n_tiles - g.first) * g.ksplit + 7) / 8 * 8;
  // 64 rounds of 256 tiles or more: the last sixteenth of the rounds is drawn from a counter by twice as many
  // workgroups as it has tiles, so that an XCD can take up to a quarter of it.  (Gate/up at 64 K tokens, 140 rounds:
  // 2.3 % faster.  With 20 - 30 rounds the drawn tiles' lost L2 neighbourhood and the tile granularity cost more than
  // the balance brings: down projection 1.7 % slower.)
  if (g.form == 256 && g.n_tiles >= 64 * kCus) {
    const int rounds = g.n_tiles / kCus, pool_rounds = (rounds + 8) / 16;
    g.first = g.n_tiles; g.ksplit = 1; g.rest_grid = 0;
    g.n_static = (rounds - pool_rounds) * kCus;
    g.pool_wgs = (2 * (g.n_tiles - g.n_static) + 7) / 8 * 8;
    g.first_grid = g.n_static + g.pool_wgs;
  }
  return g;
}

}  // namespace hyp
