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
  if (KT % g.nw != 0) g.nw = 4;
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

}  // namespace hyp
