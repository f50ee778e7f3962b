// Rules by which a call's work is cut into workgroups.  Plain C++ without HIP, so that they can be compiled and checked on a
// host on their own.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

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

}  // namespace hyp
