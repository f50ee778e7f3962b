// Attention kernels of the MFMA path: causal grouped-query attention over the
// prompt (flash-style: the score matrix is never written), and split-KV
// attention of one new token per request against the cache (bandwidth-bound).
// Both follow the GQA-with-RoPE sub-layer of Sec. III-A; RoPE was already
// applied to q and to the cached keys by the QKV epilogue.
#include <type_traits>
#include "mfma_common.h"
#include "mfma_kernels.h"

namespace hyp {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

// The two halves of a wave exchanged in the vector ALU (v_permlane32_swap: lanes 32..63 of its first operand
// trade places with lanes 0..31 of its second), not through the LDS crossbar and its wait: with both operands v
// the first result holds v's lower half in both halves, the second its upper half.
struct HalfPair { float lo, hi; };
__device__ __forceinline__ HalfPair both_halves(float v) {
  const unsigned u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float xhalf_max(float v) { const HalfPair h = both_halves(v); return fmaxf(h.lo, h.hi); }
__device__ __forceinline__ float xhalf_sum(float v) { const HalfPair h = both_halves(v); return h.lo + h.hi; }

__device__ __forceinline__ bf16x8_t probs_operand(const float *p /*16*/, int m) {
  // MFMA step m of the P V product contracts keys 16m + 8(e/4) + 4hh + e%4: registers 8m .. 8m+7
  bf16x8_t r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (__bf16)p[8 * m + e];
  return r;
}

// ----------------------------------------------------------------------------
// Prefill.  One workgroup = one KV head x one tile of 64 query rows.  It has two
// waves per query head of the group (32 query rows each), so a K / V stage of 64
// keys (32 KiB, already in fragment order) is fetched once into LDS by direct
// loads and read by all 2G waves.  Per wave: S^T = K Q^T (keys on the MFMA M axis,
// so a lane owns one query column and the softmax reductions stay inside a lane
// plus one cross-half exchange), online softmax in fp32, O^T += V^T P^T.
//
// The loop is software-pipelined over stages: the scores of stage s + 1 are
// formed (MFMA) in the same straight-line block in which the probabilities of
// stage s are exponentiated, summed and rounded (VALU), so the matrix pipe works
// under the softmax arithmetic, which is the longer of the two; three LDS buffers
// keep stage s (values), s + 1 (keys, then values) and s + 2 (arriving) apart.
// The running maximum is only moved - and the accumulators rescaled - when it has
// grown by more than 2^8 in some row: probabilities stay below 256, sums and
// outputs are formed against the same reference, and the rescale leaves the loop's
// steady state.  Only the last stage of a tile touches the diagonal and is masked.
// ----------------------------------------------------------------------------
constexpr int kKvStageKeys = 64;
constexpr int kKvStageBytes = 2 * 16384;  // per 32 keys: 8 K tiles + 8 V tiles
constexpr int kKvBufs = 3;
constexpr int kAttnPrefillLds = kKvBufs * kKvStageBytes;
constexpr float kRescaleLog2 = 8.0f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// max of three: one v_max3_f32, because this file is compiled with -fno-honor-nans (scores are never
// NaN; otherwise the compiler puts a canonicalising self-maximum in front of every fmaxf operand).
// Not inline assembly: the compiler's hazard logic must see that the operands come out of MFMAs.
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

template <int G>
__global__ void __launch_bounds__(128 * G) k_attn_prefill(const bf16_t *__restrict__ q,
                                                      const bf16_t *__restrict__ Kc,
                                                      bf16_t *Vc, CacheGeom geom,
                                                      bf16_t *__restrict__ out,
                                                      const PrefillTile *__restrict__ tiles,
                                                      const int *__restrict__ req_len, int nq) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  // wave-uniform values in scalar registers: the LDS destination of a direct load has to be uniform, and a wave index
  // the compiler takes for divergent turns every such load into a loop over lanes
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, hh = lane >> 5, tl = lane & 31;
  constexpr int nw = 2 * G;  // waves per workgroup
  const PrefillTile tile = tiles[blockIdx.x];
  const int kvh = blockIdx.y;
  const int head = kvh * G + (wave >> 1);
  const int tq = wave & 1;                 // which 32-row block of the tile
  const int qblk = tile.qblk0 + tq;        // its index inside the request
  const int qd = nq * 128;
  const int len = req_len[tile.req];
  const int n_kb = min(tile.qblk0 + 2, (len + 31) >> 5);  // 32-key blocks the tile needs
  const int n_st = (n_kb + 1) >> 1;                        // 64-key stages; every wave of the tile needs all of them
  const int rb = (tile.row0 >> 5) + tq;
  const int orow = tile.out0 + tq * 32 + tl;  // row of out
  const float c = kLog2e * 0.08838834764831845f;  // log2(e) / sqrt(128)
  const int qpos = qblk * 32 + tl;

  bf16x8_t qf[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
    qf[dt] = *(const bf16x8_t *)(q + ((size_t)rb * (qd >> 4) + head * 8 + dt) * kTileElems + lane * 8);
  // rows of q behind the request hold whatever an earlier call left: they count as zero (a wave moves its maxima together)
  if (qpos >= len) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[dt][e] = (__bf16)0.f;
  }

  f32x16_t o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // A stage is the pair of key blocks 2 st, 2 st + 1: 16 KiB contiguous in either cache layout
  // (the block count of a request is even and a page holds four blocks).  Its offset is uniform
  // over the workgroup and, with a paged cache, costs a table lookup: it is formed one stage
  // before the loads that use it are issued.
  auto stage_off = [&](int st) { return geom.off(tile.req, kvh, min(st * 2, geom.key_blocks - 2)); };
  auto issue = [&](size_t off, int buf) {
    // 32 tiles of 1 KiB: [key block 0: 8 K, 8 V][key block 1: 8 K, 8 V]; the second
    // block of the last stage may lie past the tile's need but is inside the cache
    // wave w fetches tiles w, w + nw, ...; with 2, 4 or 8 waves everything about a tile but w itself is known at
    // compile time, and the loop unrolls into straight scalar address arithmetic
    if constexpr (nw == 2 || nw == 4 || nw == 8) {
      constexpr int per8 = 8 / nw;
#pragma unroll
      for (int j = 0; j < 32 / nw; ++j) {
        const int hi = j / per8, lo = nw * (j % per8);  // tile t = 8 hi + lo + wave
        const bf16_t *src = ((hi & 1) ? Vc : Kc) + off + (size_t)(hi >> 1) * (32 * 128) + (size_t)(lo + wave) * kTileElems + lane * 8;
        __builtin_amdgcn_global_load_lds((gbl_ptr_t *)src, (lds_ptr_t *)(lds + buf * kKvStageBytes + (8 * hi + lo + wave) * 1024), 16, 0, 0);
      }
    } else {
      for (int t = wave; t < 32; t += nw) {
        const bf16_t *src = ((t & 8) ? Vc : Kc) + off + (size_t)(t >> 4) * (32 * 128) + (size_t)(t & 7) * kTileElems + lane * 8;
        __builtin_amdgcn_global_load_lds((gbl_ptr_t *)src, (lds_ptr_t *)(lds + buf * kKvStageBytes + t * 1024), 16, 0, 0);
      }
    }
  };
  // scores of both 32-key blocks of the stage in `buf`: two independent accumulator chains
  auto scores = [&](int buf, f32x16_t &a0, f32x16_t &a1) {
    const char *base = lds + buf * kKvStageBytes + lane * 16;
#pragma unroll
    for (int r = 0; r < 16; ++r) { a0[r] = 0.f; a1[r] = 0.f; }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      bf16x8_t k0 = *(const bf16x8_t *)(base + dt * 1024);
      bf16x8_t k1 = *(const bf16x8_t *)(base + 16384 + dt * 1024);
      a0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0, qf[dt], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1, qf[dt], a1, 0, 0, 0);
    }
  };
  // move the running maximum when some row's has grown by more than 2^kRescaleLog2 (always on the
  // first stage, where the old maximum is -inf and the factor 0)
  auto follow_max = [&](float mx) {
    float m_new = fmaxf(m_run, xhalf_max(mx));  // finite from the first stage on: key 0 is visible to every row
    if (__any((m_new - m_run) * c > kRescaleLog2)) {
      float alpha = fast_exp2((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      m_run = m_new;
    }
  };
  // O^T += V^T P^T for the stage in `buf`
  // (the last stage's; key slots from `end` on, counted from the stage, hold anything and count as zero)
  auto values = [&](int buf, const bf16x8_t *pf, int end) {
    const char *base = lds + buf * kKvStageBytes + lane * 16;
#pragma unroll
    for (int h2 = 0; h2 < 4; ++h2)   // (key block, MFMA step) pairs
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        bf16x8_t vf = *(const bf16x8_t *)(base + (h2 >> 1) * 16384 + (8 + (h2 & 1) * 4 + db) * 1024);
        if (end < kKvStageKeys) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (h2 * 16 + 8 * (e >> 2) + 4 * hh + (e & 3) >= end) vf[e] = (__bf16)0.f;
        }
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[h2], o[db], 0, 0, 0);
      }
  };

  issue(stage_off(0), 0);
  if (n_st > 1) issue(stage_off(1), 1);
  size_t off_next = stage_off(2);
  __builtin_amdgcn_s_waitcnt(0x0070);  // my loads of the first two stages have landed
  __syncthreads();
  f32x16_t s0, s1;
  scores(0, s0, s1);
  float mx = max3(s0[0], s1[0], -INFINITY);
#pragma unroll
  for (int r = 1; r < 16; ++r) mx = max3(mx, s0[r], s1[r]);

  // A wave issues in order: an MFMA that finds the matrix pipe still busy with the previous one
  // holds up the arithmetic behind it.  So each iteration is laid out as two phases in which
  // every MFMA (32 cycles) is followed by about as many cycles of independent VALU work:
  //   phase 1   scores of stage st + 1 (16 MFMAs)  |  exponentials and rounding of stage st
  //   phase 2   P V of stage st (16 MFMAs)         |  row sums of stage st, maxima of stage st + 1
  // The scheduling-group builtins fix that interleaving; left alone the compiler bunches the MFMAs.
  bf16x8_t pf[4];
  int buf = 0;  // buffer of stage st
  // one stage of the loop: consumes the scores c0, c1 of stage st, leaves those of stage st + 1 in n0, n1
  auto stage = [&](int st, const f32x16_t &c0, const f32x16_t &c1, f32x16_t &n0, f32x16_t &n1) {
    const int buf1 = buf + 1 == kKvBufs ? 0 : buf + 1, buf2 = buf1 + 1 == kKvBufs ? 0 : buf1 + 1;
    if (st + 2 < n_st) issue(off_next, buf2);  // over stage st - 1, which every wave has left
    // Fragments come from LDS in batches of four, each batch requested one group of four MFMAs ahead
    // (while LDS-direct loads are in flight the compiler only emits full LDS waits, so a batch is
    // awaited as a whole, long after it was requested).
    const char *kbase = lds + buf1 * kKvStageBytes + lane * 16;
    const char *vbase = lds + buf * kKvStageBytes + lane * 16 + 8 * 1024;
    auto kfrag = [&](int i) { return *(const bf16x8_t *)(kbase + (i & 1) * 16384 + (i >> 1) * 1024); };  // i = 2 dt + key block
    auto vfrag = [&](int i) { return *(const bf16x8_t *)(vbase + (i >> 3) * 16384 + (i & 7) * 1024); };  // i = 8 key block + 4 step + d block
    bf16x8_t fr[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) fr[0][u] = kfrag(u);
    __builtin_amdgcn_sched_barrier(0);
    follow_max(mx);
    const float mc = m_run * c;
    // ---- phase 1: scores of stage st + 1 | probabilities of stage st
#pragma unroll
    for (int r = 0; r < 16; ++r) { n0[r] = 0.f; n1[r] = 0.f; }
    float p[32];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int g = i >> 2, u = i & 3;
      if (i & 1) n1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g & 1][u], qf[i >> 1], n1, 0, 0, 0);
      else n0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g & 1][u], qf[i >> 1], n0, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (u == 0) {  // the next batch: keys of the next group, or the first values of phase 2
#pragma unroll
        for (int w = 0; w < 4; ++w) fr[(g + 1) & 1][w] = g < 3 ? kfrag(4 * (g + 1) + w) : vfrag(w);
      }
      // two probabilities and their rounding per MFMA: registers 2 i and 2 i + 1 of the 32 scores
      {
        const int r0 = 2 * i, r1 = 2 * i + 1;
        p[r0] = fast_exp2((r0 < 16 ? c0[r0] : c1[r0 - 16]) * c - mc);
        p[r1] = fast_exp2((r1 < 16 ? c0[r1] : c1[r1 - 16]) * c - mc);
        pf[r0 >> 3][r0 & 7] = (__bf16)p[r0];
        pf[r0 >> 3][r1 & 7] = (__bf16)p[r1];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- phase 2: P V of stage st | row sums of stage st, maxima of stage st + 1
    float rowsum = 0.f;
    mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int g = i >> 2, u = i & 3;
      o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g & 1][u], pf[i >> 2], o[i & 3], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (u == 0 && g < 3) {
#pragma unroll
        for (int w = 0; w < 4; ++w) fr[(g + 1) & 1][w] = vfrag(4 * (g + 1) + w);
      }
      rowsum += p[2 * i];
      rowsum += p[2 * i + 1];
      mx = max3(mx, n0[i], n1[i]);
      // an empty statement that "uses" both: without it the two chains are sunk as a whole below the loop's last
      // MFMA (they are only needed there), and the matrix pipe runs phase 2 alone
      asm volatile("" : "+v"(rowsum), "+v"(mx));
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run += rowsum;
    buf = buf1;
    // a paged cache answers this with a scalar load; issued here, it completes under the wait below -
    // outstanding during the phases it would turn every LDS wait into a full one
    off_next = stage_off(st + 3);
    __builtin_amdgcn_s_waitcnt(0x0070);  // my loads of stage st + 2 landed, my LDS reads of stage st done
    __syncthreads();
  };
  // two stages per trip with the roles of the two accumulator pairs swapped, so that no stage ends by copying
  // the next scores into the current ones; an odd stage count starts with a single stage (one copy per tile)
  {
    f32x16_t t0, t1;
    int st = 0;
    if ((n_st - 1) & 1) {
      stage(0, s0, s1, t0, t1);
      s0 = t0; s1 = t1;
      st = 1;
    }
    for (; st + 1 < n_st; st += 2) {
      stage(st, s0, s1, t0, t1);
      stage(st + 1, t0, t1, s0, s1);
    }
  }
  // last stage: the only one that touches the diagonal (a block past the tile's need is fully
  // masked here: its keys lie after every row)
  {
    const int kb0 = (n_st - 1) * 2, qlast = min(qpos, len - 1);
    float p[32];
    mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      int koff = 8 * (r >> 2) + 4 * hh + (r & 3);
      p[r] = (kb0 * 32 + koff > qlast) ? -INFINITY : s0[r];
      p[16 + r] = (kb0 * 32 + 32 + koff > qlast) ? -INFINITY : s1[r];
      mx = fmaxf(mx, fmaxf(p[r], p[16 + r]));
    }
    follow_max(mx);
    const float mc = m_run * c;
    float rowsum = 0.f;
#pragma unroll
    for (int r = 0; r < 32; ++r) {
      p[r] = fast_exp2(p[r] * c - mc);
      rowsum += p[r];
    }
    l_run += rowsum;
    pf[0] = probs_operand(p, 0); pf[1] = probs_operand(p, 1); pf[2] = probs_operand(p + 16, 0); pf[3] = probs_operand(p + 16, 1);
    values(buf, pf, len - kb0 * 32);
  }

  // normalise and store into P(rows, qd): lane owns query tl, features 8g + 4hh + e of each d block
  float inv = 1.0f / xhalf_sum(l_run);
  if (qpos < len) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int f0 = head * 128 + db * 32;
        size_t off = ((size_t)(orow >> 5) * (qd >> 4) + ((f0 + 8 * g) >> 4)) * kTileElems + (((g & 1) << 5) + (orow & 31)) * 8 + hh * 4;
        *(bf16x4_t *)(out + off) = pack4(o[db][4 * g] * inv, o[db][4 * g + 1] * inv, o[db][4 * g + 2] * inv,
                                         o[db][4 * g + 3] * inv);
      }
  }
  // Decode steps multiply the slots behind the last key by probabilities of zero: the tile that ends the request clears
  // them up to a multiple of 64 keys (no other workgroup reads that stage, and this one masks it above).
  if ((tile.qblk0 + 2) * 32 >= len) {
    const int pad = (-len) & 63;
    for (int i = threadIdx.x; i < pad * 128; i += 128 * G) {
      const int key = len + (i >> 7), d = i & 127;
      int m, khh;
      const int e = vtile_slot_of_key(key & 31, &m, &khh);
      Vc[geom.off(tile.req, kvh, key >> 5) + (size_t)(m * 4 + (d >> 5)) * kTileElems + (khh * 32 + (d & 31)) * 8 + e] = 0;
    }
  }
}

// ----------------------------------------------------------------------------
// Decode.  The query buffer holds, per (request, KV head), the G query heads as
// rows 0..G-1 of a P(32, 128) block (other rows zero), so the same MFMA shape
// serves: S^T[key, head] = K q^T.  K and V fragments go straight from HBM into
// registers (fragment order = operand order), 16 wave loads of 1 KiB per 32-key
// block, no LDS.  One wave owns a chunk of chunk_keys keys of one
// (request, KV head).  Every chunk
// writes (max, sum, unnormalised output) and a second small kernel merges the
// chunks of a head in index order, so the result does not depend on scheduling.
// part layout: [request][head][chunk][130] = {m, l, o[128]}
// ----------------------------------------------------------------------------
constexpr int kPartStride = 130;

struct DecodeAcc {
  f32x16_t o[4];
  float m, l;  // running maximum; sum of this lane's half of the keys
};
__device__ __forceinline__ void decode_clear(DecodeAcc &a) {
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) a.o[db][r] = 0.f;
  a.m = -INFINITY;
  a.l = 0.f;
}
__device__ __forceinline__ void decode_load(const bf16_t *cache, size_t off, bf16x8_t (&f)[8]) {
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = __builtin_nontemporal_load((const bf16x8_t *)(cache + off + t * kTileElems));
}
__device__ __forceinline__ void decode_load(const bf16_t *Kc, const bf16_t *Vc, size_t off, bf16x8_t (&kf)[8], bf16x8_t (&vf)[8]) {
  decode_load(Kc, off, kf);
  decode_load(Vc, off, vf);
}
// fragments of a block, in registers or fetched as they are used (read ahead they would cost every launch registers, and
// half its waves)
struct RegFrags {
  const bf16x8_t *f;
  __device__ __forceinline__ const bf16x8_t &operator()(int t) const { return f[t]; }
};
struct MemFrags {
  const bf16_t *p;
  __device__ __forceinline__ bf16x8_t operator()(int t) const {
    __builtin_amdgcn_sched_barrier(0);
    return *(const bf16x8_t *)(p + t * kTileElems);
  }
};
// one block of 32 keys, the first `nkeys` of the request visible; at least one of the block's is.  What is there already
// is rescaled when some maximum of the wave has moved, always, or - the first block - never: the same bits, an unmoved
// maximum's factor is 1.
enum { RESCALE_MOVED, RESCALE_ALWAYS, RESCALE_NEVER };
// q(dt), k(dt), v(4 step + d block): the fragments; keys_read(), values_read(): called once those of k and v are no longer needed.
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <int RESCALE, typename Q, typename K, typename V, typename KeysRead = Nothing, typename ValuesRead = Nothing>
__device__ __forceinline__ void decode_block(DecodeAcc &a, int kb, int nkeys, int hh, Q q, K k, V v,
                                             KeysRead keys_read = KeysRead(), ValuesRead values_read = ValuesRead()) {
  const float c = kLog2e * 0.08838834764831845f;
  f32x16_t s;
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k(dt), q(dt), s, 0, 0, 0);
  keys_read();
  float p[16];
  float mx = -INFINITY;
  if ((kb + 1) * 32 > nkeys) {  // only the last block of a request can hold keys past the end
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      int kpos = kb * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
      p[r] = kpos < nkeys ? s[r] : -INFINITY;
      mx = fmaxf(mx, p[r]);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = s[r];
      mx = fmaxf(mx, p[r]);
    }
  }
  mx = xhalf_max(mx);
  float m_new = fmaxf(a.m, mx);  // finite: the first key of a block is visible
  float mc = m_new * c, rowsum = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    p[r] = fast_exp2(p[r] * c - mc);
    rowsum += p[r];
  }
  if (RESCALE == RESCALE_ALWAYS || (RESCALE == RESCALE_MOVED && __any(m_new > a.m))) {
    float alpha = fast_exp2((a.m - m_new) * c);  // 0 on the first block
    a.l *= alpha;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) a.o[db][r] *= alpha;
    a.m = m_new;
  }
  if (RESCALE == RESCALE_NEVER) a.m = m_new;
  {
#pragma clang fp contract(off)
    a.l += rowsum;
  }
  bf16x8_t pf0 = probs_operand(p, 0), pf1 = probs_operand(p, 1);
#pragma unroll
  for (int db = 0; db < 4; ++db) {
    a.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v(db), pf0, a.o[db], 0, 0, 0);
    a.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v(4 + db), pf1, a.o[db], 0, 0, 0);
  }
  values_read();
}

// A batch whose contexts are all short runs another form (k_attn_decode_short).  The host chooses by the lengths it knows;
// in a step that the caller records, the kernels choose by the lengths they find.
// A wave looks at all of them: lane b holds the length of request b.
__device__ __forceinline__ int batch_len(const int *lens, int batch, int lane) { return lane < batch ? lens[lane] : 0; }  // batch <= 32
__device__ __forceinline__ bool all_short(int batch_len) { return !__any(batch_len + 1 > kShortKeys); }
// the operations of a merge, spelled out so that every kernel that merges rounds alike
__device__ __forceinline__ float merge_sum(float sum, float w, float l) {
#pragma clang fp contract(off)
  return sum + w * l;
}
__device__ __forceinline__ float merge_out(float acc, float w, float o) { return fmaf(w, o, acc); }

// A wave streams its chunk through one register set of keys and one of values: the next block's keys are requested as soon as
// the scores are formed, its values behind P V.  That is 192 registers and two waves per SIMD, which wait in turn; two sets of
// each left room for one.  The pairs are the fastest dimension of the grid: workgroup i runs on XCD i % 8, and with the chunks
// fastest the few that a short context has fell on the same XCDs (4 or 8 chunks of which 1 is there: on two or one of the eight).
// Together, traced: 8 x 10 pairs of 8200 keys in room for 9216 53.8 -> 52.4 us (6.4 TB/s), in room for 8256 55.2 -> 55.5; 32 x 8 of 1000
// 31.5 -> 26.2; 32 x 10 ragged of 1K - 4K in pages 71.9 -> 70.2 (5.8 TB/s); 32 x 10 of 1000 in room for 4000 81.7 -> 29.0.
// The last block stands behind the loop: no load sits under a condition between two uses, which would make the compiler wait
// for everything.
template <bool RECORDED>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_attn_decode(const bf16_t *__restrict__ qdec, const bf16_t *__restrict__ Kc, const bf16_t *__restrict__ Vc, CacheGeom geom,
              const int *__restrict__ lens, float *__restrict__ part, int nq, int G, int max_chunks, int chunk_keys) {
  const int lane = threadIdx.x, hh = lane >> 5, tl = lane & 31;
  const int kvh = blockIdx.x, req = blockIdx.y, chunk = blockIdx.z;
  int len;
  if (RECORDED) {
    const int mine = batch_len(lens, gridDim.y, lane);
    if (all_short(mine)) return;
    len = __builtin_amdgcn_readlane(mine, req);
  } else {
    len = lens[req];
  }
  const int nkeys = len + 1;  // the new token's key is already in the cache
  const int k0 = chunk * chunk_keys;
  if (k0 >= nkeys) return;
  const int kb_begin = k0 >> 5;
  const int kb_end = min((k0 + chunk_keys) >> 5, (nkeys + 31) >> 5);

  bf16x8_t qf[8];
  const bf16_t *qb = qdec + ((size_t)req * geom.nkv + kvh) * (32 * 128);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) qf[dt] = *(const bf16x8_t *)(qb + dt * kTileElems + lane * 8);

  DecodeAcc acc;
  decode_clear(acc);
  bf16x8_t kf[8], vf[8];
  auto place = [&](int kb) { return geom.off(req, kvh, min(kb, kb_end - 1)) + lane * 8; };
  auto load = [](const bf16_t *cache, size_t at, bf16x8_t (&f)[8]) {
    __builtin_amdgcn_sched_barrier(0);
    decode_load(cache, at, f);
    __builtin_amdgcn_sched_barrier(0);
  };
  size_t at = place(kb_begin);
  load(Kc, at, kf);
  load(Vc, at, vf);
  at = place(kb_begin + 1);
  for (int kb = kb_begin; kb < kb_end - 1; ++kb) {
    decode_block<RESCALE_MOVED>(acc, kb, nkeys, hh, RegFrags{qf}, RegFrags{kf}, RegFrags{vf},
                                [&] { load(Kc, at, kf); }, [&] { load(Vc, at, vf); });
    at = place(kb + 2);
  }
  decode_block<RESCALE_MOVED>(acc, kb_end - 1, nkeys, hh, RegFrags{qf}, RegFrags{kf}, RegFrags{vf});
  // lanes tl < G hold real heads
  float l_tot = xhalf_sum(acc.l);
  if (tl < G) {
    int head = kvh * G + tl;
    float *dst = part + (((size_t)req * nq + head) * max_chunks + chunk) * kPartStride;
    if (hh == 0) { dst[0] = acc.m; dst[1] = l_tot; }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[2 + db * 32 + 8 * (r >> 2) + 4 * hh + (r & 3)] = acc.o[db][r];
  }
}

// ----------------------------------------------------------------------------
// Decode attention while every context is short (kShortKeys): one workgroup per (request, KV
// head), whose 8 waves take the 32-key blocks in turn (the first AHEAD requested at once, then
// whatever is left one by one) and meet in LDS in wave order.  No partial results in memory and no
// merging launch, which is what a short context costs: at 16 requests of up to 440 keys of a stage
// with room for 4043 the chunked pair of kernels takes 15.2 + 5.3 us, this one 8.3; at one request
// of 64 - 192 keys 5.9 + 5.4 us against 5.4.
// ----------------------------------------------------------------------------
constexpr int kShortWaves = 8;
struct ShortLds {
  float m[kShortWaves][4], l[kShortWaves][4], o[kShortWaves][4][132];
};

template <int AHEAD>  // blocks per wave that are requested at once
__device__ __forceinline__ void decode_short(const bf16_t *qdec, const bf16_t *Kc, const bf16_t *Vc, const CacheGeom &geom, const int *lens,
                                             bf16_t *out, int nq, int G, int kvh, int req, ShortLds &lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, hh = lane >> 5, tl = lane & 31;
  bf16x8_t qf[8];
  const bf16_t *qb = qdec + ((size_t)req * geom.nkv + kvh) * (32 * 128);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) qf[dt] = *(const bf16x8_t *)(qb + dt * kTileElems + lane * 8);
  const int nkeys = lens[req] + 1;  // the new token's key is already in the cache
  const int n_kb = (nkeys + 31) >> 5;
  DecodeAcc acc;
  decode_clear(acc);
  bf16x8_t kS[AHEAD][8], vS[AHEAD][8];
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (wave + u * kShortWaves < n_kb) decode_load(Kc, Vc, geom.off(req, kvh, wave + u * kShortWaves) + lane * 8, kS[u], vS[u]);
  if (wave < n_kb) decode_block<RESCALE_NEVER>(acc, wave, nkeys, hh, RegFrags{qf}, RegFrags{kS[0]}, RegFrags{vS[0]});
#pragma unroll
  for (int u = 1; u < AHEAD; ++u)
    if (wave + u * kShortWaves < n_kb)
      decode_block<RESCALE_ALWAYS>(acc, wave + u * kShortWaves, nkeys, hh, RegFrags{qf}, RegFrags{kS[u]}, RegFrags{vS[u]});
  // In a step launched by the host nothing is left, normally: it chose AHEAD, and this form, from the lengths it knows.
  // Replays of a step that the caller recorded move the device's lengths alone, so a step launched after them may find
  // more keys here, as a recorded step does between 256 and 512 keys.
#pragma unroll 1
  for (int kb = wave + AHEAD * kShortWaves; kb < n_kb; kb += kShortWaves) {
    const size_t off = geom.off(req, kvh, kb) + lane * 8;
    const bf16_t *qp = qb + lane * 8;
    asm volatile("" : "+v"(qp));  // or the query's fragments are fetched ahead of the loop into registers of their own
    decode_block<RESCALE_ALWAYS>(acc, kb, nkeys, hh, MemFrags{qp}, MemFrags{Kc + off}, MemFrags{Vc + off});
  }
  const float l_tot = xhalf_sum(acc.l);
  if (tl < G) {  // lanes tl < G hold real heads
    if (hh == 0) { lds.m[wave][tl] = acc.m; lds.l[wave][tl] = l_tot; }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(f32x4_t *)&lds.o[wave][tl][db * 32 + 8 * q + 4 * hh] =
            f32x4_t{acc.o[db][4 * q], acc.o[db][4 * q + 1], acc.o[db][4 * q + 2], acc.o[db][4 * q + 3]};
  }
  __syncthreads();
  const int g = threadIdx.x >> 7, d = threadIdx.x & 127;
  if (g >= G) return;
  const float c = kLog2e * 0.08838834764831845f;
  float m = lds.m[0][g];
#pragma unroll
  for (int w = 1; w < kShortWaves; ++w) m = fmaxf(m, lds.m[w][g]);  // -inf: a wave without a block
  float o = 0.f, l = 0.f;
#pragma unroll
  for (int w = 0; w < kShortWaves; ++w) {
    const float wgt = w < n_kb ? fast_exp2((lds.m[w][g] - m) * c) : 0.f;  // waves without a block hold zeros
    l = merge_sum(l, wgt, lds.l[w][g]);
    o = merge_out(o, wgt, lds.o[w][g][d]);
  }
  out[frag_offset(req, (kvh * G + g) * 128 + d, nq * 128)] = f2bf_dev(o / l);
}

// Workgroup e = id - first beyond those of the attention proper: the first bytes of one row group of the next launch's weights, into
// the L2 of the XCD that is going to stream them (workgroups go to the XCDs in turn, from the same one in every launch; what L2
// holds outlives a launch).  Attention over short contexts leaves HBM idle while it waits for lengths, keys and its waves.
// (With 28 MiB of the 50 of the O projection of a Phi-3 block: batch 1, 64 - 192 keys: attention 4.8 -> 5.8 us, O 11.4 -> 9.4;
// a decode block of batch 16 x 400 keys 132.9 -> 132.0 us, of 32 x 100 146.3 -> 143.5; Llama3-8B, batch 16 x 400: 100.8 -> 98.5.
// Beside the merge of longer contexts, which is shorter, it made a block 0.7 % slower.)
__device__ __forceinline__ void read_ahead(const ReadAhead &r, int first, int id) {
  const int group = (id - first) / 8 * 8 + id % 8;
  if (group >= r.groups) return;
  constexpr int kRound = kShortWaves * 64 * 16, kAtOnce = 8;
  const char *p = (const char *)r.W + (size_t)group * r.group_stride + threadIdx.x * 16;
  for (int at = 0; at < r.group_bytes; at += kAtOnce * kRound) {
    f32x4_t v[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) v[u] = *(const f32x4_t *)(p + min(at + u * kRound, r.group_bytes - kRound));
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) asm volatile("" ::"v"(v[u]));
  }
}

// READS: with workgroups that read ahead; looking for them costs the others 0.2 us
template <int AHEAD, bool READS>
__global__ void __launch_bounds__(kShortWaves * 64) __attribute__((amdgpu_waves_per_eu(AHEAD == 1 ? 4 : 2)))
k_attn_decode_short(const bf16_t *__restrict__ qdec, const bf16_t *__restrict__ Kc, const bf16_t *__restrict__ Vc, CacheGeom geom,
                    const int *__restrict__ lens, bf16_t *__restrict__ out, int nq, int G, int batch, ReadAhead ahead) {
  __shared__ ShortLds lds;
  if (READS && (int)blockIdx.y >= batch) {
    read_ahead(ahead, batch * gridDim.x, blockIdx.y * gridDim.x + blockIdx.x);
    return;
  }
  decode_short<AHEAD>(qdec, Kc, Vc, geom, lens, out, nq, G, blockIdx.x, blockIdx.y, lds);
}

// 128 threads (d) combine the chunks of one (request, query head) in chunk order.  Lane i of their first wave takes
// chunk i (max, sum -> weight); then thread d accumulates output feature d over all chunks, eight loads in flight at a
// time.  Threads that are not `live` only meet the barrier.
// One round trip: the first 16 chunks' outputs, the maxima and the sums are requested for every chunk slot the buffer
// has, without waiting for the request's length; slots past n_chunks hold whatever an earlier step left there and are
// dropped below without entering any arithmetic.
struct MergeLoads {
  const float *src;
  float v0[16], m, l;
  __device__ __forceinline__ MergeLoads(const float *part, int nq, int max_chunks, int head, int req, int d, bool live) {
    src = part + ((size_t)req * nq + head) * max_chunks * kPartStride;
#pragma unroll
    for (int u = 0; u < 16; ++u) v0[u] = live && u < max_chunks ? src[u * kPartStride + 2 + d] : 0.f;
    m = l = 0.f;
    if (live && d < 64 && d < max_chunks) { m = src[d * kPartStride]; l = src[d * kPartStride + 1]; }
  }
};
__device__ __forceinline__ void merge_chunks(const MergeLoads &in, int len, bf16_t *out, int nq, int chunk_keys, int head, int req, int d,
                                             bool live, float *wgt /*64*/, float *lsum) {
  const int n_chunks = (len + 1 + chunk_keys - 1) / chunk_keys;  // <= 64 by the host's choice of chunk_keys
  const float c = kLog2e * 0.08838834764831845f;
  const float *src = in.src;
  if (live && d < 64) {
    float mi = d < n_chunks ? in.m : -INFINITY;
    float li = d < n_chunks ? in.l : 0.f;
    float m = mi;
    for (int o2 = 32; o2 > 0; o2 >>= 1) m = fmaxf(m, __shfl_xor(m, o2, 64));
    float w = d < n_chunks ? exp2f((mi - m) * c) : 0.f;
    wgt[d] = w;
    float wl = merge_sum(0.f, w, li), tot = 0.f;
    for (int i = 0; i < n_chunks; ++i) tot += __shfl(wl, i, 64);  // chunk order
    if (d == 0) *lsum = tot;
  }
  __syncthreads();
  if (!live) return;
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 16; ++u)
    if (u < n_chunks) acc = merge_out(acc, wgt[u], in.v0[u]);
  int i = 16;
  for (; i + 8 <= n_chunks; i += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[(i + u) * kPartStride + 2 + d];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = merge_out(acc, wgt[i + u], v[u]);
  }
  for (; i < n_chunks; ++i) acc = merge_out(acc, wgt[i], src[i * kPartStride + 2 + d]);
  out[frag_offset(req, head * 128 + d, nq * 128)] = f2bf_dev(acc / *lsum);
}

// one workgroup per (request, query head)
__global__ void __launch_bounds__(128) k_attn_decode_merge(const float *__restrict__ part,
                                                           const int *__restrict__ lens,
                                                           bf16_t *__restrict__ out, int nq,
                                                           int max_chunks, int chunk_keys) {
  __shared__ float wgt[64];
  __shared__ float lsum;
  const MergeLoads in(part, nq, max_chunks, blockIdx.x, blockIdx.y, threadIdx.x, true);
  merge_chunks(in, lens[blockIdx.y], out, nq, chunk_keys, blockIdx.x, blockIdx.y, threadIdx.x, true, wgt, &lsum);
}

// The second kernel of a recorded step, one workgroup per (request, KV head): the merge, or the whole of a short batch's
// attention, whose first kernel returned at once.  (A step that the caller replays must give what a direct call gives at
// the same context, and the two forms add up in different orders.)  Latency: a replayed 256-wide block of 8 requests takes
// 32.9 us at 200 keys (39.1 as chunks) and 62.6 at 4500 (62.0 with the merge in workgroups of one head each).
__global__ void __launch_bounds__(kShortWaves * 64) __attribute__((amdgpu_waves_per_eu(4)))
k_attn_decode_recorded_end(const bf16_t *__restrict__ qdec, const bf16_t *__restrict__ Kc, const bf16_t *__restrict__ Vc, CacheGeom geom,
                           const int *__restrict__ lens, const float *__restrict__ part, bf16_t *__restrict__ out, int nq, int G,
                           int max_chunks, int chunk_keys) {
  static_assert(kShortWaves * 64 == 4 * 128, "128 threads for each of up to 4 query heads");
  __shared__ ShortLds lds;
  __shared__ float wgt[4][64], lsum[4];
  const int kvh = blockIdx.x, req = blockIdx.y, g = threadIdx.x >> 7, head = kvh * G + min(g, G - 1), d = threadIdx.x & 127;
  const int mine = batch_len(lens, gridDim.y, threadIdx.x & 63);
  const MergeLoads in(part, nq, max_chunks, head, req, d, g < G);  // on their way while the lengths arrive
  asm volatile("" ::: "memory");
  if (all_short(mine)) decode_short<1>(qdec, Kc, Vc, geom, lens, out, nq, G, kvh, req, lds);
  else merge_chunks(in, __builtin_amdgcn_readlane(mine, req), out, nq, chunk_keys, head, req, d, g < G, wgt[g], &lsum[g]);
}

}  // namespace

hipError_t mfma_attn_prefill(const bf16_t *q, const bf16_t *Kc, bf16_t *Vc, CacheGeom geom,
                             bf16_t *out, const PrefillTile *tiles, int n_tiles, const int *req_len,
                             int nq, int nkv, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  const int G = nq / nkv;
  const dim3 grid(n_tiles, nkv);
  switch (G) {
    case 1: k_attn_prefill<1><<<grid, 128, kAttnPrefillLds, s>>>(q, Kc, Vc, geom, out, tiles, req_len, nq); break;
    case 2: k_attn_prefill<2><<<grid, 256, kAttnPrefillLds, s>>>(q, Kc, Vc, geom, out, tiles, req_len, nq); break;
    case 3: k_attn_prefill<3><<<grid, 384, kAttnPrefillLds, s>>>(q, Kc, Vc, geom, out, tiles, req_len, nq); break;
    case 4: k_attn_prefill<4><<<grid, 512, kAttnPrefillLds, s>>>(q, Kc, Vc, geom, out, tiles, req_len, nq); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t mfma_attn_init() {
  hipError_t e = hipFuncSetAttribute((const void *)k_attn_prefill<1>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnPrefillLds);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_attn_prefill<2>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnPrefillLds);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_attn_prefill<3>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnPrefillLds);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_attn_prefill<4>, hipFuncAttributeMaxDynamicSharedMemorySize, kAttnPrefillLds);
  return e;
}

size_t mfma_attn_decode_part_floats(int nq, int batch, int max_chunks) {
  return (size_t)batch * nq * max_chunks * kPartStride;
}

hipError_t mfma_attn_decode(const bf16_t *qdec, const bf16_t *Kc, const bf16_t *Vc, CacheGeom geom,
                            const int *lens, float *part, bf16_t *out, int nq, int nkv, int batch,
                            int max_chunks, int chunk_keys, int form, const ReadAhead &ahead, hipStream_t s) {
  int G = nq / nkv;
  const dim3 chunks(nkv, batch, max_chunks), heads(nkv, batch);
  // the workgroups that read ahead: one per row group, whole rounds of the XCDs, behind the others; whole rounds of their threads
  ReadAhead ra = ahead;
  constexpr int kRound = kShortWaves * 64 * 16;
  ra.group_bytes = std::min(ra.group_bytes, ra.group_stride) / kRound * kRound;
  if (ra.group_bytes == 0) ra.groups = 0;
  const dim3 short_grid(nkv, batch + ((ra.groups + 7) / 8 * 8 + nkv - 1) / nkv);
  auto launch_short = [&](auto ahead) {
    constexpr int kAhead = decltype(ahead)::value;
    if (ra.groups) k_attn_decode_short<kAhead, true><<<short_grid, kShortWaves * 64, 0, s>>>(qdec, Kc, Vc, geom, lens, out, nq, G, batch, ra);
    else k_attn_decode_short<kAhead, false><<<heads, kShortWaves * 64, 0, s>>>(qdec, Kc, Vc, geom, lens, out, nq, G, batch, ra);
  };
  hipError_t e = hipSuccess;
  switch (form) {
    case DEC_ATTN_SHORT: launch_short(std::integral_constant<int, 1>()); break;
    case DEC_ATTN_SHORT2: launch_short(std::integral_constant<int, 2>()); break;
    case DEC_ATTN_CHUNKED:
      k_attn_decode<false><<<chunks, 64, 0, s>>>(qdec, Kc, Vc, geom, lens, part, nq, G, max_chunks, chunk_keys);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      k_attn_decode_merge<<<dim3(nq, batch), 128, 0, s>>>(part, lens, out, nq, max_chunks, chunk_keys);
      break;
    case DEC_ATTN_RECORDED:
      k_attn_decode<true><<<chunks, 64, 0, s>>>(qdec, Kc, Vc, geom, lens, part, nq, G, max_chunks, chunk_keys);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      k_attn_decode_recorded_end<<<heads, kShortWaves * 64, 0, s>>>(qdec, Kc, Vc, geom, lens, part, out, nq, G, max_chunks, chunk_keys);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace hyp
