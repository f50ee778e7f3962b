// Decode-step kernels of the MFMA path: the weight-streaming skinny GEMM
// (<= 32 tokens against a [N, K] matrix, bandwidth-bound) with its consumers fused
// into the workgroup that finishes a row group (RoPE + cache append, SwiGLU,
// residual + next norm), and the kernel that opens a step, for the KV-cached
// generation phase of the decoder block of Sec. III-A.
#include "mfma_common.h"
#include "mfma_kernels.h"

namespace hyp {

namespace {

// ----------------------------------------------------------------------------
// Skinny GEMM of a decode step with its consumer fused in.
//
//   sum[token, n] = sum_k W[n, k] x[token, k]        (<= 32 tokens, W streamed once)
//
// W = P(N, K): the 1 KiB tiles of one 32-row block are contiguous along K and a
// tile is the MFMA A fragment as it stands, so every wave streams its slice
// with fully coalesced 1 KiB loads straight into registers.  x = P(32, K) is
// tiny and stays in L2.  A workgroup owns 64 packed rows (2 blocks), or 32 in unsplit
// forms of QKV and the O / down projections; its NW waves (4 or 8) split the
// workgroup's K slice and are reduced through LDS in wave order; the
// `ksplit` workgroups of one row group (two or four times as many for the row groups that would
// otherwise form a thin second round of the launch) write fp32 partial sums, and the one that
// arrives last (a counter per row group) adds them up in slice order - so the
// result does not depend on which one that is - and runs the epilogue.  The
// partial sums are written with device-scope (write-through) stores that have
// completed before the counter is bumped, which keeps cache write-backs and
// invalidations out of the protocol.  Epilogues:
//   DEC_QKV    scale by the RMS Norm factor, RoPE at position lens[b], write q
//              to the decode query buffer and k, v into the cache
//   DEC_QKV_OPEN  DEC_QKV for the first block of a stage: x is hidden_in, as the caller gives it or copied to be aligned, and
//              gain, rounding and sums of squares of the norm happen on the way to the MFMAs (30 vector instructions per KiB
//              of weights, hidden under them); every workgroup sees all of K.  Also leaves the residual stream
//   DEC_SWIGLU scale, m = silu(gate) * up -> P(32, I)
//   DEC_RESID  x += sum ; xres = x ; y' = x * gain -> P(32, H) ; per-token sum of
//              squares of this row group -> ssq_out   (RMS Norm of the next
//              sub-layer, applied by that sub-layer's epilogue as a scale:
//              W (x * rstd * g) = rstd * W (x * g))
//   DEC_FINAL  x += sum ; hidden_out = x ; the finisher of row group 0 also counts the
//              step's token into the cached lengths (every reader of them in this
//              step ran in an earlier kernel)
// ----------------------------------------------------------------------------
// A wave keeps 10 weight loads of 1 KiB in flight (a window of 5 k-tiles of two row blocks, or 10 of
// one); 16 such waves per CU (124 registers, kWavesPerCu) measured better than 20 loads in flight at 12 waves.
constexpr int kBeginRows = 64;  // rows per workgroup of the kernel that opens a step (and per sum of squares it writes)

struct DecGemvParams {
  const bf16_t *W, *x;
  float *partial;
  unsigned *counters;
  int N, KT, ksplit, tiles_per_wave, batch;
  // row groups from `groups1` on are split `tail` times as fine (they run last and keep the launch's tail short)
  int groups1, n_groups, tail;
  const float *ssq_in;  // [n_ssq][32]
  int n_ssq;
  float inv_H, eps;
  const int *lens;
  const float *cos_tab, *sin_tab;
  bf16_t *qdec, *Kc, *Vc;
  CacheGeom geom;
  int nq, nkv;
  bf16_t *m_out;
  int I;
  float *xres;
  const bf16_t *gain;
  bf16_t *y_out;
  float *ssq_out;
  bf16_t *hidden_out;
  int H;
  int *lens_advance;  // DEC_FINAL: cached lengths to bump once the step's last kernel finishes
};

// FBW row blocks of 32 per workgroup: 2 where the epilogue pairs rows of two blocks (gate and up) and for long K; 1 or 2 for QKV,
// whose RoPE partners lie in one block; 1 for the residual epilogues at short K, where 32-row workgroups with
// a 10-tile window give as many waves with as much in flight as two slices of 64-row workgroups
// would, without partial sums, counter and gather at the end.
// CLS (a hyp_kernel_class_t) only gives each GEMM of a block its own kernel name in a trace.
// NW waves per workgroup share the k-tiles of the workgroup's K slice: more waves per workgroup mean
// fewer K slices across workgroups (fewer partial sums in memory, or none) for the same number of
// waves in flight.
// SHORT: one window (mfma_gemv_one_window).
template <int EPI, int FBW, int NW, int CLS, bool SHORT>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(EPI == DEC_QKV_OPEN || SHORT ? 2 : 4))) k_dec_gemv(DecGemvParams p) {
  constexpr bool kOpen = EPI == DEC_QKV_OPEN, kQkv = EPI == DEC_QKV || kOpen, kSsqIn = EPI == DEC_QKV || EPI == DEC_SWIGLU;
  constexpr int UNROLL = gemv_window(FBW, SHORT);
  constexpr int kGroupRows = FBW * 32;
  constexpr int kRedStride = kGroupRows + 4;  // keeps 16-byte alignment, spreads tokens over banks
  constexpr int kSsqParts = NW * 2;  // interleaved partial sums of the row groups' sums of squares (one per 32 threads)
  // the waves' sums as [wave][token][row], tokens of the batch only: rows contiguous so that the
  // cross-wave add reads without bank conflicts; reused as fin[token][kGroupRows + 1] once reduced
  extern __shared__ __attribute__((aligned(16))) float red_raw[];
  float (*red)[kRedStride] = (float (*)[kRedStride])red_raw;  // red[wave * batch + token][row]
  __shared__ unsigned is_last;
  float (*fin)[kGroupRows + 1] = (float (*)[kGroupRows + 1])red_raw;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // 1-D grid: first the `ksplit` slices of row groups [0, groups1), slice-major, then the
  // tail * ksplit slices of the remaining groups
  int group, ks, ksplit = p.ksplit, tiles_per_wave = p.tiles_per_wave;
  {
    const int first = p.groups1 * p.ksplit, id = blockIdx.x;
    if (id < first) { group = id % p.groups1; ks = id / p.groups1; }
    else {
      const int g2 = p.n_groups - p.groups1, id2 = id - first;
      group = p.groups1 + id2 % g2; ks = id2 / g2; ksplit *= p.tail; tiles_per_wave /= p.tail;
    }
  }
  const int fb0 = group * FBW;
  const bool split = !kQkv && !SHORT && ksplit > 1;  // QKV is never split
  // partial sums [slice][32 tokens][rows]: the finely cut last groups have a narrow array of their own behind the
  // main one (rows of those groups only), so their extra slices do not cost room over all N rows
  const bool fine = group >= p.groups1;
  float *const part = fine ? p.partial + (size_t)p.ksplit * 32 * p.N : p.partial;
  const int part_n = fine ? (p.n_groups - p.groups1) * kGroupRows : p.N;        // rows per token
  const int part_r0 = fine ? (group - p.groups1) * kGroupRows : fb0 * 32;       // this group's first row
  // positions of the step's tokens (the QKV epilogue's rotary angles depend on them): fetched under the streaming loop, a
  // thread's pairs of up to 32 tokens
  constexpr int kPairs = FBW * 16, kPf = (32 * kPairs + NW * 64 - 1) / (NW * 64);
  static_assert(!kQkv || kPf <= 2, "registers");
  int pos_pf[kPf] = {};
  if (kQkv) {
#pragma unroll
    for (int j = 0; j < kPf; ++j) {
      int idx = threadIdx.x + j * NW * 64;
      if (idx < p.batch * kPairs) pos_pf[j] = p.lens[idx / kPairs];
    }
  }
  // the workgroup's NW waves take the k-tiles of its slice in turn, so that each step of
  // the workgroup reads NW KiB contiguous per row block (HBM serves that pattern ~10 % faster
  // than separate 1 KiB streams)
  const int kt0 = ks * NW * tiles_per_wave + wave;
  constexpr size_t kStep = (size_t)NW * kTileElems;
  f32x16_t acc[FBW];
#pragma unroll
  for (int i = 0; i < FBW; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  // token columns beyond the batch feed output columns nobody reads: their lanes all read
  // token 0's chunk, so the x tile costs one cache line more instead of a whole tile
  const bf16_t *xp = kOpen ? p.x + (size_t)((lane & 31) < p.batch ? lane & 31 : 0) * p.H + kt0 * 16 + (lane >> 5) * 8
                           : p.x + (size_t)kt0 * kTileElems + ((lane & 31) < p.batch ? lane : (lane & 32)) * 8;
  const bf16_t *wp[FBW];
#pragma unroll
  for (int i = 0; i < FBW; ++i) wp[i] = p.W + ((size_t)(fb0 + i) * p.KT + kt0) * kTileElems + lane * 8;
  // A window of UNROLL k-tiles lives in registers; as soon as a tile has gone through the
  // MFMAs its registers are reloaded with the tile UNROLL further on, so the wave keeps
  // about 2 (UNROLL - 1) KiB of weights in flight all the time.
  bf16x8_t xf[UNROLL], wf[FBW][UNROLL];
  auto load_tile = [&](int u, int tile) {
#pragma unroll
    for (int i = 0; i < FBW; ++i) {
      const bf16x8_t *w = (const bf16x8_t *)(wp[i] + (size_t)tile * kStep);
      wf[i][u] = SHORT ? *w : __builtin_nontemporal_load(w);
    }
    xf[u] = *(const bf16x8_t *)(xp + (size_t)tile * (kOpen ? NW * 16 : kStep));
  };
  // DEC_QKV_OPEN: gain and rounding of the norm on the way to the MFMA, and the tokens' sums of squares of this wave's k-tiles
  bf16_t *const gain_s = (bf16_t *)(red_raw + NW * p.batch * kRedStride);  // behind the waves' sums
  float sq = 0.f;
  auto open_tile = [&](int u, int tile) {
    const bf16x8_t g = *(const bf16x8_t *)(gain_s + (kt0 + tile * NW) * 16 + (lane >> 5) * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = (float)xf[u][e];
      sq += x * x;
      xf[u][e] = (__bf16)(x * (float)g[e]);
    }
  };
  auto open = [&] {
    if constexpr (kOpen) {
      for (int c = threadIdx.x; c < p.H / 8; c += NW * 64) *(u16x8_t *)(gain_s + c * 8) = *(const u16x8_t *)(p.gain + c * 8);
      // the residual stream: 64 features of every token per workgroup
      if (blockIdx.x < (unsigned)p.H / 64)
        for (int c = threadIdx.x; c < p.batch * 8; c += NW * 64) {
          const size_t at = (size_t)(c >> 3) * p.H + blockIdx.x * 64 + (c & 7) * 8;
          const u16x8_t h = *(const u16x8_t *)(p.x + at);
#pragma unroll
          for (int e = 0; e < 8; e += 4)
            *(f32x4_t *)(p.xres + at + e) = f32x4_t{bf16_to_f32(h.v[e]), bf16_to_f32(h.v[e + 1]), bf16_to_f32(h.v[e + 2]), bf16_to_f32(h.v[e + 3])};
        }
      __syncthreads();
    }
  };
  auto use_tile = [&](int u, int tile) {
    if constexpr (kOpen) open_tile(u, tile);
#pragma unroll
    for (int i = 0; i < FBW; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][u], xf[u], acc[i], 0, 0, 0);
  };
  const int n_pairs = p.batch * kGroupRows;
  // What the epilogue needs from memory besides the sums, requested at once: rotary angles, residual stream and next norm's
  // gain, the sums of squares behind the RMS Norm factor (16 row groups per thread).
  float cos_pf[kPf] = {}, sin_pf[kPf] = {};
  constexpr int kPfR = 32 * kGroupRows / (NW * 64);  // (token, row) pairs of a thread
  float xres_pf[kPfR], gain_pf[kPfR];
  float ssq_v[16];
  const int ssq_tkn = threadIdx.x & 31, ssq_part_id = threadIdx.x >> 5;
  auto fetch_angles = [&] {
    if (kQkv) {
#pragma unroll
      for (int j = 0; j < kPf; ++j) {
        int idx = threadIdx.x + j * NW * 64;
        if (idx < p.batch * kPairs) {
          int d0 = (fb0 & 3) * 16 + idx % kPairs;
          cos_pf[j] = p.cos_tab[(size_t)pos_pf[j] * 64 + d0];
          sin_pf[j] = p.sin_tab[(size_t)pos_pf[j] * 64 + d0];
        }
      }
    }
  };
  auto fetch = [&] {
    if (EPI == DEC_RESID || EPI == DEC_FINAL) {
#pragma unroll
      for (int j = 0; j < kPfR; ++j) {
        int idx = threadIdx.x + j * NW * 64;
        xres_pf[j] = 0.f; gain_pf[j] = 0.f;
        if (idx < n_pairs) {
          int f = idx % kGroupRows, b = idx / kGroupRows;
          xres_pf[j] = p.xres[(size_t)b * p.H + fb0 * 32 + f];
          if (EPI == DEC_RESID) gain_pf[j] = bf16_to_f32(p.gain[fb0 * 32 + f]);
        }
      }
    }
    if (kSsqIn) {
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        int g = ssq_part_id + kSsqParts * u;
        ssq_v[u] = g < p.n_ssq && ssq_tkn < p.batch ? p.ssq_in[g * 32 + ssq_tkn] : 0.f;
      }
    }
  };
  const int n_win = SHORT ? 0 : tiles_per_wave / UNROLL, rem = tiles_per_wave - n_win * UNROLL;
  if (SHORT) fetch();
  if (n_win > 0) {
    int t = 0;
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) load_tile(u, u);
    open();
    for (int wi = 1; wi < n_win; ++wi, t += UNROLL) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        use_tile(u, t + u);
        load_tile(u, t + UNROLL + u);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // last full window; the rem (< UNROLL) tiles left over move into its registers as they free up
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      use_tile(u, t + u);
      if (u < rem) load_tile(u, t + UNROLL + u);
    }
  } else {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
      if (u < rem) load_tile(u, u);
    if (SHORT) fetch_angles();
    open();
  }
#pragma unroll
  for (int u = 0; u < UNROLL; ++u)
    if (u < rem) use_tile(u, n_win * UNROLL + u);
  // An unsplit workgroup finishes for sure: the requests go out ahead of the waves' meeting (512-wide blocks: 1.1 of 4.4 us
  // of QKV and gate/up were this round trip, with the epilogue's turn through LDS); a slice waits to know that it is the last.
  if (!split && !SHORT) {
    fetch_angles();
    fetch();
  }
  // The RMS Norm factor of a token: the row groups' sums of squares, added in a fixed order (kSsqParts interleaved partial sums,
  // which meet in LDS with the products, then those in order, by every thread that needs the factor: a barrier and a chain of
  // one wave's additions less).
  constexpr bool kNorm = kQkv || EPI == DEC_SWIGLU;
  __shared__ float ssq_part[kNorm ? kSsqParts : 1][32];
  auto sum_squares = [&] {
    if constexpr (kOpen) {
      ssq_part[ssq_part_id][ssq_tkn] = sq;  // a wave's two halves of its k-tiles
    } else if constexpr (kNorm) {
      float ss = 0.f;
#pragma unroll
      for (int u = 0; u < 16; ++u) ss += ssq_v[u];
      for (int g = ssq_part_id + kSsqParts * 16; g < p.n_ssq; g += kSsqParts) ss += p.ssq_in[g * 32 + ssq_tkn];
      ssq_part[ssq_part_id][ssq_tkn] = ss;
    }
  };
  auto rstd = [&](int token) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < kSsqParts; ++i) ss += ssq_part[kNorm ? i : 0][token];
    return 1.0f / sqrtf(ss * p.inv_H + p.eps);
  };
  if (!split) sum_squares();
  // accumulator register r of lane l of block i is packed row 32 i + 8 (r/4) + 4 (l/32) + r%4 of
  // token l % 32: four consecutive rows per 16-byte store; token columns beyond the batch stay home
  if ((lane & 31) < p.batch) {
#pragma unroll
    for (int i = 0; i < FBW; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4_t v = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
        *(f32x4_t *)&red[wave * p.batch + (lane & 31)][32 * i + 8 * q + 4 * (lane >> 5)] = v;
      }
  }
  __syncthreads();
  // a row's sum over the waves, in wave order
  auto wave_sum = [&](int token, int f) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w * p.batch + token][f];
    return s;
  };
  if (split) {
#pragma unroll
    for (int j = 0; j < kPfR; ++j) {
      int idx = threadIdx.x + j * NW * 64;
      if (idx < n_pairs) {
        int f = idx % kGroupRows, token = idx / kGroupRows;
        // write-through store: visible to the other XCDs once it has completed
        __hip_atomic_store(&part[((size_t)ks * 32 + token) * part_n + part_r0 + f], wave_sum(token, f), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);  // this thread's partial sums have completed ...
    __syncthreads();
    if (threadIdx.x == 0) {  // ... before it is counted
      unsigned old = atomicAdd(&p.counters[group], 1u);
      is_last = (old == (unsigned)ksplit - 1) ? 1u : 0u;
      if (is_last) p.counters[group] = 0;  // ready for the next launch
    }
    __syncthreads();  // `red` is free from here on
    if (!is_last) return;
    fetch();
    // The finishing workgroup.  Its loads are device-scope ones (load_shared): `partial` is the same room in every split GEMV of
    // every step, and what this XCD's L2 holds of it from an earlier launch must not be taken for this one's.  (Against plain
    // loads: steps of one block of four widths, 5120 / 17920 to 8192 / 28672, batch 1 - 32, within 0.2 % either way.  An acquire fence,
    // which invalidates L2 under the other workgroups' streams, costs 10 % of a step.)  With more than four slices, two (token, row)
    // pairs per thread and GW slices of each are in flight at once; slices beyond ksplit are masked
    // rather than peeled, so the gather costs ceil(ksplit / GW) round trips.
    constexpr int GW = 16;
    if (ksplit <= 4) {
      // few slices: four of the thread's pairs at once (16 tokens' worth per round trip)
      for (int j0 = 0; j0 * NW * 64 < n_pairs; j0 += 4) {
        float v[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int idx = threadIdx.x + (j0 + j) * NW * 64;
          const bool has = idx < n_pairs;
          const unsigned off = has ? (unsigned)((idx / kGroupRows) * part_n + part_r0 + idx % kGroupRows) : 0u;
#pragma unroll
          for (int u = 0; u < 4; ++u) v[j][u] = has && u < ksplit ? load_shared(part + (size_t)u * 32 * part_n + off) : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int idx = threadIdx.x + (j0 + j) * NW * 64;
          if (idx < n_pairs) fin[idx / kGroupRows][idx % kGroupRows] = ((v[j][0] + v[j][1]) + v[j][2]) + v[j][3];
        }
      }
    } else {
      for (int idx0 = threadIdx.x; idx0 < n_pairs; idx0 += 2 * NW * 64) {
        const int idx1 = idx0 + NW * 64;
        const bool has1 = idx1 < n_pairs;
        // slice bases are uniform (scalar registers); one 32-bit offset per pair serves every slice
        const unsigned off0 = (unsigned)((idx0 / kGroupRows) * part_n + part_r0 + idx0 % kGroupRows);
        const unsigned off1 = (unsigned)(((has1 ? idx1 : idx0) / kGroupRows) * part_n + part_r0 + (has1 ? idx1 : idx0) % kGroupRows);
        float sum0 = 0.f, sum1 = 0.f;
        for (int s = 0; s < ksplit; s += GW) {
          float v0[GW], v1[GW];
#pragma unroll
          for (int u = 0; u < GW; ++u) {
            const bool in = s + u < ksplit;
            const float *slice = part + (size_t)(s + u) * 32 * part_n;
            v0[u] = in ? load_shared(slice + off0) : 0.f;
            v1[u] = in && has1 ? load_shared(slice + off1) : 0.f;
          }
#pragma unroll
          for (int u = 0; u < GW; ++u) { sum0 += v0[u]; sum1 += v1[u]; }
        }
        fin[idx0 / kGroupRows][idx0 % kGroupRows] = sum0;
        if (has1) fin[idx1 / kGroupRows][idx1 % kGroupRows] = sum1;
      }
    }
    sum_squares();
    __syncthreads();
  }
  auto total = [&](int token, int f) { return split ? fin[token][f] : wave_sum(token, f); };

  if (kQkv) {
    const int head = fb0 >> 2;
#pragma unroll
    for (int j = 0; j < kPf; ++j) {
      int idx = threadIdx.x + j * NW * 64;
      if (idx >= p.batch * kPairs) break;
      int x = idx % kPairs, b = idx / kPairs, f = (x >> 4) * 32 + (x & 15);
      const float rs = rstd(b);
      float a = total(b, f) * rs, c = total(b, f + 16) * rs;
      int d0 = (fb0 & 3) * 16 + x, d1 = d0 + 64;
      const int pos = pos_pf[j];
      if (head < p.nq + p.nkv) {
        const float cs = cos_pf[j], sn = sin_pf[j];
        float lo = a * cs - c * sn, hi = c * cs + a * sn;
        if (head < p.nq) {
          int G = p.nq / p.nkv;
          bf16_t *dst = p.qdec + ((size_t)b * p.nkv + head / G) * (32 * 128);
          dst[frag_offset(head % G, d0, 128)] = f2bf_dev(lo);
          dst[frag_offset(head % G, d1, 128)] = f2bf_dev(hi);
        } else {
          bf16_t *dst = p.Kc + p.geom.off(b, head - p.nq, pos >> 5);
          dst[frag_offset(pos & 31, d0, 128)] = f2bf_dev(lo);
          dst[frag_offset(pos & 31, d1, 128)] = f2bf_dev(hi);
        }
      } else {
        bf16_t *dst = p.Vc + p.geom.off(b, head - p.nq - p.nkv, pos >> 5);
        // The feature's 32 slots are four runs of 8: MFMA steps m, lane halves khh.  The token that opens a block clears the
        // rest of it: decode attention multiplies the slots behind the last key by probabilities of zero, and whatever an
        // earlier request left there need not be finite (prefill does the same behind a prompt's last key).  One step in 32;
        // no request's time moved, where masking in the attention kernels cost 0.2 - 0.4 % of it.
        int m, khh;
        const int e = vtile_slot_of_key(pos & 31, &m, &khh);
        auto put = [&](int d, float v) {
          bf16_t *row = dst + (size_t)(d >> 5) * kTileElems + (d & 31) * 8;
          if ((pos & 31) == 0) {
            u16x8_t run = {};
            *(u16x8_t *)(row + 32 * 8) = run;
            *(u16x8_t *)(row + 4 * kTileElems) = run;
            *(u16x8_t *)(row + 4 * kTileElems + 32 * 8) = run;
            run.v[0] = f2bf_dev(v);
            *(u16x8_t *)row = run;
          } else {
            row[(size_t)m * 4 * kTileElems + khh * 32 * 8 + e] = f2bf_dev(v);
          }
        };
        put(d0, a);
        put(d1, c);
      }
    }
  } else if (EPI == DEC_SWIGLU) {
    const int f0 = (fb0 >> 3) * 128 + ((fb0 >> 1) & 3) * 32;
    for (int idx = threadIdx.x; idx < p.batch * 32; idx += NW * 64) {
      int x = idx & 31, b = idx >> 5;
      const float rs = rstd(b);
      float g = total(b, x) * rs, u = total(b, 32 + x) * rs;
      p.m_out[frag_offset(b, f0 + x, p.I)] = f2bf_dev(g / (1.0f + __expf(-g)) * u);
    }
  } else {
    const int n0 = fb0 * 32;
#pragma unroll
    for (int j = 0; j < kPfR; ++j) {
      int idx = threadIdx.x + j * NW * 64;
      if (idx >= n_pairs) break;
      int f = idx % kGroupRows, b = idx / kGroupRows;
      float xn = xres_pf[j] + total(b, f);
      if (EPI == DEC_RESID) {
        p.xres[(size_t)b * p.H + n0 + f] = xn;
        p.y_out[frag_offset(b, n0 + f, p.H)] = f2bf_dev(xn * gain_pf[j]);
        const float ss = lanes_sum_squares<kGroupRows>(xn);  // over the lanes of the token
        if (f == 0) p.ssq_out[group * 32 + b] = ss;
      } else {
        p.hidden_out[(size_t)b * p.H + n0 + f] = f2bf_dev(xn);
      }
    }
    if (EPI == DEC_FINAL && group == 0 && p.lens_advance && threadIdx.x < p.batch) p.lens_advance[threadIdx.x] += 1;
  }
}

// first kernel of a decode step that does not open with its QKV contraction (mfma_dec_opens): x = hidden_in ; xres = x ; y' = x * gain ; ssq
// grid H / 64, 512 threads: a wave per token, a lane per feature, the sum of squares over the wave's lanes.  (Added
// thread by thread through LDS a request of 16 chat prompts took 0.4 % longer; in a trace the kernel sits at the launch
// floor, 4.7 us, either way.)
constexpr int kBeginWaves = 8;
__global__ void __launch_bounds__(kBeginWaves * 64) k_dec_begin(const bf16_t *__restrict__ hidden_in, float *__restrict__ xres,
                                                   const bf16_t *__restrict__ gain, bf16_t *__restrict__ y_out,
                                                   float *__restrict__ ssq_out, int H, int batch) {
  static_assert(kBeginRows == 64, "a lane per feature");
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = blockIdx.x * kBeginRows + lane;
  const float g = bf16_to_f32(gain[n]);
  float x[32 / kBeginWaves];
#pragma unroll
  for (int u = 0; u < 32 / kBeginWaves; ++u) {
    const int b = wave + u * kBeginWaves;
    x[u] = b < batch ? bf16_to_f32(hidden_in[(size_t)b * H + n]) : 0.f;
  }
#pragma unroll
  for (int u = 0; u < 32 / kBeginWaves; ++u) {
    const int b = wave + u * kBeginWaves;
    if (b >= batch) break;
    xres[(size_t)b * H + n] = x[u];
    y_out[frag_offset(b, n, H)] = f2bf_dev(x[u] * g);
    const float ss = lanes_sum_squares<64>(x[u]);
    if (lane == 0) ssq_out[blockIdx.x * 32 + b] = ss;
  }
}

// rows of a step that are not aligned to 16 bytes, next to each other and aligned, as DEC_QKV_OPEN reads them
__global__ void __launch_bounds__(256) k_dec_align(const bf16_t *__restrict__ in, bf16_t *__restrict__ out, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = in[i];
}

__global__ void k_export_kv(const bf16_t *__restrict__ Kc, const bf16_t *__restrict__ Vc, CacheGeom geom,
                            bf16_t *__restrict__ k_out, bf16_t *__restrict__ v_out, int request, int len,
                            int nkv) {
  size_t n = (size_t)len * nkv * 128;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    int pos = (int)(i / (nkv * 128)), e = (int)(i % (nkv * 128));
    int h = e >> 7, d = e & 127;
    size_t blk = geom.off(request, h, pos >> 5);
    k_out[i] = Kc[blk + frag_offset(pos & 31, d, 128)];
    int m, khh;
    int slot = vtile_slot_of_key(pos & 31, &m, &khh);
    v_out[i] = Vc[blk + (size_t)(m * 4 + (d >> 5)) * kTileElems + (khh * 32 + (d & 31)) * 8 + slot];
  }
}

__global__ void k_fill_zero(uint4 *p, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  uint4 z = {0, 0, 0, 0};
  for (; i < n16; i += stride) p[i] = z;
}

}  // namespace

// Row groups [0, groups1) run as plan.ksplit workgroups each, the rest (beyond the first round of the launch, if the plan
// cuts those finer) as plan.ksplit * tail.
static void gemv_cut(const GemvPlan &g, int N, int K, int *groups1, int *tail) {
  const int groups = N / (g.fbw * 32), slots = kWavesPerCu / g.nw * 256, tpw = K / 16 / (g.ksplit * g.nw);
  *groups1 = groups; *tail = 1;
  if (g.tail > 1 && groups * g.ksplit > slots && tpw % g.tail == 0) { *groups1 = slots / g.ksplit; *tail = g.tail; }
}

// floats of partial sums a GEMM cut this way needs: [ksplit][32][N], then [ksplit * tail][32][rows of the finely cut groups]
size_t mfma_gemv_partial_floats(const GemvPlan &g, int N, int K) {
  int groups1, tail;
  gemv_cut(g, N, K, &groups1, &tail);
  const int fine_rows = (N / (g.fbw * 32) - groups1) * g.fbw * 32;
  return (size_t)g.ksplit * 32 * N + (size_t)g.ksplit * tail * 32 * fine_rows;
}

// LDS of the gain beside 68 KiB and less of sums (64 rows of 32 tokens in eight waves)
constexpr int kMaxGainBytes = 65536;
bool mfma_dec_opens(int H, int N, const GemvPlan &g) {
  return sizeof(bf16_t) * H <= (size_t)kMaxGainBytes && N / (32 * g.fbw) >= H / 64;  // a workgroup per 64 features
}

bool mfma_gemv_counts(const GemvPlan &g, int N, int K) {
  int groups1, tail;
  gemv_cut(g, N, K, &groups1, &tail);
  return g.ksplit > 1 || tail > 1;
}

// the (epilogue, blocks per workgroup, waves per workgroup, class, one window) combinations a plan may ask for; one window ends at
// 1024 features of K with four waves and at 1280 with eight, and eight share the K of a 32-row workgroup, or of a residual GEMV, only far beyond
#define HYP_GEMV_VARIANTS(X)                                                                                                   \
  X(DEC_QKV, 1, 4, HYP_K_GEMV_QKV, false) X(DEC_QKV, 1, 8, HYP_K_GEMV_QKV, false) X(DEC_QKV, 2, 8, HYP_K_GEMV_QKV, false)      \
  X(DEC_QKV, 1, 4, HYP_K_GEMV_QKV, true) X(DEC_QKV, 2, 8, HYP_K_GEMV_QKV, true)                                                \
  X(DEC_QKV_OPEN, 1, 4, HYP_K_GEMV_QKV, false) X(DEC_QKV_OPEN, 1, 8, HYP_K_GEMV_QKV, false) X(DEC_QKV_OPEN, 2, 8, HYP_K_GEMV_QKV, false) \
  X(DEC_QKV_OPEN, 1, 4, HYP_K_GEMV_QKV, true) X(DEC_QKV_OPEN, 2, 8, HYP_K_GEMV_QKV, true)                                      \
  X(DEC_SWIGLU, 2, 8, HYP_K_GEMV_GATEUP, false) X(DEC_SWIGLU, 2, 8, HYP_K_GEMV_GATEUP, true)                                   \
  X(DEC_RESID, 1, 4, HYP_K_GEMV_O, false) X(DEC_RESID, 2, 8, HYP_K_GEMV_O, false) X(DEC_RESID, 1, 4, HYP_K_GEMV_O, true)       \
  X(DEC_RESID, 1, 4, HYP_K_GEMV_DOWN, false) X(DEC_RESID, 2, 8, HYP_K_GEMV_DOWN, false) X(DEC_RESID, 1, 4, HYP_K_GEMV_DOWN, true) \
  X(DEC_FINAL, 1, 4, HYP_K_GEMV_DOWN, false) X(DEC_FINAL, 2, 8, HYP_K_GEMV_DOWN, false) X(DEC_FINAL, 1, 4, HYP_K_GEMV_DOWN, true)

// the waves' sums of 32 tokens can pass the 64 KiB a workgroup gets by default
hipError_t mfma_gemv_init() {
  hipError_t e = hipSuccess;
#define X(EPI, FBW, NW, CLS, SHORT)                                                                                          \
  if (e == hipSuccess)                                                                                                       \
    e = hipFuncSetAttribute((const void *)k_dec_gemv<EPI, FBW, NW, CLS, SHORT>, hipFuncAttributeMaxDynamicSharedMemorySize,  \
                            (int)(sizeof(float) * NW * 32 * (FBW * 32 + 4)) + (EPI == DEC_QKV_OPEN ? kMaxGainBytes : 0));
  HYP_GEMV_VARIANTS(X)
#undef X
  return e;
}

hipError_t mfma_dec_gemv(int epi, int cls, const DecGemv &a, hipStream_t s) {
  DecGemvParams p = {};
  const int fbw = a.plan.fbw, nw = a.plan.nw, ksplit = a.plan.ksplit;
  p.W = a.W; p.x = a.x; p.partial = a.partial; p.counters = a.counters;
  p.N = a.N; p.KT = a.K / 16; p.ksplit = ksplit; p.tiles_per_wave = p.KT / (ksplit * nw); p.batch = a.batch;
  if ((epi == DEC_QKV || epi == DEC_QKV_OPEN) && ksplit != 1) return hipErrorInvalidValue;
  if (p.tiles_per_wave * ksplit * nw != p.KT || a.N % (fbw * 32) != 0 || kWavesPerCu % nw != 0) return hipErrorInvalidValue;
  p.ssq_in = a.ssq_in; p.n_ssq = a.n_ssq; p.inv_H = a.n_ssq || epi == DEC_QKV_OPEN ? 1.0f / (float)a.K : 0.f; p.eps = a.eps;
  p.lens = a.lens; p.cos_tab = a.cos_tab; p.sin_tab = a.sin_tab; p.qdec = a.qdec; p.Kc = a.Kc; p.Vc = a.Vc;
  p.geom = a.geom; p.nq = a.nq; p.nkv = a.nkv; p.m_out = a.m_out; p.I = a.I; p.xres = a.xres; p.gain = a.gain;
  p.y_out = a.y_out; p.ssq_out = a.ssq_out; p.hidden_out = a.hidden_out; p.H = a.H; p.lens_advance = a.lens_advance;
  // the plan's finer cut of the row groups beyond the first round
  const int groups = a.N / (fbw * 32);
  p.n_groups = groups;
  gemv_cut(a.plan, a.N, a.K, &p.groups1, &p.tail);
  if (mfma_gemv_partial_floats(a.plan, a.N, a.K) > a.partial_floats) return hipErrorInvalidValue;
  dim3 grid(p.groups1 * ksplit + (groups - p.groups1) * p.tail * ksplit);
  // the waves' sums of the live tokens, and the norm's gain
  const size_t lds = sizeof(float) * nw * a.batch * (fbw * 32 + 4) + (epi == DEC_QKV_OPEN ? sizeof(bf16_t) * a.H : 0);
  if (epi == DEC_QKV_OPEN && (a.K != a.H || (uintptr_t)a.x % 16 != 0 || !mfma_dec_opens(a.H, a.N, a.plan))) return hipErrorInvalidValue;
  const bool one_window = mfma_gemv_one_window(a.plan, a.N, a.K);
  bool launched = false;
#define X(EPI, FBW, NW, CLS, SHORT)                                                                   \
  if (!launched && epi == EPI && fbw == FBW && nw == NW && cls == CLS && one_window == SHORT) {         \
    k_dec_gemv<EPI, FBW, NW, CLS, SHORT><<<grid, NW * 64, lds, s>>>(p);                                 \
    launched = true;                                                                                    \
  }
  HYP_GEMV_VARIANTS(X)
#undef X
  if (!launched) return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t mfma_dec_begin(const bf16_t *hidden_in, float *xres, const bf16_t *gain, bf16_t *y_out, float *ssq_out,
                          int H, int batch, hipStream_t s) {
  k_dec_begin<<<H / kBeginRows, kBeginWaves * 64, 0, s>>>(hidden_in, xres, gain, y_out, ssq_out, H, batch);
  return hipGetLastError();
}

hipError_t mfma_dec_align(const bf16_t *hidden_in, bf16_t *out, int H, int batch, hipStream_t s) {
  const int n = H * batch;
  k_dec_align<<<(n + 255) / 256, 256, 0, s>>>(hidden_in, out, n);
  return hipGetLastError();
}

hipError_t mfma_export_kv(const bf16_t *Kc, const bf16_t *Vc, CacheGeom geom, bf16_t *k_out,
                          bf16_t *v_out, int request, int len, int nkv, hipStream_t s) {
  if (len == 0) return hipSuccess;
  size_t n = (size_t)len * nkv * 128;
  int grid = (int)((n + 255) / 256 > 4096 ? 4096 : (n + 255) / 256);
  k_export_kv<<<grid, 256, 0, s>>>(Kc, Vc, geom, k_out, v_out, request, len, nkv);
  return hipGetLastError();
}

hipError_t mfma_fill_zero(void *p, size_t bytes, hipStream_t s) {
  size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  int grid = (int)((n16 + 255) / 256 > 16384 ? 16384 : (n16 + 255) / 256);
  k_fill_zero<<<grid, 256, 0, s>>>((uint4 *)p, n16);
  return hipGetLastError();
}

}  // namespace hyp
