// Shape-generic kernels of a decode step (Sec. III-A of the paper): contractions of up to 32 token rows and attention of one
// new token per request over the cache.  A step is a chain of short dependent kernels, so what counts in each of them is the
// number of memory round trips one behind the other: everything that does not depend on another load is requested at the start.
#include "plain_common.h"

namespace hyp {

namespace {

// The sum over the wave's four rows of 16 lanes of four registers: row rho of the result holds register quad_reg(rho).
// v_permlane32_swap / v_permlane16_swap exchange halves (odd and even rows) of two registers, so three exchanges and three
// additions do what eight shuffles would, and no lane repeats another.
__device__ __forceinline__ int quad_reg(int rho) { return (rho >> 1) | ((rho & 1) << 1); }
__device__ __forceinline__ float rows_sum4(f32x4 v) {
  auto add32 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  const float lo = add32(v[0], v[1]), hi = add32(v[2], v[3]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ----------------------------------------------------------------------------
// out^T[N, rows] = W[N, K] X[rows, K]^T for up to TB token columns, the epilogues as for prompts (plain_epilogue).
//
// A workgroup owns 16 features; its KW waves take the tiles along K in turn, up to U of them requested at once, and meet in
// LDS, in wave order.  Behind the first tiles follow the sums of squares (a KW-th of them per wave, combined in LDS with the
// products) and what the epilogue needs, so that a workgroup waits for memory once.  (When every wave added up all the sums
// of squares behind its K loop, that took 2.2 - 3.6 of the kernel's 4.8 - 5.6 us, 64 sums, 1024 wide.)
//
// Up to 8 tokens are staged through LDS, each chunk requested once per workgroup: fetched by the lanes of each wave as an MFMA
// operand the four live rows of sixteen, or four copies of them, cost as many requests as the weights (float, 4 tokens, QKV
// of 1024 x 2048: 6.1 -> 5.3 us).
//
// 4 tokens, 1024 wide, FFN 4096, two blocks (traced; before: one form of the prompt's kernel): QKV 7.7 -> 5.3 us float, 6.4 ->
// 4.7 bf16; O 5.3 -> 4.1, 4.1 -> 3.8; gate/up 9.9 -> 8.2 (4.1 TB/s), 7.5 -> 5.6; down 10.3 -> 6.7, 5.6 -> 5.0.
//
// Float with up to 8 tokens multiplies with v_mfma_f32_4x4x1_16b_f32, whose sixteen blocks are (4 rows of the tile) x (K
// group of the lane): the tile is its operand as it stands and four token columns replace sixteen, of which batch 4 would
// fill a quarter (32 against 128 cycles of the matrix pipe per KiB of weights).
// ----------------------------------------------------------------------------
constexpr int kStage = 8;  // 16-byte chunks of the tokens that a thread stages at most

// FIRST: the contraction that opens a decode step.  Its staging does the opening kernel's work - gain, rounding, sums of squares
// of 16 features, added in the same order - on the rows as the caller gives them, and its epilogue leaves the tokens' rotary
// angles for the blocks behind; the first residual epilogue takes the residual from the caller's rows.  A launch less per step:
// 1.7 - 3 us on the device and 2.5 on the host.
template <typename T, int EPI, int TB, int KW, bool FIRST>
__global__ void __launch_bounds__(KW * 64) __attribute__((amdgpu_waves_per_eu(FIRST && KW == 8 ? 2 : 4))) k_plain_gemv(GemmArgs<T> a) {
  constexpr bool kStaged = TB <= 8, kQuads = kStaged && sizeof(T) == 4;
  constexpr int NB = kStaged ? 1 : TB / 16;   // 16-token blocks
  constexpr int NX = kQuads ? TB / 4 : NB;    // token operands: quads, or 16-token blocks
  constexpr int NA = kQuads ? 2 : 1;          // accumulator chains of an operand
  constexpr int U = NB == 1 ? 8 : 4, kSsq = 4;  // registers: four waves per SIMD
  extern __shared__ __attribute__((aligned(16))) u32x4 x_s[];  // staged tokens: [tile][4][TB]
  const PlainGemm<T> &g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, tl = lane & 15, row = lane >> 4;
  const int ft = blockIdx.x;
  const bool finisher = wave < NB;  // this wave runs the epilogue of token block `wave`
  PlainAhead<T> pf;

  const int chunks = a.tiles * 4 * TB, n_stage = (chunks + KW * 64 - 1) / (KW * 64);
  // sixteen waves have 128 registers each: rows and gain of all eight chunks of a thread would not fit beside the tiles (18
  // spilled in bf16), so the second four, which only more than 4096 chunks need, are requested behind the first
  constexpr int kHeld = FIRST && KW == 16 ? kStage / 2 : kStage;
  u32x4 st[kStaged ? kHeld : 1], st_gain[FIRST ? kHeld : 1];
  constexpr int E = plain_chunk<T>();
  auto request = [&](int i0) {
#pragma unroll
    for (int i = 0; i < kHeld; ++i)
      if (i0 + i < n_stage) {
        const int c = min((int)threadIdx.x + (i0 + i) * KW * 64, chunks - 1);
        if constexpr (FIRST) {
          const int k = c / TB * E, r = c % TB;
          st[i] = st_gain[i] = u32x4{0, 0, 0, 0};  // no such row, or padding along K
          if (k < g.K && r < g.rows) {
            st[i] = *(const u32x4 *)(g.first_in + (size_t)r * g.K + k);
            st_gain[i] = *(const u32x4 *)(g.first_gain + k);
          }
        } else {
          st[i] = ((const u32x4 *)g.X)[(c / TB) * 16 + c % TB];
        }
      }
  };
  if constexpr (kStaged) request(0);
  const int tile0 = min(wave, a.tiles - 1);  // a wave without a tile rereads the last one and uses nothing
  const u32x4 *wp = (const u32x4 *)g.W + ((size_t)ft * a.tiles + tile0) * 64 + lane;
  const u32x4 *xp[NX];
#pragma unroll
  for (int j = 0; j < NX; ++j)
    xp[j] = kStaged ? x_s + (wave * 4 + row) * TB + (kQuads ? (lane & 3) + 4 * j : tl % TB)
                    : (const u32x4 *)g.X + ((size_t)min(j, a.tt - 1) * a.tiles + tile0) * 64 +
                          (j * 16 + tl < g.rows ? lane : lane & 48);  // no token: the block's first again
  constexpr int kXStep = KW * (kStaged ? 4 * TB : 64);
  u32x4 wf[U], xf[kStaged ? 1 : NX][kStaged ? 1 : U];
  f32x4 acc[NX][NA];
#pragma unroll
  for (int j = 0; j < NX; ++j)
#pragma unroll
    for (int c = 0; c < NA; ++c) acc[j][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int u, int i) {
    wf[u] = wp[(size_t)i * KW * 64];
    if constexpr (!kStaged)
#pragma unroll
      for (int j = 0; j < NX; ++j) xf[j][u] = xp[j][(size_t)i * kXStep];
  };
  auto use = [&](int u, int i) {
    u32x4 x[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j)
      if constexpr (kStaged) x[j] = xp[j][i * kXStep];
      else x[j] = xf[j][u];
#pragma unroll
    for (int e = 0; e < kMmaSteps<T>; ++e)
#pragma unroll
      for (int j = 0; j < NX; ++j) {
        if constexpr (kQuads)
          acc[j][e % NA] = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(wf[u][e]), __uint_as_float(x[j][e]), acc[j][e % NA], 0, 0, 0);
        else acc[j][0] = mma<T>(wf[u], x[j], acc[j][0], e);
      }
  };
  // sums of squares of this wave's share of the parts, lane = (token, part modulo 4)
  constexpr bool kNorm = EPI == PLAIN_QKV || EPI == PLAIN_SWIGLU;
  float sq[NB][kSsq];
  float *ps = (float *)(x_s + n_stage * KW * 64);  // FIRST: the sums of squares, [part][TB]
  const float *ssq = g.ssq_in + (size_t)(wave * 4 + row) * g.rows_pad + tl;
  // what follows the first tiles' requests
  auto early = [&] {
    if constexpr (kNorm && !FIRST) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < kSsq; ++i)
          sq[j][i] = wave * 4 + row + i * 4 * KW < g.ssq_parts ? ssq[(size_t)i * 4 * KW * g.rows_pad + min(j, a.tt - 1) * 16] : 0.f;
    }
    if (finisher) plain_fetch<T, EPI>(pf, g, wave * 16 + tl, ft * 16 + row * 4);
    if constexpr (kStaged) {
      auto stage = [&](int i0) {
#pragma unroll
        for (int i = 0; i < kHeld; ++i)
          if (i0 + i < n_stage) {
            const int c = threadIdx.x + (i0 + i) * KW * 64;
            if constexpr (FIRST) {
              union { u32x4 v; T e[E]; } x, w;
              x.v = st[i]; w.v = st_gain[i];
              float q[E / 4];
              {
#pragma clang fp contract(off)
#pragma unroll
                for (int h = 0; h < E / 4; ++h) {
                  float s[4];
#pragma unroll
                  for (int e = 0; e < 4; ++e) { const float f = load_f32(&x.e[4 * h + e]); s[e] = f * f; }
                  q[h] = (s[0] + s[1]) + (s[2] + s[3]);
                }
                // 16 features: the lanes of four (float) or two (bf16) neighbouring chunks of the row
                float s = E == 4 ? q[0] : q[0] + q[E / 4 - 1];
                s += TB == 4 ? lane_on<4>(s) : lane_round<8>(s);
                if (E == 4) {
                  if (TB == 4) s += lane_round<8>(s);
                  else { const LanePair r = both_rows(s); s = r.a + r.b; }
                }
                const int chunk = c / TB, per = 16 / E;
                if (c < chunks && chunk % per == 0) ps[chunk / per * TB + c % TB] = s;
              }
#pragma unroll
              for (int e = 0; e < E; ++e) store_f32(&x.e[e], load_f32(&x.e[e]) * load_f32(&w.e[e]));
              st[i] = x.v;
            }
            x_s[c] = st[i];
          }
      };
      stage(0);
      if (kHeld < kStage && n_stage > kHeld) {
        request(kHeld);
        stage(kHeld);
      }
      __syncthreads();
      if constexpr (FIRST)
#pragma unroll
        for (int i = 0; i < kSsq; ++i) {
          const int p = wave * 4 + row + i * 4 * KW;
          sq[0][i] = p < g.ssq_parts ? ps[p * TB + tl % TB] : 0.f;
        }
    }
  };
  const int n = (a.tiles - wave + KW - 1) / KW;  // this wave's tiles: wave, wave + KW, ...
  // Full windows: a tile's registers are refilled as soon as it has gone through the MFMAs.  The first window is requested
  // without a condition (past the end: the first tile again), so that each wait is for one tile only.
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (U == 4 || u < 4) load(u, u < n ? u : 0);
    else if (u < n) load(u, u);
  early();
  int t = 0;
  for (; t + 2 * U <= n; t += U)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      use(u, t + u);
      load(u, t + U + u);
    }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (t + u < n) {
      use(u, t + u);
      if (t + U + u < n) load(u, t + U + u);
    }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (t + U + u < n) use(u, t + U + u);

  // [wave][operand]: 16 features x 16 tokens as the epilogue's lanes hold them, or x 4 tokens
  __shared__ float red[KW][NX][kQuads ? 64 : 256];
  __shared__ float sq_s[KW][NB][16];
#pragma unroll
  for (int j = 0; j < NX; ++j) {
    if constexpr (kQuads) {
      f32x4 s = acc[j][0];
#pragma unroll
      for (int c = 1; c < NA; ++c) s += acc[j][c];
      red[wave][j][tl * 4 + quad_reg(row)] = rows_sum4(s);  // rows 4 (tl / 4) .. + 3 of token tl % 4
    } else {
      *(f32x4 *)&red[wave][j][lane * 4] = acc[j][0];
    }
  }
  if constexpr (kNorm) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float s = (sq[j][0] + sq[j][1]) + (sq[j][2] + sq[j][3]);
      for (int p = wave * 4 + row + kSsq * 4 * KW; p < g.ssq_parts; p += 4 * KW)
        s += FIRST ? ps[p * TB + tl % TB] : g.ssq_in[(size_t)p * g.rows_pad + min(j, a.tt - 1) * 16 + tl];
      s = rows_sum(s);
      if (lane < 16) sq_s[wave][j][lane] = s;
    }
  }
  __syncthreads();
  if (finisher) {
    const float *src = kQuads ? &red[0][NX == 1 ? 0 : (tl >> 2) & 1][(row * 4 + (tl & 3)) * 4] : &red[0][wave][lane * 4];
    constexpr int kStride = NX * (kQuads ? 64 : 256);
    f32x4 sum = *(const f32x4 *)src;
#pragma unroll
    for (int w = 1; w < KW; ++w) sum += *(const f32x4 *)(src + w * kStride);
    float rs = 1.f;
    if constexpr (kNorm) {
      float s = sq_s[0][wave][tl];
#pragma unroll
      for (int w = 1; w < KW; ++w) s += sq_s[w][wave][tl];
      rs = 1.0f / sqrtf(s * a.inv_K + g.eps);
    }
    plain_epilogue<T, EPI, true>(g, a.out_tiles, ft, wave * 16 + tl, row * 4, sum, rs, pf);
  }
  if (EPI == PLAIN_FINAL && g.lens_advance && blockIdx.x == 0 && (int)threadIdx.x < g.rows) g.lens_advance[threadIdx.x] += 1;
}

// ----------------------------------------------------------------------------
// Attention of one new token per request.  A workgroup owns four query heads of a KV head (or a share of their keys); its KW
// waves take the 16-key blocks in turn.  Four heads are the columns of v_mfma_f32_4x4x1_16b_f32, whose sixteen blocks are
// (4 keys or features of a tile) x (16-byte chunk of the lane), so key and value tiles are operands as they lie in the cache
// and no column is padding for a group of four; sixteen columns, of which a group of two fills an eighth, kept the matrix
// pipe busy for 4 times as long and bounded the kernel (4 requests x 4 KV heads of 2 x 128 features in float, 536 keys: 9.8 us
// and a merging launch of 2.9, now 10.7 without one; bf16, 64 features: 9.4 -> 6.8).  Larger groups read the cache once for
// every four heads, which costs less than the columns did (16 heads to a KV head, 4 requests of 4000 keys, 128 features: a block
// 41.9 -> 31.9 us in bf16, 63.2 -> 36.9 in float).  bf16 scores take v_mfma_f32_16x16x32_bf16 with the four heads repeated over its sixteen columns.  Online
// softmax, probabilities and their products with the values in fp32 for either storage type; the waves' (max, sum, output)
// meet in LDS, in wave order.
// ----------------------------------------------------------------------------
// NF: 16-feature blocks the registers hold, a multiple of what d needs
// FULL: the head size fills them, so that no access is under a condition
// NV: blocks of them whose values this workgroup takes, of part `part`; fewer than NF: with FULL only
template <typename T, int NF, int NV, int KW, bool FULL>
__device__ __forceinline__ void plain_dec_attn(const AttnArgs<T> &a, int col0, int part) {
  static_assert(NV == NF || FULL, "parts of a head that fills its registers");
  constexpr int NC = NF * (int)sizeof(T) / 4;  // K tiles: 16 floats or 32 bf16 each
  constexpr int kSets = NF <= 8 ? 2 : 1;       // blocks of a wave in flight or in use
  extern __shared__ __attribute__((aligned(16))) f32x4 o_s[];  // [KW][nv][64]
  __shared__ float m_s[KW][4], l_s[KW][4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, row = lane >> 4, g4 = row * 4;
  const int d = FULL ? NF * 16 : a.cache.d, nf = (d + 15) / 16, nv = NV < NF ? NV : nf, f0 = part * NV, nc = plain_tiles(d, sizeof(T));
  const int req = blockIdx.x / a.split, share = blockIdx.x % a.split, kvh = blockIdx.y;
  const int col = col0 + (lane & 3), head = kvh * a.G + min(col, a.G - 1);  // this lane's column
  const int last = a.lens[req];
  const u32x4 *kp = (const u32x4 *)(a.Kc + ((size_t)req * a.cache.nkv + kvh) * a.cache.k_elems(sizeof(T))) + lane;
  const T *vp = a.Vc + ((size_t)req * a.cache.nkv + kvh) * a.cache.v_elems() + lane * 4;
  const u32x4 *qp = (const u32x4 *)(a.q + ((size_t)req * a.nq + head) * a.q_ld) + row;
  const int first = share * KW + wave, step = a.split * KW;
  u32x4 kS[kSets][NC], qf[NC];
  typename VRaw<T>::V vS[kSets][NV];
  auto load = [&](u32x4 (&k)[NC], typename VRaw<T>::V (&v)[NV], int kb) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) k[c] = kp[((size_t)kb * nc + c) * 64];
#pragma unroll
    for (int f = 0; f < NV; ++f)
      if (f < nv) v[f] = *(const typename VRaw<T>::V *)(vp + ((size_t)kb * nf + f0 + f) * 256);
  };
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c < nc) qf[c] = qp[c * 4];
  // before the context's length is known: the request's room bounds what may be read
  load(kS[0], vS[0], min(first, a.cache.key_blocks - 1));
  f32x4 o[NV];
#pragma unroll
  for (int f = 0; f < NV; ++f) o[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const int n_kb = (last >> 4) + 1;
  auto block = [&](u32x4 (&kf)[NC], typename VRaw<T>::V (&v)[NV], int kb) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, s1 = s;  // two chains
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc)
#pragma unroll
        for (int e = 0; e < kMmaSteps<T>; ++e) {
          f32x4 &to = (c * kMmaSteps<T> + e) & 1 ? s1 : s;
          if constexpr (sizeof(T) == 4) to = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(kf[c][e]), __uint_as_float(qf[c][e]), to, 0, 0, 0);
          else to = mma<T>(kf[c], qf[c], to, e);
        }
    s += s1;
    f32x4 vf[NV];
#pragma unroll
    for (int f = 0; f < NV; ++f)
      if (f < nv) vf[f] = widen_v4<T>(v[f]);
    const bool edge = kb == n_kb - 1;  // the only block with slots past the last key
    float p[4], mx = -INFINITY;
    if constexpr (sizeof(T) == 4) {
      // a lane's score is that of one key: 4 ((lane / 4) % 4) + quad_reg(row)
      p[0] = rows_sum4(s) * a.scale;
      if (edge && kb * 16 + (lane & 12) + quad_reg(row) > last) p[0] = -INFINITY;
      mx = fmaxf(p[0], lane_round<8>(p[0]));
      mx = fmaxf(mx, lane_round<4>(mx));
    } else {
      // a lane's scores are those of keys 4 row .. + 3
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[i] = s[i] * a.scale;
        if (edge && kb * 16 + g4 + i > last) p[i] = -INFINITY;
        mx = fmaxf(mx, p[i]);
      }
    }
    mx = rows_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float ref = m_new == -INFINITY ? 0.f : m_new;
    const float corr = expf(m_run - ref);
    m_run = m_new;
    if constexpr (sizeof(T) == 4) {
      const float w = expf(p[0] - ref);
      l_run = l_run * corr + w;
      // keys 4 row .. + 3 of this lane's head
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = __shfl(w, (((i >> 1) | ((i & 1) << 1)) << 4) | g4 | (lane & 3), 64);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = expf(p[i] - ref);
      l_run = l_run * corr + ((p[0] + p[1]) + (p[2] + p[3]));
    }
#pragma unroll
    for (int f = 0; f < NV; ++f) o[f] *= corr;
    if (edge)
      // slots past the last cached key hold anything: no product may meet them
#pragma unroll
      for (int f = 0; f < NV; ++f)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (f < nv && kb * 16 + g4 + i > last) vf[f][i] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int f = 0; f < NV; ++f)
        if (f < nv) o[f] = __builtin_amdgcn_mfma_f32_4x4x1f32(vf[f][i], p[i], o[f], 0, 0, 0);
  };
  if constexpr (kSets == 2) {
    load(kS[1], vS[1], min(first + step, n_kb - 1));  // past the end: the last block again, not used
    for (int kb = first; kb < n_kb; kb += 2 * step) {
      block(kS[0], vS[0], kb);
      if (kb + step >= n_kb) break;
      load(kS[0], vS[0], min(kb + 2 * step, n_kb - 1));
      block(kS[1], vS[1], kb + step);
      load(kS[1], vS[1], min(kb + 3 * step, n_kb - 1));
    }
  } else {
    for (int kb = first; kb < n_kb; kb += step) {
      block(kS[0], vS[0], kb);
      load(kS[0], vS[0], min(kb + step, n_kb - 1));
    }
  }
  // The lane's places once more, from an opaque copy: kept over the loop they took the float form of 65 - 127 features past 256
  // registers (8 spilled; 8 requests of 1500 keys, 80 features: a block 41.1 -> 40.1 us) and that of 128 to 250 (195 now).  Wider
  // heads have registers to spare, and in float took 2 - 3 % longer this way.
  int at = lane;
  if constexpr (NF <= 8) asm volatile("" : "+v"(at));
  // sum of the probabilities over the lanes that hold different keys
  if constexpr (sizeof(T) == 4) {
    l_run += lane_round<8>(l_run);
    l_run += lane_round<4>(l_run);
  }
  l_run = rows_sum(l_run);
  if (at < 4) { m_s[wave][at] = m_run; l_s[wave][at] = l_run; }
#pragma unroll
  for (int f = 0; f < NV; ++f)
    if (f < nv) o_s[(wave * nv + f) * 64 + at] = o[f];
  __syncthreads();
  const int c = at & 3;
  float m = m_s[0][c];  // -inf: a share without a key, whose weights and sums are 0
#pragma unroll
  for (int w = 1; w < KW; ++w) m = fmaxf(m, m_s[w][c]);
  float wgt[KW], l = 0.f;
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    wgt[w] = m_s[w][c] == -INFINITY ? 0.f : expf(m_s[w][c] - m);
    l += wgt[w] * l_s[w][c];
  }
  const int col_at = col0 + c, head_at = kvh * a.G + min(col_at, a.G - 1);
  for (int f = wave; f < nv; f += KW) {
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; ++w)
      r += o_s[(w * nv + f) * 64 + at] * wgt[w];  // zeros of a share without a key
    const float v = rows_sum4(r);  // the rows hold the sums over different keys
    const int feat = (f0 + f) * 16 + (at & 12) + quad_reg(at >> 4);
    if (col_at >= a.G || feat >= d) continue;
    if (a.split > 1) {
      float *dst = a.part + (((size_t)req * a.nq + head_at) * a.split + share) * (2 + d);
      if (feat == 0) { dst[0] = m; dst[1] = l; }
      dst[2 + feat] = v;
    } else {
      store_f32(a.out + plain_offset<T>(req, head_at * d + feat, a.out_tiles), v / l);
    }
  }
}

template <typename T, int NF, int KW, bool FULL>
__global__ void __launch_bounds__(KW * 64) k_plain_dec_attn(AttnArgs<T> a) {
  plain_dec_attn<T, NF, NF, KW, FULL>(a, blockIdx.z * 4, 0);
}

// A few heads of a short context: each in PARTS workgroups, which all form the head's probabilities and take a share of the value
// features.  A CU takes 64 bytes a clock, so one of 16 workgroups (4 requests, 4 KV heads) needs 3.6 us for the 536 float keys and
// values of 128 features alone; nothing has to be merged.  (That kernel: 10.1 us in one part, 8.1 in two, 7.3 in four; bf16 of 64
// features 6.8, 6.2, 6.0; float of 64 features, one request of 80 keys, 2 heads: 3.7, 3.6, 4.4.)
template <typename T, int NF, int PARTS, int KW>
__global__ void __launch_bounds__(KW * 64) k_plain_dec_attn_parts(AttnArgs<T> a) {
  plain_dec_attn<T, NF, NF / PARTS, KW, true>(a, blockIdx.z / PARTS * 4, blockIdx.z % PARTS);
}

// one workgroup per (head, request): the shares of a split decode attention in order
// (a thread per feature; everything is requested before the first value is used)
template <typename T> __global__ void __launch_bounds__(256) k_plain_attn_merge(AttnArgs<T> a) {
  const int head = blockIdx.x, req = blockIdx.y, d = a.cache.d, f = min((int)threadIdx.x, d - 1);
  const float *src = a.part + ((size_t)req * a.nq + head) * a.split * (2 + d);
  float ms[kPlainMaxSplit], ls[kPlainMaxSplit], os[kPlainMaxSplit];
#pragma unroll
  for (int s = 0; s < kPlainMaxSplit; ++s) {
    const float *p = src + min(s, a.split - 1) * (2 + d);
    ms[s] = p[0]; ls[s] = p[1]; os[s] = p[2 + f];
  }
  float m = ms[0];
#pragma unroll
  for (int s = 1; s < kPlainMaxSplit; ++s) m = fmaxf(m, ms[s]);  // slots past the last repeat it
  float l = 0.f, o = 0.f;
#pragma unroll
  for (int s = 0; s < kPlainMaxSplit; ++s) {
    const float w = s >= a.split || ms[s] == -INFINITY ? 0.f : expf(ms[s] - m);
    if (s < a.split) { l += w * ls[s]; o += w * os[s]; }
  }
  if ((int)threadIdx.x < d) store_f32(a.out + plain_offset<T>(req, head * d + f, a.out_tiles), o / l);
}

}  // namespace

// groups of four query heads per KV head
static int column_groups(const Dims &dm) { return (dm.nq / dm.nkv + 3) / 4; }

// Where every CU holds one workgroup at most and eight waves would take more than one round of loads, sixteen share K.
static int gemv_threads(int ft, int tiles) { return ft <= 256 && tiles > 64 ? 1024 : 512; }
// token columns that are staged in LDS: up to 8 rows, as long as their copy is at most 128 KiB and kStage chunks a thread; 0: none
static int gemv_staged(int rows, int ft, int tiles) {
  for (int tb = 4; tb <= 8; tb += 4)
    if (rows <= tb && tiles * 4 * tb <= std::min(kStage * gemv_threads(ft, tiles), 8192)) return tb;
  return 0;
}

// LDS of the staged tokens: whole rounds of the threads; with `first` up to two sums of squares a tile and token behind them
static size_t gemv_lds(int threads, int tiles, int tb, bool first) {
  return (size_t)(tiles * 4 * tb + threads - 1) / threads * threads * 16 + (first ? sizeof(float) * tb * tiles * 2 : 0);
}
constexpr size_t kGemvMaxLds = 8192 * 16;

template <typename T> bool plain_gemv_opens(const T *hidden_in, int rows, int N, int K) {
  const int ft = (N + 15) / 16, tiles = plain_tiles(K, sizeof(T)), tb = gemv_staged(rows, ft, tiles);
  return tb != 0 && gemv_lds(gemv_threads(ft, tiles), tiles, tb, true) <= kGemvMaxLds && K % plain_chunk<T>() == 0 && (uintptr_t)hidden_in % 16 == 0;
}

template <typename T, int EPI, bool FIRST>
static hipError_t launch_gemv(const PlainGemm<T> &g, hipStream_t s) {
  GemmArgs<T> a = gemm_args<T, EPI>(g);
  const int threads = gemv_threads(a.ft, a.tiles), tb = gemv_staged(g.rows, a.ft, a.tiles);
  const size_t lds = gemv_lds(threads, a.tiles, tb, FIRST);
#define X(TB, LDS, F)                                                        \
  {                                                                          \
    if (threads == 1024) k_plain_gemv<T, EPI, TB, 16, F><<<a.ft, 1024, LDS, s>>>(a); \
    else k_plain_gemv<T, EPI, TB, 8, F><<<a.ft, 512, LDS, s>>>(a);           \
    return hipGetLastError();                                                \
  }
  if (tb == 4) X(4, lds, FIRST)
  if (tb == 8) X(8, lds, FIRST)
  if (FIRST) return hipErrorInvalidValue;
  if (g.rows <= 16) X(16, 0, false)
  X(32, 0, false)
#undef X
}

template <typename T> hipError_t plain_gemv(int epi, const PlainGemm<T> &g, hipStream_t s) {
  if (g.rows == 0) return hipSuccess;
  if (g.rows > kPlainGemvRows) return hipErrorInvalidValue;
  switch (epi) {
    case PLAIN_QKV: return g.first_in ? launch_gemv<T, PLAIN_QKV, true>(g, s) : launch_gemv<T, PLAIN_QKV, false>(g, s);
    case PLAIN_SWIGLU: return launch_gemv<T, PLAIN_SWIGLU, false>(g, s);
    case PLAIN_RESID: return launch_gemv<T, PLAIN_RESID, false>(g, s);
    case PLAIN_FINAL: return launch_gemv<T, PLAIN_FINAL, false>(g, s);
  }
  return hipErrorInvalidValue;
}

// (register blocks, waves): enough for d features; the waves' outputs pass 64 KiB of LDS at 8 waves of 128 features and more
#define HYP_PLAIN_ATTN(X) X(4, 8, true) X(8, 8, true) X(4, 8, false) X(8, 8, false) X(16, 4, false)

hipError_t plain_decode_init() {
  hipError_t e = hipSuccess;
#define X(T, EPI, TB, KW, FIRST) \
  if (e == hipSuccess)           \
    e = hipFuncSetAttribute((const void *)k_plain_gemv<T, EPI, TB, KW, FIRST>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemvMaxLds);
#define Y(T, TB, KW)                                                                                                    \
  X(T, PLAIN_QKV, TB, KW, false) X(T, PLAIN_QKV, TB, KW, true) X(T, PLAIN_SWIGLU, TB, KW, false) X(T, PLAIN_RESID, TB, KW, false) \
  X(T, PLAIN_FINAL, TB, KW, false)
  Y(float, 4, 8) Y(float, 4, 16) Y(float, 8, 8) Y(float, 8, 16) Y(bf16_t, 4, 8) Y(bf16_t, 4, 16) Y(bf16_t, 8, 8) Y(bf16_t, 8, 16)
#undef Y
#undef X
#define X(NF, KW, FULL)                                                                                                              \
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_plain_dec_attn<float, NF, KW, FULL>, hipFuncAttributeMaxDynamicSharedMemorySize, NF * KW * 1024);  \
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_plain_dec_attn<bf16_t, NF, KW, FULL>, hipFuncAttributeMaxDynamicSharedMemorySize, NF * KW * 1024);
  HYP_PLAIN_ATTN(X)
#undef X
  return e;
}

// a split of c needs batch * heads in flight * c <= kPlainSplitGroups: so many shares of all requests together
size_t plain_attn_part_floats(const Dims &dm, int batch) {
  const size_t per_request = (size_t)dm.nkv * column_groups(dm);
  return std::min((size_t)batch * kPlainMaxSplit, kPlainSplitGroups / per_request) * dm.nq * (2 + dm.d);
}

template <typename T>
hipError_t plain_attn_decode(const T *q, int q_ld, const T *Kc, const T *Vc, T *out, const int *lens, int batch, int longest,
                             float *part, const PlainCache &cache, const Dims &dm, hipStream_t s) {
  if (batch == 0) return hipSuccess;
  AttnArgs<T> a = attn_args<T>(q, q_ld, Kc, Vc, out, cache, dm);
  a.lens = lens; a.part = part;
  const int groups = column_groups(dm), nf = (dm.d + 15) / 16, nc = plain_tiles(dm.d, sizeof(T));
  a.split = plain_attn_split((int)sizeof(T), dm.d, (size_t)batch * dm.nkv * groups, longest);
  const int parts = plain_attn_parts(dm.d, (size_t)batch * dm.nkv * groups, a.split);
  if (parts > 1) {
    const dim3 grid(batch, dm.nkv, groups * parts);
    if (dm.d == 64) k_plain_dec_attn_parts<T, 4, 2, 8><<<grid, 8 * 64, 8 * 2 * 1024, s>>>(a);
    else k_plain_dec_attn_parts<T, 8, 4, 8><<<grid, 8 * 64, 8 * 2 * 1024, s>>>(a);
    return hipGetLastError();
  }
  const dim3 grid(batch * a.split, dm.nkv, groups);
  const int nf_tiles = nc * 4 / (int)sizeof(T);
  hipError_t e = hipErrorInvalidValue;
#define X(NF, KW, FULL)                                                                    \
  if (e == hipErrorInvalidValue && (FULL ? dm.d == NF * 16 : nf_tiles <= NF)) {      \
    k_plain_dec_attn<T, NF, KW, FULL><<<grid, KW * 64, (size_t)KW * nf * 1024, s>>>(a); \
    e = hipGetLastError();                                                           \
    if (e != hipSuccess) return e;                                                   \
  }
  HYP_PLAIN_ATTN(X)
#undef X
  if (e != hipSuccess || a.split == 1) return e;
  k_plain_attn_merge<T><<<dim3(dm.nq, batch), (dm.d + 63) / 64 * 64, 0, s>>>(a);
  return hipGetLastError();
}

#define HYP_INSTANTIATE(T)                                                                                            \
  template hipError_t plain_gemv<T>(int, const PlainGemm<T> &, hipStream_t);                                          \
  template bool plain_gemv_opens<T>(const T *, int, int, int);                                                        \
  template hipError_t plain_attn_decode<T>(const T *, int, const T *, const T *, T *, const int *, int, int, float *,  \
                                           const PlainCache &, const Dims &, hipStream_t);
HYP_INSTANTIATE(float)
HYP_INSTANTIATE(bf16_t)

}  // namespace hyp
