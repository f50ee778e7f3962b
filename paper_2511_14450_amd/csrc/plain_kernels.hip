// Shape-generic HIP kernels of the decoder block (Sec. III-A of the paper): matrix-core
// contractions with fp32 accumulation on float or bf16 storage for any width, head size up to 256
// and batch.  They are the whole fp32 path and serve bf16 stages whose shape the large bf16
// kernels do not cover.
#include "plain_common.h"

namespace hyp {

namespace {

// packed row -> row of the stacked matrices.  Rows an epilogue combines sit next to each other:
// the rotary partners i, i + d/2 of every query and key head; gate and up of an FFN feature.
__device__ inline int plain_src_row(int r, int N, int mode, int d, int qk_rows) {
  if (mode == PLAIN_PAIRS_QKV && r < qk_rows) {
    const int head = r / d, w = r % d;
    return head * d + (w >> 1) + (w & 1) * (d >> 1);
  }
  if (mode == PLAIN_PAIRS_GATEUP) return (r >> 1) + (r & 1) * (N >> 1);
  return r;
}

// one thread per 16-byte chunk of the destination
template <typename T>
__global__ void __launch_bounds__(256) k_plain_pack(const T *__restrict__ src0, const T *__restrict__ src1,
                                                    const T *__restrict__ src2, int rows0, int rows1, T *__restrict__ dst,
                                                    int N, int K, int tiles, int mode, int d, int qk_rows, size_t chunks) {
  constexpr int E = plain_chunk<T>();
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t c = (size_t)blockIdx.x * 256 + threadIdx.x; c < chunks; c += stride) {
    const size_t tile = c >> 6;
    const int lane = c & 63, r = (int)(tile / tiles) * 16 + (lane & 15), k = (int)(tile % tiles) * 4 * E + (lane >> 4) * E;
    union { T e[E]; u32x4 v; } u;
    u.v = u32x4{0, 0, 0, 0};
    if (r < N) {
      const int sr = plain_src_row(r, N, mode, d, qk_rows);
      const T *s = sr < rows0 ? src0 + (size_t)sr * K : sr < rows0 + rows1 ? src1 + (size_t)(sr - rows0) * K
                                                                           : src2 + (size_t)(sr - rows0 - rows1) * K;
      if (k + E <= K && (uintptr_t)(s + k) % 16 == 0) u.v = *(const u32x4 *)(s + k);
      else
        for (int e = 0; e < E; ++e)
          if (k + e < K) u.e[e] = s[k + e];
    }
    *(u32x4 *)(dst + c * E) = u.v;
  }
}

// x = hidden_in ; residual = x ; y = x * gain -> F(rows, H) ; sum of squares per 16 features.
// grid (rows, ceil(max(H, half) / 256)); a thread per feature, 16 neighbouring lanes share a sum.  A decode step also copies
// its tokens' rotary angles next to each other: the contractions of all blocks then find them without looking at the lengths
// first (one round trip less in each).
template <typename T>
__global__ void __launch_bounds__(256) k_plain_begin(const T *__restrict__ in, float *__restrict__ xres,
                                                     const T *__restrict__ gain, T *__restrict__ y,
                                                     float *__restrict__ ssq, int H, int rows_pad, int tiles, PlainAngles ang) {
  const int f = blockIdx.y * 256 + threadIdx.x;
  const size_t row = blockIdx.x;
  float x = 0.f;
  if (ang.pos && f < ang.half) {
    const size_t from = (size_t)ang.pos[row] * ang.half + f, to = row * ang.half + f;
    ang.cos_row[to] = ang.cos_tab[from];
    ang.sin_row[to] = ang.sin_tab[from];
  }
  if (f < H) {
    x = load_f32(in + row * H + f);
    xres[row * H + f] = x;
    store_f32(y + plain_offset<T>(row, f, tiles), x * load_f32(gain + f));
  }
  // added in the order of the residual epilogue below, so that a stage that starts here gives the
  // bits of one that comes from the block before
  float s;
  {
#pragma clang fp contract(off)
    s = x * x;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
  }
  if ((threadIdx.x & 15) == 0 && f < (H + 15) / 16 * 16) ssq[(size_t)(f >> 4) * rows_pad + row] = s;
}

// ----------------------------------------------------------------------------
// out^T[N, rows] = W[N, K] X[rows, K]^T on fragment-order operands, features on the MFMA M axis:
// lane l of a 16 x 16 block holds features 4 (l / 16) .. + 3 of token l % 16 in its four registers.
//
// Two ways for the operands.  From L2 straight into registers (the first kernel below, <2, 2, 1, 1, 4>): a wave owns WM x WN
// blocks and requests U tiles of K ahead of their use, KW waves share the K loop and meet in LDS, in wave order.  No barrier in
// the loop and 32 x 32 outputs a workgroup, so it is the form of short prompts and narrow layers, whose few tiles it spreads
// over the most CUs.  Through LDS (the second kernel): 64 x 64 or 128 x 128 outputs, for everything that fills the chip with
// them.  Which one: plain_gemm_form.  More than kPlainGemvRows rows (fewer: plain_gemv).
// ----------------------------------------------------------------------------
template <typename T, int EPI, int WM, int WN, int FW, int TW, int KW>
__global__ void __launch_bounds__(FW * TW * KW * 64) k_plain_gemm(GemmArgs<T> a) {
  constexpr int U = 2;
  static_assert(KW >= WM * WN, "a wave finishes one block at most");
  const PlainGemm<T> &g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int kw = wave % KW, fw = wave / KW % FW, tw = wave / KW / FW;
  const int f_groups = (a.ft + WM * FW - 1) / (WM * FW);
  const int ft0 = ((int)(blockIdx.x % f_groups) * FW + fw) * WM, tt0 = ((int)(blockIdx.x / f_groups) * TW + tw) * WN;

  f32x4 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // tiles past the edge reread the last one; what they give is not stored
  const u32x4 *wp[WM], *xp[WN];
#pragma unroll
  for (int i = 0; i < WM; ++i) wp[i] = (const u32x4 *)g.W + (size_t)min(ft0 + i, a.ft - 1) * a.tiles * 64 + lane;
#pragma unroll
  for (int j = 0; j < WN; ++j) xp[j] = (const u32x4 *)g.X + (size_t)min(tt0 + j, a.tt - 1) * a.tiles * 64 + lane;
  u32x4 wf[2][U][WM], xf[2][U][WN];
  // this wave's tiles are kw, kw + KW, ...; a load past the end rereads the last one, which is not used
  auto load = [&](u32x4 (&w)[U][WM], u32x4 (&x)[U][WN], int t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t at = (size_t)min(t0 + u * KW, a.tiles - 1) * 64;
#pragma unroll
      for (int i = 0; i < WM; ++i) w[u][i] = wp[i][at];
#pragma unroll
      for (int j = 0; j < WN; ++j) x[u][j] = xp[j][at];
    }
  };
  auto use = [&](auto whole, u32x4 (&w)[U][WM], u32x4 (&x)[U][WN], int t0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (decltype(whole)::value || t0 + u * KW < a.tiles)
#pragma unroll
        for (int e = 0; e < kMmaSteps<T>; ++e)  // neighbouring MFMAs on different accumulators
#pragma unroll
          for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) acc[i][j] = mma<T>(w[u][i], x[u][j], acc[i][j], e);
  };
  constexpr int kStep = U * KW;
  const int tl = lane & 15, q4 = (lane >> 4) * 4;
  load(wf[0], xf[0], kw);
  // What the epilogue needs from memory is requested under the first tiles: positions, rotary angles, residual and gain of the
  // block that this wave finishes, kw / WN, kw % WN.
  PlainAhead<T> pf;
  if (kw < WM * WN) plain_fetch<T, EPI>(pf, g, (tt0 + kw % WN) * 16 + tl, (ft0 + kw / WN) * 16 + q4);
  // RMS Norm factors: the sums of squares of this wave's tokens, added up by lane groups (four parts at a time), a share of them
  // per wave, requested here, under the first tiles.  (Pairs of parts one after the other behind the loop took 4 of 14 us in
  // bf16: 1065 rows, 64 parts.)
  constexpr bool kNorm = EPI == PLAIN_QKV || EPI == PLAIN_SWIGLU;
  constexpr int kSsq = 4;
  const int row = lane >> 4;
  float sq[WN][kSsq];
  auto part = [&](int p, int j) { return p < g.ssq_parts ? g.ssq_in[(size_t)p * g.rows_pad + min(tt0 + j, a.tt - 1) * 16 + tl] : 0.f; };
  if constexpr (kNorm) {
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int i = 0; i < kSsq; ++i) sq[j][i] = part((i * KW + kw) * 4 + row, j);
  }
  // pairs of whole groups, then what is left (checked tile by tile)
  int t = kw;
  for (; t + 2 * kStep - KW < a.tiles; t += 2 * kStep) {
    load(wf[1], xf[1], t + kStep);
    use(std::true_type(), wf[0], xf[0], t);
    load(wf[0], xf[0], t + 2 * kStep);
    use(std::true_type(), wf[1], xf[1], t + kStep);
  }
  load(wf[1], xf[1], t + kStep);
  use(std::false_type(), wf[0], xf[0], t);
  use(std::false_type(), wf[1], xf[1], t + kStep);
  float rs[WN];
  if constexpr (kNorm) {
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      rs[j] = (sq[j][0] + sq[j][1]) + (sq[j][2] + sq[j][3]);
      for (int p = (kSsq * KW + kw) * 4 + row; p < g.ssq_parts; p += 4 * KW) rs[j] += part(p, j);
      rs[j] = rows_sum(rs[j]);
    }
  }

  __shared__ f32x4 red[KW][FW * TW][WM * WN][64];
  const int slot = fw + FW * tw;
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) red[kw][slot][i * WN + j][lane] = acc[i][j];
  __shared__ float sq_s[KW][FW * TW][WN][16];
  if (kNorm && lane < 16)
#pragma unroll
    for (int j = 0; j < WN; ++j) sq_s[kw][slot][j][lane] = rs[j];
  __syncthreads();
  if constexpr (kNorm)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      rs[j] = sq_s[0][slot][j][tl];
#pragma unroll
      for (int w = 1; w < KW; ++w) rs[j] += sq_s[w][slot][j][tl];
    }
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      if ((i * WN + j) % KW != kw) continue;  // block b is finished by wave b % KW
      f32x4 s = red[0][slot][i * WN + j][lane];
#pragma unroll
      for (int w = 1; w < KW; ++w) s += red[w][slot][i * WN + j][lane];
      acc[i][j] = s;
    }

  if constexpr (kNorm)
#pragma unroll
    for (int j = 0; j < WN; ++j) rs[j] = 1.0f / sqrtf(rs[j] * a.inv_K + g.eps);

#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      if ((i * WN + j) % KW != kw) continue;
      if (ft0 + i >= a.ft || tt0 + j >= a.tt) continue;  // uniform over the wave
      plain_epilogue<T, EPI, true>(g, a.out_tiles, ft0 + i, (tt0 + j) * 16 + tl, q4, acc[i][j],
                                     EPI == PLAIN_QKV || EPI == PLAIN_SWIGLU ? rs[j] : 1.f, pf);
    }
  if (EPI == PLAIN_FINAL && g.lens_advance && blockIdx.x == 0)
    for (int b = threadIdx.x; b < g.rows; b += FW * TW * KW * 64) g.lens_advance[b] += 1;
}

// The same contraction with its operands staged through LDS: WF x WT waves of WM x WN blocks side by side, KW sets of them that
// share K; NST stages of KW x KS tiles along K rotate through LDS, filled by direct global->LDS wave loads.  A tile of 1 KiB is
// read back as it lies, a lane's 16 bytes each (no bank conflicts).  Bound by the matrix pipe in float (32 cycles an MFMA of
// 2 KFLOP), by LDS and the meeting of the waves at each stage in bf16, whose products take an eighth of that: so a stage's
// fragments are read a stage ahead of its products, behind the barrier that opens the stage before.  (With the reads behind
// their own barrier: float 1000 x 1024 x 4096 in 64 x 64 82 us, as here, but bf16 19.6 against 17.2, and 128 x 128 32.2 against
// 23.8 at 1000 x 8192 x 1024.)
//   <2, 2, 2, 2, 2, 1, 4>  64 x 64, two sets of four waves: 1000 x 1024 x 4096 bf16 26.5 us from registers, 17.2; float 91, 82
//   <2, 4, 4, 2, 1, 1, 4>  128 x 128 bf16: 1000 x 8192 x 1024 33.3 us from registers (as 128 x 128 of four waves), 23.8 = 720
//                          TFLOP/s; 4000 x 17920 x 5120 1098, 862 = 850
//   <4, 4, 2, 2, 1, 1, 3>  the same in four waves, three workgroups to a CU: 4600 x 4192 x 664 45.3 us in the form above, 42.0;
//                          4000 x 4480 x 5120 323, 316; with one or two workgroups to a CU slower (800 x 4688 x 600: 15.1, 16.1)
//   <2, 4, 4, 2, 1, 2, 2>  128 x 128 float, two tiles along K a stage: 800 x 8192 x 1024 157 us from registers, 143; 4000 x 17920 x
//                          5120 6215, 5730 = 128 TFLOP/s; with one tile a stage 166, 6461
template <typename T, int EPI, int WM, int WN, int WF, int WT, int KW, int KS, int NST>
__global__ void __launch_bounds__(WF * WT * KW * 64) __attribute__((amdgpu_waves_per_eu(2))) k_plain_gemm(GemmArgs<T> a) {
  constexpr int FT = WM * WF, TT = WN * WT, WAVES = WF * WT * KW, TPS = KW * KS, LPW = (FT + TT) * TPS / WAVES, STAGE = (FT + TT) * TPS * 1024;
  static_assert(LPW * WAVES == (FT + TT) * TPS, "every wave issues the same number of loads");
  typedef __attribute__((address_space(3))) void lds_t;
  typedef __attribute__((address_space(1))) const void gbl_t;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  const PlainGemm<T> &g = a.g;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, tl = lane & 15, q4 = (lane >> 4) * 4;
  const int kw = wave % KW, fw = wave / KW % WF, tw = wave / KW / WF;
  const int f_groups = (a.ft + FT - 1) / FT, ft0 = (int)(blockIdx.x % f_groups) * FT, tt0 = (int)(blockIdx.x / f_groups) * TT;
  const int steps = (a.tiles + TPS - 1) / TPS;

  f32x4 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // wave load i of a stage: tile `blk` of the workgroup (features, then tokens), the stage's `lk`-th along K; past an edge the
  // last tile again, whose products are not stored (features, tokens) or not formed (K)
  const char *src[LPW];
  int lk[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int lid = wave * LPW + i, blk = lid % (FT + TT);
    lk[i] = lid / (FT + TT);
    src[i] = (blk < FT ? (const char *)g.W + (size_t)min(ft0 + blk, a.ft - 1) * a.tiles * 1024
                       : (const char *)g.X + (size_t)min(tt0 + blk - FT, a.tt - 1) * a.tiles * 1024) + lane * 16;
  }
  auto issue = [&](int step, int buf) {  // buf: byte offset of the stage's buffer
#pragma unroll
    for (int i = 0; i < LPW; ++i)
      __builtin_amdgcn_global_load_lds((gbl_t *)(src[i] + (size_t)min(step * TPS + lk[i], a.tiles - 1) * 1024),
                                       (lds_t *)(lds + buf + (wave * LPW + i) * 1024), 16, 0, 0);
  };
#pragma unroll
  for (int s = 0; s < NST; ++s) issue(s, s * STAGE);
  // sums of squares of the workgroup's tokens, while the first stages arrive: [interleaved parts][token]
  constexpr bool kNorm = EPI == PLAIN_QKV || EPI == PLAIN_SWIGLU;
  constexpr int kToks = TT * 16, kParts = WAVES * 64 / kToks;
  __shared__ float sq_s[kNorm ? kParts : 1][kToks];
  if constexpr (kNorm) {
    const int tok = threadIdx.x % kToks, p0 = threadIdx.x / kToks;
    const float *from = g.ssq_in + min(tt0 * 16 + tok, a.tt * 16 - 1);
    float s = 0.f;
    for (int p = p0; p < g.ssq_parts; p += 8 * kParts) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p + u * kParts < g.ssq_parts ? from[(size_t)(p + u * kParts) * g.rows_pad] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    sq_s[p0][tok] = s;
  }
  const char *wbase = lds + (kw * KS * (FT + TT) + fw * WM) * 1024 + lane * 16, *xbase = lds + (kw * KS * (FT + TT) + FT + tw * WN) * 1024 + lane * 16;
  u32x4 w[2][KS][WM], x[2][KS][WN];
  auto read = [&](auto which, int at) {
    constexpr int W = decltype(which)::value;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
#pragma unroll
      for (int i = 0; i < WM; ++i) w[W][k][i] = *(const u32x4 *)(wbase + at + (k * (FT + TT) + i) * 1024);
#pragma unroll
      for (int j = 0; j < WN; ++j) x[W][k][j] = *(const u32x4 *)(xbase + at + (k * (FT + TT) + j) * 1024);
    }
  };
  // all loads but those of the youngest NST - 1 stages have landed (vmcnt), all LDS accesses are done (lgkmcnt 0)
  constexpr auto wait_for = [](int loads) { return 0x0070 | (loads & 15) | ((loads >> 4) << 14); };
  static_assert((NST - 1) * LPW < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt(wait_for((NST - 1) * LPW));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  read(std::integral_constant<int, 0>(), 0);
  int at = 0;
  // One stage: its fragments are in registers, and behind the barrier the next one's have landed everywhere and this one's buffer
  // is nobody's any more.
  auto stage = [&](auto which, int s) {
    constexpr int W = decltype(which)::value;
    __builtin_amdgcn_s_waitcnt(wait_for((NST - 2) * LPW));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int next = at + STAGE == NST * STAGE ? 0 : at + STAGE;
    read(std::integral_constant<int, W ^ 1>(), next);
    issue(s + NST, at);  // past the end: the last tiles again, in a buffer nobody reads
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < KS; ++k)
      if (TPS == 1 || s * TPS + kw * KS + k < a.tiles)
#pragma unroll
        for (int e = 0; e < kMmaSteps<T>; ++e)
#pragma unroll
          for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int i = 0; i < WM; ++i) acc[i][j] = mma<T>(w[W][k][i], x[W][k][j], acc[i][j], e);
    at = next;
  };
  // Float sums are taken out of the accumulators every kRun stages, so that no chain of additions is longer than 256 products.
  // (Two 1024-wide blocks, FFN 4096, against 64 bits: 2.1e-6 in one chain, 1.0e-6 so, 1.7e-6 in the register form's four.)
  constexpr int kRun = sizeof(T) == 4 ? 8 : 0;
  f32x4 sum[kRun != 0 ? WM : 1][kRun != 0 ? WN : 1] = {};
  auto take_out = [&] {
    if constexpr (kRun != 0)
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
          sum[i][j] += acc[i][j];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
  };
  int s = 0;
  for (; s + 2 <= steps; s += 2) {
    stage(std::integral_constant<int, 0>(), s);
    stage(std::integral_constant<int, 1>(), s + 1);
    if (kRun != 0 && (s + 2) % kRun == 0) take_out();
  }
  if (s < steps) stage(std::integral_constant<int, 0>(), s);
  if constexpr (kRun != 0)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) acc[i][j] += sum[i][j];
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the loads past the end have landed
  if constexpr (KW > 1) {
    __syncthreads();
    f32x4 (*red)[WF * WT][WM * WN][64] = (f32x4 (*)[WF * WT][WM * WN][64])lds;
    static_assert(KW * WF * WT * WM * WN <= NST * (FT + TT) * TPS, "the waves' sums fit the stages");
    const int slot = fw + WF * tw;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) red[kw][slot][i * WN + j][lane] = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        if ((i * WN + j) % KW != kw) continue;  // block b is finished by wave b % KW
        f32x4 s = red[0][slot][i * WN + j][lane];
#pragma unroll
        for (int w = 1; w < KW; ++w) s += red[w][slot][i * WN + j][lane];
        acc[i][j] = s;
      }
  }
  float rs[WN];
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    rs[j] = 1.f;
    if constexpr (kNorm) {
      const int tok = (tw * WN + j) * 16 + tl;
      float s = sq_s[0][tok];
#pragma unroll
      for (int p = 1; p < kParts; ++p) s += sq_s[p][tok];
      rs[j] = 1.0f / sqrtf(s * a.inv_K + g.eps);
    }
  }
  const PlainAhead<T> none;
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int ft = ft0 + fw * WM + i, tt = tt0 + tw * WN + j;
      if (KW > 1 && (i * WN + j) % KW != kw) continue;
      if (ft >= a.ft || tt >= a.tt) continue;  // uniform over the wave
      plain_epilogue<T, EPI, false>(g, a.out_tiles, ft, tt * 16 + tl, q4, acc[i][j], rs[j], none);
    }
  if (EPI == PLAIN_FINAL && g.lens_advance && blockIdx.x == 0)
    for (int b = threadIdx.x; b < g.rows; b += WAVES * 64) g.lens_advance[b] += 1;
}

// ----------------------------------------------------------------------------
// Attention of a prompt over the cache.  A workgroup owns 16 consecutive prompt tokens of one head and its KW waves take the
// 16-key blocks in turn.  S^T = K q^T (keys on the M axis: a lane holds four keys of one query),
// online softmax in fp32, O^T += V^T P^T with fp32 probabilities against fp32 products for either
// storage type; the waves' (max, sum, output) meet in LDS in wave order.  Bound by the fp32 matrix pipe.
// ----------------------------------------------------------------------------
// NF: 16-feature blocks the registers hold, a multiple of what d needs
template <typename T, int NF, int KW>
__global__ void __launch_bounds__(KW * 64) k_plain_attn(AttnArgs<T> a) {
  constexpr int NC = NF * (int)sizeof(T) / 4;  // K tiles: 16 floats or 32 bf16 each
  extern __shared__ __attribute__((aligned(16))) f32x4 o_s[];  // [KW][nf][64]
  __shared__ float m_s[KW][16], l_s[KW][16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, tl = lane & 15, g4 = (lane >> 4) * 4;
  const int d = a.cache.d, nf = (d + 15) / 16, nc = plain_tiles(d, sizeof(T));
  const PlainTile t = a.tiles[blockIdx.x];
  const int head = blockIdx.y, kvh = head / a.G, req = t.req, row = t.row0 + min(tl, t.n - 1), qpos = t.pos0 + min(tl, t.n - 1);
  const int last = t.pos0 + t.n - 1;
  const bool live = tl < t.n;
  const u32x4 *kp = (const u32x4 *)(a.Kc + ((size_t)req * a.cache.nkv + kvh) * a.cache.k_elems(sizeof(T))) + lane;
  const T *vp = a.Vc + ((size_t)req * a.cache.nkv + kvh) * a.cache.v_elems() + lane * 4;
  const u32x4 *qp = (const u32x4 *)(a.q + ((size_t)row * a.nq + head) * a.q_ld) + (lane >> 4);
  u32x4 qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c < nc) qf[c] = qp[c * 4];
  f32x4 o[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) o[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const int n_kb = (last >> 4) + 1;
  // a wave's next block is requested before the current one is used, where the registers allow it
  constexpr int kSets = NF * (int)sizeof(T) <= 16 ? 2 : 1;
  u32x4 kS[kSets][NC];
  typename VRaw<T>::V vS[kSets][NF];
  auto load = [&](u32x4 (&k)[NC], typename VRaw<T>::V (&v)[NF], int kb) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc) k[c] = kp[((size_t)kb * nc + c) * 64];
#pragma unroll
    for (int f = 0; f < NF; ++f)
      if (f < nf) v[f] = *(const typename VRaw<T>::V *)(vp + ((size_t)kb * nf + f) * 256);
  };
  auto block = [&](u32x4 (&kf)[NC], typename VRaw<T>::V (&v)[NF], int kb) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, s1 = s;  // two chains
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < nc)
#pragma unroll
        for (int e = 0; e < kMmaSteps<T>; ++e) {
          if ((c * kMmaSteps<T> + e) & 1) s1 = mma<T>(kf[c], qf[c], s1, e);
          else s = mma<T>(kf[c], qf[c], s, e);
        }
    s += s1;
    f32x4 vf[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
      if (f < nf) vf[f] = widen_v4<T>(v[f]);
    const bool edge = kb == n_kb - 1;  // the only block with keys some query must not see
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] *= a.scale;
      if (edge && kb * 16 + g4 + i > qpos) s[i] = -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    mx = rows_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float ref = m_new == -INFINITY ? 0.f : m_new;  // nothing visible yet
    const float corr = expf(m_run - ref);
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = expf(s[i] - ref);
    l_run = l_run * corr + ((p[0] + p[1]) + (p[2] + p[3]));
    m_run = m_new;
#pragma unroll
    for (int f = 0; f < NF; ++f) o[f] *= corr;
    bool shared = true;
    if (edge) {
      // slots past the last cached key hold anything: no product may meet them
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (f < nf && kb * 16 + g4 + i > last) vf[f][i] = 0.f;
      {
        // a value that is not finite must not reach the queries in front of it (0 * inf): such a
        // block - no ordinary one - is added key by key
        bool odd = false;
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
          for (int i = 0; i < 4; ++i) odd |= f * 16 + tl < d && !(fabsf(vf[f][i]) < INFINITY);  // features past d hold anything
        shared = !__any(odd);
        if (!shared) {
#pragma unroll 1
          for (int jq = 0; jq < 4; ++jq)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float pj = __shfl(p[j], jq * 16 + tl, 64);
#pragma unroll
              for (int f = 0; f < NF; ++f)
                if (f < nf)
#pragma unroll
                  for (int i = 0; i < 4; ++i) {
                    const float v = __shfl(vf[f][j], jq * 16 + g4 + i, 64);
                    if (kb * 16 + 4 * jq + j <= qpos) o[f][i] = fmaf(pj, v, o[f][i]);
                  }
            }
        }
      }
    }
    if (shared)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int f = 0; f < NF; ++f)
          if (f < nf) o[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[f][i], p[i], o[f], 0, 0, 0);
  };
  if constexpr (kSets == 2) {
    if (wave < n_kb) load(kS[0], vS[0], wave);
    for (int kb = wave; kb < n_kb; kb += 2 * KW) {
      load(kS[1], vS[1], min(kb + KW, n_kb - 1));  // past the end: the last block again, not used
      block(kS[0], vS[0], kb);
      if (kb + KW >= n_kb) break;
      load(kS[0], vS[0], min(kb + 2 * KW, n_kb - 1));
      block(kS[1], vS[1], kb + KW);
    }
  } else {
    for (int kb = wave; kb < n_kb; kb += KW) {
      load(kS[0], vS[0], kb);
      block(kS[0], vS[0], kb);
    }
  }
  l_run = rows_sum(l_run);
  if (lane < 16) { m_s[wave][tl] = m_run; l_s[wave][tl] = l_run; }
#pragma unroll
  for (int f = 0; f < NF; ++f)
    if (f < nf) o_s[(wave * nf + f) * 64 + lane] = o[f];
  __syncthreads();
  float m = m_s[0][tl];  // -inf: a share without a key, whose weights and sums are 0
#pragma unroll
  for (int w = 1; w < KW; ++w) m = fmaxf(m, m_s[w][tl]);
  float wgt[KW], l = 0.f;
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    wgt[w] = m_s[w][tl] == -INFINITY ? 0.f : expf(m_s[w][tl] - m);
    l += wgt[w] * l_s[w][tl];
  }
  for (int f = wave; f < nf; f += KW) {
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; ++w)
      if (w < n_kb) r += o_s[(w * nf + f) * 64 + lane] * wgt[w];
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = r[i] / l;
    const int f0 = f * 16 + g4, n = min(4, d - f0), k = head * d + f0;
    if (!live || n <= 0) continue;
    if (d % 4 == 0) put4(a.out + plain_offset<T>(row, k, a.out_tiles), v, n, true);
    else
      for (int i = 0; i < n; ++i) store_f32(a.out + plain_offset<T>(row, k + i, a.out_tiles), v[i]);
  }
}

template <typename T>
__global__ void k_plain_export_kv(const T *__restrict__ Kc, const T *__restrict__ Vc, T *__restrict__ k_out,
                                  T *__restrict__ v_out, int request, int len, PlainCache c) {
  const int kvd = c.nkv * c.d, tk = plain_tiles(c.d, sizeof(T));
  const size_t n = (size_t)len * kvd, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int pos = (int)(i / kvd), e = (int)(i % kvd), h = e / c.d, f = e % c.d;
    const size_t rh = (size_t)request * c.nkv + h;
    k_out[i] = Kc[rh * c.k_elems(sizeof(T)) + plain_offset<T>(pos, f, tk)];
    v_out[i] = Vc[rh * c.v_elems() + c.v_offset(pos, f)];
  }
}

__global__ void k_plain_fill_zero(uint4 *p, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = uint4{0, 0, 0, 0};
}

inline int grid_for(size_t n, int block) {
  size_t g = (n + block - 1) / block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

template <typename T>
hipError_t plain_pack_weight(const T *src0, const T *src1, const T *src2, int rows0, int rows1, T *dst, int N, int K,
                             int mode, int head_dim, int qk_rows, hipStream_t s) {
  const int tiles = plain_tiles(K, sizeof(T));
  const size_t chunks = (size_t)((N + 15) / 16) * tiles * 64;
  k_plain_pack<T><<<grid_for(chunks, 256), 256, 0, s>>>(src0, src1, src2, rows0, rows1, dst, N, K, tiles, mode, head_dim, qk_rows, chunks);
  return hipGetLastError();
}

template <typename T>
hipError_t plain_begin(const T *hidden_in, float *xres, const T *gain, T *y, float *ssq_out, int rows, int rows_pad, int H,
                       const PlainAngles &ang, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  // grid.x carries the row (up to 2^31 - 1)
  k_plain_begin<T><<<dim3(rows, (std::max(H, ang.pos ? ang.half : 0) + 255) / 256), 256, 0, s>>>(hidden_in, xres, gain, y, ssq_out, H, rows_pad,
                                                                                                 plain_tiles(H, sizeof(T)), ang);
  return hipGetLastError();
}

// The forms of k_plain_gemm that stage through LDS, <WM, WN, WF, WT, KW, KS, NST>
#define HYP_PLAIN_GEMM_SMALL 2, 2, 2, 2, 2, 1, 4
#define HYP_PLAIN_GEMM_WIDE_FLOAT 2, 4, 4, 2, 1, 2, 2
#define HYP_PLAIN_GEMM_WIDE_BF16 2, 4, 4, 2, 1, 1, 4
#define HYP_PLAIN_GEMM_MANY_BF16 4, 4, 2, 2, 1, 1, 3
constexpr int plain_gemm_lds(int WM, int WN, int WF, int WT, int KW, int KS, int NST) { return NST * (WM * WF + WN * WT) * KW * KS * 1024; }

template <typename T, int EPI>
static hipError_t launch_gemm(const PlainGemm<T> &g, hipStream_t s) {
  GemmArgs<T> a = gemm_args<T, EPI>(g);
  auto groups = [](int n, int per) { return (unsigned)((n + per - 1) / per); };
  const int form = plain_gemm_form((int)sizeof(T), g.rows, g.N, g.K, EPI == PLAIN_QKV, EPI == PLAIN_SWIGLU);
  const unsigned wide = groups(a.ft, 8) * groups(a.tt, 8);
#define LAUNCH(GRID, THREADS, ...) k_plain_gemm<T, EPI, __VA_ARGS__><<<GRID, THREADS, plain_gemm_lds(__VA_ARGS__), s>>>(a)
  if (form == PLAIN_GEMM_REGISTERS) k_plain_gemm<T, EPI, 2, 2, 1, 1, 4><<<groups(a.ft, 2) * groups(a.tt, 2), 256, 0, s>>>(a);
  else if (form == PLAIN_GEMM_SMALL) LAUNCH(groups(a.ft, 4) * groups(a.tt, 4), 512, HYP_PLAIN_GEMM_SMALL);
  else if constexpr (sizeof(T) == 4) LAUNCH(wide, 512, HYP_PLAIN_GEMM_WIDE_FLOAT);
  else if (form == PLAIN_GEMM_MANY) LAUNCH(wide, 256, HYP_PLAIN_GEMM_MANY_BF16);
  else LAUNCH(wide, 512, HYP_PLAIN_GEMM_WIDE_BF16);
#undef LAUNCH
  return hipGetLastError();
}

template <typename T> hipError_t plain_gemm(int epi, const PlainGemm<T> &g, hipStream_t s) {
  if (g.rows <= kPlainGemvRows) return plain_gemv<T>(epi, g, s);
  switch (epi) {
    case PLAIN_QKV: return launch_gemm<T, PLAIN_QKV>(g, s);
    case PLAIN_SWIGLU: return launch_gemm<T, PLAIN_SWIGLU>(g, s);
    case PLAIN_RESID: return launch_gemm<T, PLAIN_RESID>(g, s);
    case PLAIN_FINAL: return launch_gemm<T, PLAIN_FINAL>(g, s);
  }
  return hipErrorInvalidValue;
}

// (register blocks, waves): enough for d features; the waves' outputs pass 64 KiB of LDS at 8 waves of 128 features and more
#define HYP_PLAIN_ATTN(X) X(4, 8) X(8, 8) X(16, 4)

template <typename T>
static hipError_t launch_attn(const AttnArgs<T> &a, dim3 grid, hipStream_t s) {
  const int nf = (a.cache.d + 15) / 16, nf_tiles = plain_tiles(a.cache.d, sizeof(T)) * 4 / (int)sizeof(T);
#define X(NF, KW)                                                                              \
  if (nf_tiles <= NF) {                                                                         \
    k_plain_attn<T, NF, KW><<<grid, KW * 64, (size_t)KW * nf * 1024, s>>>(a);           \
    return hipGetLastError();                                                                  \
  }
  HYP_PLAIN_ATTN(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t plain_init() {
  hipError_t e = plain_decode_init();
#define X(NF, KW)                                                                                                              \
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_plain_attn<float, NF, KW>, hipFuncAttributeMaxDynamicSharedMemorySize, NF * KW * 1024);  \
  if (e == hipSuccess) e = hipFuncSetAttribute((const void *)k_plain_attn<bf16_t, NF, KW>, hipFuncAttributeMaxDynamicSharedMemorySize, NF * KW * 1024); \
  HYP_PLAIN_ATTN(X)
#undef X
#define X(T, EPI, ...)  \
  if (e == hipSuccess) \
    e = hipFuncSetAttribute((const void *)k_plain_gemm<T, EPI, __VA_ARGS__>, hipFuncAttributeMaxDynamicSharedMemorySize, plain_gemm_lds(__VA_ARGS__));
#define Y(T, ...) X(T, PLAIN_QKV, __VA_ARGS__) X(T, PLAIN_SWIGLU, __VA_ARGS__) X(T, PLAIN_RESID, __VA_ARGS__) X(T, PLAIN_FINAL, __VA_ARGS__)
  Y(float, HYP_PLAIN_GEMM_SMALL) Y(float, HYP_PLAIN_GEMM_WIDE_FLOAT)
  Y(bf16_t, HYP_PLAIN_GEMM_SMALL) Y(bf16_t, HYP_PLAIN_GEMM_WIDE_BF16) Y(bf16_t, HYP_PLAIN_GEMM_MANY_BF16)
#undef Y
#undef X
  return e;
}

template <typename T>
hipError_t plain_attn_prefill(const T *q, int q_ld, const T *Kc, const T *Vc, T *out, const PlainTile *tiles, int n_tiles,
                              const PlainCache &cache, const Dims &dm, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  AttnArgs<T> a = attn_args<T>(q, q_ld, Kc, Vc, out, cache, dm);
  a.tiles = tiles;
  return launch_attn<T>(a, dim3(n_tiles, dm.nq), s);
}

template <typename T>
hipError_t plain_export_kv(const T *Kc, const T *Vc, T *k_out, T *v_out, int request, int len,
                           const PlainCache &cache, hipStream_t s) {
  if (len == 0) return hipSuccess;
  k_plain_export_kv<T><<<grid_for((size_t)len * cache.nkv * cache.d, 256), 256, 0, s>>>(Kc, Vc, k_out, v_out, request, len, cache);
  return hipGetLastError();
}

hipError_t plain_fill_zero(void *p, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  if (n16) k_plain_fill_zero<<<grid_for(n16, 256), 256, 0, s>>>((uint4 *)p, n16);
  return hipGetLastError();
}

#define HYP_INSTANTIATE(T)                                                                                                   \
  template hipError_t plain_pack_weight<T>(const T *, const T *, const T *, int, int, T *, int, int, int, int, int, hipStream_t); \
  template hipError_t plain_begin<T>(const T *, float *, const T *, T *, float *, int, int, int, const PlainAngles &, hipStream_t); \
  template hipError_t plain_gemm<T>(int, const PlainGemm<T> &, hipStream_t);                                                 \
  template hipError_t plain_attn_prefill<T>(const T *, int, const T *, const T *, T *, const PlainTile *, int,               \
                                            const PlainCache &, const Dims &, hipStream_t);                                  \
  template hipError_t plain_export_kv<T>(const T *, const T *, T *, T *, int, int, const PlainCache &, hipStream_t);
HYP_INSTANTIATE(float)
HYP_INSTANTIATE(bf16_t)

}  // namespace hyp
