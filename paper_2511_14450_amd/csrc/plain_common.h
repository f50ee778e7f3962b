// What the shape-generic kernels of a prompt (plain_kernels.hip) and of a decode step
// (plain_decode.hip) share: MFMA steps on fragment-order operands, kernel arguments and the
// epilogues of the four contractions of a block.
#pragma once

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch_rules.h"

namespace hyp {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// MFMA steps that the 64 bytes of K of one fragment pair take, and the i-th of them: acc += A B
template <typename T> constexpr int kMmaSteps = 1;
template <> constexpr int kMmaSteps<float> = 4;
template <typename T> __device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 acc, int i);
template <> __device__ __forceinline__ f32x4 mma<float>(u32x4 a, u32x4 b, f32x4 acc, int i) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i]), __uint_as_float(b[i]), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma<bf16_t>(u32x4 a, u32x4 b, f32x4 acc, int) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// Exchanges between the lanes of a wave without the LDS pipe, whose shuffles take 60 ns each, one behind the other: the values of
// both rows of 16 lanes of a half, of both halves; a lane's value O lanes on in its row, or behind.
struct LanePair { float a, b; };
__device__ __forceinline__ LanePair both_rows(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair both_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
template <int CTRL> __device__ __forceinline__ float lane_dpp(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <int O> __device__ __forceinline__ float lane_on(float v) { return lane_dpp<0x100 + O>(v); }      // row_shl; 0 past the row
template <int O> __device__ __forceinline__ float lane_round(float v) { return lane_dpp<0x120 + O>(v); }   // row_ror
// over the four lanes l % 16 of the wave's rows: as __shfl_xor 16, then 32
__device__ __forceinline__ float rows_sum(float v) {
  const LanePair r = both_rows(v), h = both_halves(r.a + r.b);
  return h.a + h.b;
}
__device__ __forceinline__ float rows_max(float v) {
  const LanePair r = both_rows(v), h = both_halves(fmaxf(r.a, r.b));
  return fmaxf(h.a, h.b);
}

// four consecutive elements: one wide access where `vec` says the address allows it
template <typename T> struct Four;
template <> struct Four<float> { typedef f32x4 V; };
template <> struct Four<bf16_t> { typedef uint2 V; };
template <typename T> __device__ __forceinline__ void put4(T *p, const float *v, int n, bool vec) {
  if (vec && n == 4) {
    union { T e[4]; typename Four<T>::V v; } u;
#pragma unroll
    for (int i = 0; i < 4; ++i) store_f32(&u.e[i], v[i]);
    *(typename Four<T>::V *)p = u.v;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < n) store_f32(p + i, v[i]);
  }
}

template <typename T> struct GemmArgs {
  PlainGemm<T> g;
  int tiles;      // tiles along K
  int ft, tt;     // 16-row tiles of features, of tokens
  int out_tiles;  // tiles along K of the output matrix in fragment order
  float inv_K;
};

template <typename T, int EPI> inline GemmArgs<T> gemm_args(const PlainGemm<T> &g) {
  GemmArgs<T> a;
  a.g = g;
  a.tiles = plain_tiles(g.K, sizeof(T));
  a.ft = (g.N + 15) / 16; a.tt = (g.rows + 15) / 16;
  a.out_tiles = plain_tiles(EPI == PLAIN_SWIGLU ? g.N / 2 : g.N, sizeof(T));
  a.inv_K = 1.0f / (float)g.K;
  return a;
}

template <typename T> struct AttnArgs {
  const T *q, *Kc, *Vc;
  T *out;
  const PlainTile *tiles;
  const int *lens;
  PlainCache cache;
  int nq, G, q_ld, out_tiles;
  float scale;
  int split;    // decode: workgroups that share the keys of a (request, head group)
  float *part;  // split > 1: [request][head][split][2 + d] = max, sum, unnormalised output
};

template <typename T>
inline AttnArgs<T> attn_args(const T *q, int q_ld, const T *Kc, const T *Vc, T *out, const PlainCache &cache, const Dims &dm) {
  AttnArgs<T> a = {};
  a.q = q; a.Kc = Kc; a.Vc = Vc; a.out = out; a.cache = cache;
  a.nq = dm.nq; a.G = dm.nq / dm.nkv; a.q_ld = q_ld; a.out_tiles = plain_tiles(dm.qd, sizeof(T));
  a.scale = 1.0f / sqrtf((float)dm.d);
  return a;
}

template <typename T> struct VRaw;
template <> struct VRaw<float> { typedef f32x4 V; };
template <> struct VRaw<bf16_t> { typedef uint2 V; };
template <typename T> __device__ __forceinline__ f32x4 widen_v4(typename VRaw<T>::V u);
template <> __device__ __forceinline__ f32x4 widen_v4<float>(f32x4 u) { return u; }
template <> __device__ __forceinline__ f32x4 widen_v4<bf16_t>(uint2 u) {
  return f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
}

// What the epilogue of a 16 x 16 block needs, requested and worked out ahead of its use by the forms that have the registers:
// rotary angles and destinations of two pairs of packed rows, residual and gain.
template <typename T> struct PlainAhead {
  float c[2] = {0.f, 0.f}, s[2] = {0.f, 0.f};
  T *dst[2] = {nullptr, nullptr};
  int second[2] = {0, 0};  // the pair's second element, behind dst
  f32x4 x = {0.f, 0.f, 0.f, 0.f}, g = {0.f, 0.f, 0.f, 0.f};
};
// where rows r, r + 1 of token `tok` go; r is even, as is every boundary between heads and matrices
template <typename T> __device__ __forceinline__ T *plain_qkv_dst(const PlainGemm<T> &g, int tok, int req, int pos, int r, int *second) {
  const int d = g.dm.d, half = d >> 1, head = r / d, e = r - head * d;
  if (head < g.dm.nq) {
    *second = half;
    return g.q + ((size_t)tok * g.dm.nq + head) * g.q_ld + (e >> 1);
  }
  if (head < g.dm.nq + g.dm.nkv) {
    const int tk = plain_tiles(d, sizeof(T)), at = (int)plain_offset<T>(pos & 15, e >> 1, tk);
    *second = (int)plain_offset<T>(pos & 15, (e >> 1) + half, tk) - at;
    return g.Kc + ((size_t)req * g.dm.nkv + head - g.dm.nq) * g.cache.k_elems(sizeof(T)) + (size_t)(pos >> 4) * tk * (1024 / sizeof(T)) + at;
  }
  const int at = (int)g.cache.v_offset(pos & 15, e);
  *second = (int)g.cache.v_offset(pos & 15, e + 1) - at;
  return g.Vc + ((size_t)req * g.dm.nkv + head - g.dm.nq - g.dm.nkv) * g.cache.v_elems() + (size_t)(pos >> 4) * ((d + 15) / 16) * 256 + at;
}
// row of the tables of rotary angles that token `tok` at position `pos` reads
template <typename T> __device__ __forceinline__ size_t plain_angle(const PlainGemm<T> &g, int tok, int pos, int r) {
  return (size_t)(g.tab_by_row ? tok : pos) * (g.dm.d >> 1) + (r % g.dm.d >> 1);
}
template <typename T, int EPI> __device__ __forceinline__ void plain_fetch(PlainAhead<T> &pf, const PlainGemm<T> &g, int tok, int f0) {
  if (tok >= g.rows || f0 >= g.N) return;
  if (EPI == PLAIN_QKV) {
    const int pos = g.tok_pos[tok], req = g.tok_req ? g.tok_req[tok] : tok;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (f0 + 2 * h < g.dm.qd + g.dm.kvd) {
        const size_t at = plain_angle(g, tok, pos, f0 + 2 * h);
        pf.c[h] = g.cos_tab[at]; pf.s[h] = g.sin_tab[at];
      }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (f0 + 2 * h < g.N) pf.dst[h] = plain_qkv_dst(g, tok, req, pos, f0 + 2 * h, &pf.second[h]);
  } else if (EPI == PLAIN_RESID || EPI == PLAIN_FINAL) {
    const float *xr = g.xres + (size_t)tok * g.N + f0;
    if (EPI == PLAIN_RESID && g.res_in) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (f0 + e < g.N) pf.x[e] = load_f32(g.res_in + (size_t)tok * g.N + f0 + e);
    } else if (g.N % 4 == 0) pf.x = *(const f32x4 *)xr;
    else
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (f0 + e < g.N) pf.x[e] = xr[e];
    if (EPI == PLAIN_RESID)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (f0 + e < g.N) pf.g[e] = load_f32(g.gain + f0 + e);
  }
}

// Epilogue of the 16 x 16 block `ft` x (16 tokens around tok): this lane holds features 16 ft + q4 .. + 3 of token `tok`
template <typename T, int EPI, bool AHEAD>
__device__ __forceinline__ void plain_epilogue(const PlainGemm<T> &g, int out_tiles, int ft, int tok, int q4, f32x4 acc, float rs,
                                               const PlainAhead<T> &pf) {
  const int f0 = ft * 16 + q4, lane = threadIdx.x & 63;
  const bool live = tok < g.rows;
  if (EPI == PLAIN_QKV) {
    if (!live || f0 >= g.N) return;
    const int req = AHEAD ? 0 : g.tok_req ? g.tok_req[tok] : tok, pos = AHEAD ? 0 : g.tok_pos[tok];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = f0 + 2 * h;
      if (r >= g.N) break;
      float v0 = acc[2 * h] * rs, v1 = acc[2 * h + 1] * rs;
      int second = pf.second[h];
      T *dst = AHEAD ? pf.dst[h] : plain_qkv_dst(g, tok, req, pos, r, &second);
      if (r < g.dm.qd + g.dm.kvd) {
        const size_t at = AHEAD ? 0 : plain_angle(g, tok, pos, r);
        const float c = AHEAD ? pf.c[h] : g.cos_tab[at], s = AHEAD ? pf.s[h] : g.sin_tab[at];
        if (AHEAD && g.cos_row && r < g.dm.d) {  // the first query head: every angle once
          g.cos_row[(size_t)tok * (g.dm.d >> 1) + (r >> 1)] = c;
          g.sin_row[(size_t)tok * (g.dm.d >> 1) + (r >> 1)] = s;
        }
        const float lo = v0 * c - v1 * s, hi = v1 * c + v0 * s;
        v0 = lo; v1 = hi;
      }
      store_f32(dst, v0);
      store_f32(dst + second, v1);
    }
  } else if (EPI == PLAIN_SWIGLU) {
    if (!live || f0 >= g.N) return;
    // FFN features f0 / 2 and f0 / 2 + 1 lie side by side (f0 / 2 is even)
    T *dst = g.m + plain_offset<T>(tok, f0 >> 1, out_tiles);
    float v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float gt = acc[2 * h] * rs, up = acc[2 * h + 1] * rs;
      v[h] = gt / (1.0f + expf(-gt)) * up;
    }
    if (f0 + 2 < g.N) {
      struct __attribute__((aligned(2 * sizeof(T)))) Two { T e[2]; } two;
      store_f32(&two.e[0], v[0]);
      store_f32(&two.e[1], v[1]);
      *(Two *)dst = two;
    } else {
      store_f32(dst, v[0]);
    }
  } else {
    const int n = min(4, g.N - f0);
    const bool vec = g.N % 4 == 0;
    float x[4] = {0.f, 0.f, 0.f, 0.f};
    if (live && n > 0) {
      float *xr = g.xres + (size_t)tok * g.N + f0;
      if (AHEAD) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < n) x[e] = pf.x[e] + acc[e];
      } else if (vec) {
        const f32x4 old = *(const f32x4 *)xr;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = old[e] + acc[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < n) x[e] = xr[e] + acc[e];
      }
      if (EPI == PLAIN_RESID) {
        put4(xr, x, n, vec);
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = e < n ? x[e] * (AHEAD ? pf.g[e] : load_f32(g.gain + f0 + e)) : 0.f;
        put4(g.y + plain_offset<T>(tok, f0, out_tiles), y, n, true);
      } else {
        put4(g.hidden_out + (size_t)tok * g.N + f0, x, n, false);
      }
    }
    if (EPI == PLAIN_RESID) {
      float s;
      {
#pragma clang fp contract(off)
        s = (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
      }
      s = rows_sum(s);
      if (lane < 16 && live) g.ssq_out[(size_t)ft * g.rows_pad + tok] = s;
    }
  }
}

}  // namespace

}  // namespace hyp
