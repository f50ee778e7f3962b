// Internal declarations shared by the translation units of the stage library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hyp_stage.h"

namespace hyp {

// ----------------------------------------------------------------------------
// bf16 <-> fp32 (bit patterns; round to nearest even)
// ----------------------------------------------------------------------------
typedef uint16_t bf16_t;

__host__ __device__ inline float bf16_to_f32(bf16_t v) {
  union { uint32_t u; float f; } c;
  c.u = (uint32_t)v << 16;
  return c.f;
}

__host__ __device__ inline bf16_t f32_to_bf16(float f) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_bit_cast(bf16_t, (__bf16)f);  // v_cvt_pk_bf16_f32 rounds as the steps below do (test_gpu_bf16_rounding.py)
#else
  union { uint32_t u; float f; } c;
  c.f = f;
  uint32_t u = c.u;
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
#endif
}

template <typename T> __device__ inline float load_f32(const T *p);
template <> __device__ inline float load_f32<float>(const float *p) { return *p; }
template <> __device__ inline float load_f32<bf16_t>(const bf16_t *p) { return bf16_to_f32(*p); }
template <typename T> __device__ inline void store_f32(T *p, float v);
template <> __device__ inline void store_f32<float>(float *p, float v) { *p = v; }
template <> __device__ inline void store_f32<bf16_t>(bf16_t *p, float v) { *p = f32_to_bf16(v); }

// ----------------------------------------------------------------------------
// Geometry of one block, as the kernels see it
// ----------------------------------------------------------------------------
struct Dims {
  int H, nq, nkv, d, I;
  int qd, kvd;       // nq*d, nkv*d
  int max_batch, max_seq;
  float eps;
};

// ----------------------------------------------------------------------------
// Plain (shape-generic) kernels, T = float or bf16_t storage, fp32 accumulation.
//
// Every matrix operand of a contraction lives in *16-row fragment order*, "F(R, K)": tiles of 16
// rows x 64 bytes of K (16 floats or 32 bf16), 1 KiB each = 64 lanes x 16 bytes; lane l holds row
// l % 16, 16-byte chunk l / 16.  That is the operand of v_mfma_f32_16x16x32_bf16 as it stands and
// of four v_mfma_f32_16x16x4_f32 (the i-th takes element i of every lane).  K is padded to whole
// tiles with zeros (weights: packed so; activations: zeroed once, never written there), rows to
// whole tiles with anything finite or not: a row only reaches its own output.
// ----------------------------------------------------------------------------
template <typename T> __host__ __device__ constexpr int plain_chunk() { return 16 / (int)sizeof(T); }   // elements per 16 bytes
template <typename T> __host__ __device__ constexpr int plain_tile_k() { return 64 / (int)sizeof(T); }  // K elements per tile
__host__ __device__ inline int plain_tiles(int k, int es) { return (k * es + 63) / 64; }  // tiles along K
template <typename T> __host__ __device__ inline size_t plain_offset(size_t row, int k, int tiles) {
  constexpr int E = plain_chunk<T>();
  return (((row >> 4) * tiles + k / (4 * E)) * 64 + (size_t)((k / E) & 3) * 16 + (row & 15)) * E + k % E;
}
// KV cache of one layer, per (request, KV head): keys F(max_seq, d); values as tiles of 16 keys x
// 16 features, lane l holding feature l % 16 and keys 4 (l / 16) .. + 3 (the operand of the P V
// product in the order in which probabilities leave the score accumulators).
struct PlainCache {
  int nkv, d, key_blocks;  // 16-key blocks per request
  __host__ __device__ size_t k_elems(int es) const { return (size_t)key_blocks * plain_tiles(d, es) * (1024 / es); }
  __host__ __device__ size_t v_elems() const { return (size_t)key_blocks * ((d + 15) / 16) * 256; }
  __host__ __device__ size_t v_offset(int pos, int f) const {
    const int w = pos & 15;
    return ((size_t)(pos >> 4) * ((d + 15) / 16) + (f >> 4)) * 256 + ((w >> 2) * 16 + (f & 15)) * 4 + (w & 3);
  }
};

enum { PLAIN_QKV = 0, PLAIN_SWIGLU = 1, PLAIN_RESID = 2, PLAIN_FINAL = 3 };

// out^T[N, rows] = W[N, K] X[rows, K]^T and what follows it in the block
template <typename T> struct PlainGemm {
  const T *W = nullptr, *X = nullptr;  // F(N, K), F(rows, K)
  int N = 0, K = 0, rows = 0;
  // sums of squares of the rows of the normalised input, [ssq_parts][rows_pad]; null: no norm
  const float *ssq_in = nullptr;
  int ssq_parts = 0, rows_pad = 0;
  float eps = 0.f;
  // PLAIN_QKV: rotary position, cache append, queries row-major [rows][nq][q_ld]
  const int *tok_req = nullptr, *tok_pos = nullptr;  // no tok_req: row r is request r
  const float *cos_tab = nullptr, *sin_tab = nullptr;  // [position][d / 2], or [row][d / 2] with tab_by_row
  bool tab_by_row = false;
  float *cos_row = nullptr, *sin_row = nullptr;  // where given: the rows' angles are left here, [row][d / 2]
  // plain_gemv_opens(): the rows as the stage gets them, [rows][K], and the norm's gain, instead of X and ssq_in
  const T *first_in = nullptr, *first_gain = nullptr;
  T *q = nullptr, *Kc = nullptr, *Vc = nullptr;
  int q_ld = 0;
  PlainCache cache = {};
  Dims dm = {};
  // PLAIN_SWIGLU: F(rows, N / 2)
  T *m = nullptr;
  // PLAIN_RESID: residual [rows][N], gain of the next norm, y = x * gain -> F(rows, N), sums of squares per 16 features
  float *xres = nullptr;
  const T *res_in = nullptr;  // the residual as the stage gets it, instead of xres (which is written)
  const T *gain = nullptr;
  T *y = nullptr;
  float *ssq_out = nullptr;
  // PLAIN_FINAL: residual in, stage output out; lens += 1 where given
  T *hidden_out = nullptr;
  int *lens_advance = nullptr;
};
struct PlainTile { int row0, pos0, n, req; };  // up to 16 consecutive prompt tokens of one request

enum { PLAIN_ROWS = 0, PLAIN_PAIRS_QKV = 1, PLAIN_PAIRS_GATEUP = 2 };
// dst = F(N, K) of the rows of [src0; src1; src2], row order by `mode` (see plain_src_row)
template <typename T>
hipError_t plain_pack_weight(const T *src0, const T *src1, const T *src2, int rows0, int rows1, T *dst, int N, int K,
                             int mode, int head_dim, int qk_rows, hipStream_t s);
// decode: positions of the rows, and their rotary angles out of the tables into [row][half]; pos null: none
struct PlainAngles {
  const int *pos = nullptr;
  const float *cos_tab = nullptr, *sin_tab = nullptr;
  float *cos_row = nullptr, *sin_row = nullptr;
  int half = 0;
};
// x = hidden_in ; xres = x ; y = x * gain -> F(rows, H) ; sums of squares per 16 features
template <typename T>
hipError_t plain_begin(const T *hidden_in, float *xres, const T *gain, T *y, float *ssq_out, int rows, int rows_pad, int H,
                       const PlainAngles &ang, hipStream_t s);
template <typename T> hipError_t plain_gemm(int epi, const PlainGemm<T> &g, hipStream_t s);
constexpr int kPlainGemvRows = 32;  // up to so many rows plain_gemm is
template <typename T> hipError_t plain_gemv(int epi, const PlainGemm<T> &g, hipStream_t s);
// whether a step of so many rows can open with its QKV contraction: what plain_begin does happens in its staging
template <typename T> bool plain_gemv_opens(const T *hidden_in, int rows, int N, int K);
// prompt: tiles of up to 16 tokens; out F(rows, nq d)
template <typename T>
hipError_t plain_attn_prefill(const T *q, int q_ld, const T *Kc, const T *Vc, T *out, const PlainTile *tiles, int n_tiles,
                              const PlainCache &cache, const Dims &dm, hipStream_t s);
// one token per request at position lens[request] <= longest, whose key is already cached; part: plain_attn_part_floats()
template <typename T>
hipError_t plain_attn_decode(const T *q, int q_ld, const T *Kc, const T *Vc, T *out, const int *lens, int batch, int longest,
                             float *part, const PlainCache &cache, const Dims &dm, hipStream_t s);
size_t plain_attn_part_floats(const Dims &dm, int batch);
hipError_t plain_decode_init();
hipError_t plain_init();  // kernel attributes
template <typename T>
hipError_t plain_export_kv(const T *Kc, const T *Vc, T *k_out, T *v_out, int request, int len,
                           const PlainCache &cache, hipStream_t s);
hipError_t plain_fill_zero(void *p, size_t bytes, hipStream_t s);

}  // namespace hyp
