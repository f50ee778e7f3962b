// Host-side launchers of the MFMA path (bf16 stages with head_dim 128).
#pragma once

#include "launch_rules.h"
#include "mfma_common.h"

namespace hyp {

enum { PACK_PLAIN = 0, PACK_QKV = 1, PACK_GATEUP = 2 };
enum { EPI_STORE = 0, EPI_SWIGLU = 1, EPI_QKV = 2, EPI_RESID = 3 };

// What the epilogue of a prefill GEMM needs besides its output; fields an epilogue does
// not use stay null.
struct GemmEpilogue {
  // EPI_QKV
  bf16_t *Kc = nullptr, *Vc = nullptr;  // caches of the layer
  CacheGeom geom = {};
  int qd = 0, kvd = 0;
  const float *cos_tab = nullptr, *sin_tab = nullptr;  // [position][64]
  const int *row_pos = nullptr, *row_req = nullptr;    // per internal row; row_req < 0: padding, nothing is written
  const int *row_q = nullptr;                          // row of q that a row's queries go to
  // EPI_QKV, EPI_SWIGLU: RMS Norm factor of every input row (the rows carry the gain only)
  const float *rstd = nullptr;
  // where mfma_gemm_adds_sums(): the sums of squares (ssq_part of the GEMM before) instead, null where rstd is given; row_ext too
  const float *ssq_in = nullptr;
  float eps = 0.f;
  // EPI_RESID: residual stream A(T', N), gains of the following norm, padding map,
  // sums of squares out [N / 64][T']
  float *xres = nullptr;
  const bf16_t *gain = nullptr;
  const int *row_ext = nullptr;
  float *ssq_part = nullptr;
  // every epilogue: scratch for GEMMs whose K loop is split across workgroups (few output tiles)
  float *split_ws = nullptr;          // mfma_gemm_split_ws_bytes()
  unsigned *split_counters = nullptr;  // kGemmShortMaxTiles + 1, zero between launches
};

size_t mfma_gemm_split_ws_bytes();

// dst = P(N, K) of the row-permuted concatenation [src0; src1; src2]
hipError_t mfma_pack_weight(const bf16_t *src0, const bf16_t *src1, const bf16_t *src2, int rows0,
                            int rows1, bf16_t *dst, int N, int K, int mode, int I, hipStream_t s);

// first block's input: x = hidden_in (external rows) -> residual A(T', H), y' = x * gain -> P(T', H), rstd
hipError_t mfma_prefill_begin(const bf16_t *hidden_in, float *xres, const bf16_t *gain, bf16_t *y, float *rstd,
                              const int *row_ext, int rows, int H, float eps, hipStream_t s);
// stage output: hidden_out (external rows) = residual + delta
hipError_t mfma_prefill_end(const float *xres, const bf16_t *delta_bf, bf16_t *hidden_out, const int *row_ext,
                            int rows, int H, hipStream_t s);
// rstd[row] from the per-group sums of squares of EPI_RESID
hipError_t mfma_rstd(const float *ssq_part, float *rstd, const int *row_ext, int rows, int H, float eps, hipStream_t s);

// whether a QKV or gate/up GEMM adds up the sums of squares of its rows itself (the short forms, and k_gemm_finish where all tiles
// are split): the launch of mfma_rstd, 4 - 5 us, is saved
bool mfma_gemm_adds_sums(int epi, int rows, int N, int K);
hipError_t mfma_gemm_init();
// out^T[N, rows] = W[N,K] X[rows,K]^T with the epilogue `epi`; rows % 32 == 0,
// N % 256 == 0, K % 32 == 0, K >= 128
// `cls` (a hyp_kernel_class_t) names the GEMM of the block; it selects a kernel symbol, not behaviour
hipError_t mfma_gemm(int epi, int cls, const bf16_t *X, const bf16_t *W, int rows, int N, int K, bf16_t *out,
                     int out_K, const GemmEpilogue &ep, hipStream_t s);

// Causal GQA attention over the prompt (flash-style, scores never stored).
//   q P(rows of q, nq*128), requests padded to 64 rows ; caches of the layer ; out P(rows, nq*128), packed
//   work items per 64-row query tile: request, first row of q, index of its first 32-row block in the request, first
//   row of out.  The tile that ends a request clears the value slots behind it, up to a multiple of 64 keys.
struct PrefillTile { int req, row0, qblk0, out0; };
hipError_t mfma_attn_init();  // kernel attributes, once per process and device
hipError_t mfma_attn_prefill(const bf16_t *q, const bf16_t *Kc, bf16_t *Vc, CacheGeom geom,
                             bf16_t *out, const PrefillTile *tiles, int n_tiles, const int *req_len,
                             int nq, int nkv, hipStream_t s);

// ------------------------------------------------------------------ decode
enum { DEC_QKV = 0, DEC_SWIGLU = 1, DEC_RESID = 2, DEC_FINAL = 3, DEC_QKV_OPEN = 4 };

// One skinny GEMM of a decode step, sum[token, n] = W[n, :] . x[token, :], with
// its consumer fused in (see k_dec_gemv).  Fields a given epilogue does not use
// stay null / 0.
struct DecGemv {
  const bf16_t *W = nullptr, *x = nullptr;  // P(N, K), P(32, K)
  float *partial = nullptr;                 // partial sums of the K slices, mfma_gemv_partial_floats(plan, N, K) floats
  unsigned *counters = nullptr;             // [N / 32], zero between launches
  int N = 0, K = 0, batch = 0;
  GemvPlan plan;                            // plan.fbw also sets the granularity of ssq_out (sums of squares per 32 or 64 rows)
  size_t partial_floats = 0;                // room behind `partial`
  const float *ssq_in = nullptr;            // [n_ssq][32] sums of squares of the normalised input
  int n_ssq = 0;
  float eps = 0.f;
  const int *lens = nullptr;
  const float *cos_tab = nullptr, *sin_tab = nullptr;
  bf16_t *qdec = nullptr, *Kc = nullptr, *Vc = nullptr;
  CacheGeom geom = {};
  int nq = 0, nkv = 0;
  bf16_t *m_out = nullptr;
  int I = 0;
  float *xres = nullptr;
  const bf16_t *gain = nullptr;
  bf16_t *y_out = nullptr;
  float *ssq_out = nullptr;
  bf16_t *hidden_out = nullptr;
  int H = 0;
  int *lens_advance = nullptr;  // DEC_FINAL: lengths to increment at the end of the step
};
hipError_t mfma_dec_gemv(int epi, int cls, const DecGemv &a, hipStream_t s);  // cls: as for mfma_gemm
size_t mfma_gemv_partial_floats(const GemvPlan &plan, int N, int K);
bool mfma_gemv_counts(const GemvPlan &plan, int N, int K);  // whether the GEMM uses its arrival counters
hipError_t mfma_gemv_init();  // kernel attributes, once per process and device
// whether a stage's steps open with DEC_QKV_OPEN (x = the rows, aligned to 16 bytes; gain, xres, H set) instead of
// mfma_dec_begin and DEC_QKV.  The rows' address has no say in it: where they are not aligned they are copied first, so that
// the bits of a step, whose sums of squares the two openings group differently, do not depend on it.
bool mfma_dec_opens(int H, int N, const GemvPlan &plan);
hipError_t mfma_dec_align(const bf16_t *hidden_in, bf16_t *out, int H, int batch, hipStream_t s);
// x = hidden_in ; xres = x ; y' = x * gain -> P(32, H) ; ssq_out[H/64][32]
hipError_t mfma_dec_begin(const bf16_t *hidden_in, float *xres, const bf16_t *gain, bf16_t *y_out, float *ssq_out,
                          int H, int batch, hipStream_t s);

// Decode attention; out row b of P(32, nq*128).  Every form is right at any context; they differ in speed and in the order
// of their sums:
//   DEC_ATTN_CHUNKED   split-KV over chunks of chunk_keys keys + fixed-order merge
//   DEC_ATTN_SHORT     one workgroup per (request, KV head), made for batches whose longest context is at most kShortKeys
//   DEC_ATTN_SHORT2    keys (the new token's included); the second requests two blocks per wave at once instead of one
//   DEC_ATTN_RECORDED  for steps that are replayed at contexts the host does not see: a batch whose longest context is at
//                      most kShortKeys keys gets the bits of the short forms, any other the chunked form's
// part: mfma_attn_decode_part_floats() floats
enum { DEC_ATTN_CHUNKED = 0, DEC_ATTN_SHORT = 1, DEC_ATTN_SHORT2 = 2, DEC_ATTN_RECORDED = 3 };
constexpr int kShortKeys = 512;
// One block per wave is all there is up to 256 keys, and half the registers let two workgroups share a CU (32 x 10 heads,
// 240 keys: 15.0 against 16.6 us; 8 x 10 heads 9.2 against 9.3); beyond, two save a round trip (8 x 10 heads, 300 keys:
// 10.1 against 13.9).
inline int mfma_decode_attn_form(int longest) {
  return longest <= kShortKeys / 2 ? DEC_ATTN_SHORT : longest <= kShortKeys ? DEC_ATTN_SHORT2 : DEC_ATTN_CHUNKED;
}
// What the short forms read into L2 beside their own work, for the launch behind them: the first group_bytes of each of `groups`
// row groups of group_stride bytes, which workgroup g of that launch is going to stream (XCD g % 8).  No groups: nothing.
struct ReadAhead {
  const bf16_t *W = nullptr;
  int groups = 0, group_stride = 0, group_bytes = 0;
};
hipError_t mfma_attn_decode(const bf16_t *qdec, const bf16_t *Kc, const bf16_t *Vc, CacheGeom geom,
                            const int *lens, float *part, bf16_t *out, int nq, int nkv, int batch,
                            int max_chunks, int chunk_keys, int form, const ReadAhead &ahead, hipStream_t s);
size_t mfma_attn_decode_part_floats(int nq, int batch, int max_chunks);
// cache -> plain [len, nkv*128] rows
hipError_t mfma_export_kv(const bf16_t *Kc, const bf16_t *Vc, CacheGeom geom, bf16_t *k_out,
                          bf16_t *v_out, int request, int len, int nkv, hipStream_t s);
hipError_t mfma_fill_zero(void *p, size_t bytes, hipStream_t s);

}  // namespace hyp
