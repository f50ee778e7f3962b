// Answers questions on the launch rules, one a line on stdin, one line each on stdout.
#include <stdio.h>
#include <string.h>

#include "launch_rules.h"

int main() {
  char what[16];
  while (scanf("%15s", what) == 1) {
    if (!strcmp(what, "attn")) {
      int esize, d, longest;
      size_t pairs;
      if (scanf("%d %d %zu %d", &esize, &d, &pairs, &longest) != 4) return 1;
      printf("%d\n", hyp::plain_attn_split(esize, d, pairs, longest));
    } else if (!strcmp(what, "gemv")) {
      int cls, N, K, batch;
      if (scanf("%d %d %d %d", &cls, &N, &K, &batch) != 4) return 1;
      const hyp::GemvPlan g = hyp::mfma_gemv_plan(cls, N, K, batch);
      printf("%d %d %d %d\n", g.fbw, g.nw, g.ksplit, g.tail);
    } else if (!strcmp(what, "window")) {
      int cls, N, K, batch;
      if (scanf("%d %d %d %d", &cls, &N, &K, &batch) != 4) return 1;
      printf("%d\n", hyp::mfma_gemv_one_window(hyp::mfma_gemv_plan(cls, N, K, batch), N, K) ? 1 : 0);
    } else if (!strcmp(what, "chunk")) {
      int max_seq, pairs, even;
      if (scanf("%d %d %d", &max_seq, &pairs, &even) != 3) return 1;
      printf("%d\n", hyp::mfma_decode_chunk_keys(max_seq, pairs, even != 0));
    } else if (!strcmp(what, "direct")) {
      int blocks;
      size_t bytes;
      if (scanf("%d %zu", &blocks, &bytes) != 2) return 1;
      printf("%d\n", hyp::decode_step_direct(blocks, bytes) ? 1 : 0);
    } else if (!strcmp(what, "gemm")) {
      int rows, N, K, swiglu;
      if (scanf("%d %d %d %d", &rows, &N, &K, &swiglu) != 4) return 1;
      const hyp::GemmCut g = hyp::mfma_gemm_cut(rows, N, K, swiglu != 0);
      printf("%d %d %d %d %d %d %d %d %d %d\n", g.form, g.tiles_t, g.n_tiles, g.first, g.ksplit, g.finish ? 1 : 0, g.n_static, g.pool_wgs, g.first_grid,
             g.rest_grid);
    } else {
      return 1;
    }
  }
  return 0;
}
