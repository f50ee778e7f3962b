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
    } else {
      return 1;
    }
  }
  return 0;
}
