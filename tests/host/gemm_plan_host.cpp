// Host driver for the rules that choose a GEMM's kernel: reads lines
// "variant act grouped M N K lda ldb" and prints "small tm tn split" (small: the
// few-token forward).
#include <cstdio>

#include "gemm_plan.h"

using namespace lrqat;

int main() {
  int v, act, grouped;
  long long M, N, K, lda, ldb;
  while (std::scanf("%d %d %d %lld %lld %lld %lld %lld", &v, &act, &grouped, &M, &N, &K, &lda, &ldb) == 8) {
    const GemmVariant gv = GemmVariant(v);
    const GemmPlan g = gemm_plan(gv, act, grouped, gemm_al16(gv, act, K, lda, ldb), M, N, K);
    std::printf("%d %d %d %d\n", gv == kFwd && fwd_small(M, N), g.tm, g.tn, g.split);
  }
  return 0;
}
