// Evaluates the product rules of gemm_plan.h: each line of standard input is one
// question, each line of standard output its answer (see tests/test_product_plan.py).
#include <cstdio>
#include <cstring>

#include "gemm_plan.h"

using namespace wici;

int main() {
  char what[16];
  int a[6];
  while (std::scanf("%15s", what) == 1) {
    for (int i = 0; i < 6; ++i)
      if (std::scanf("%d", &a[i]) != 1) return 1;
    const int wt = a[0], nt = a[1], M = a[2], N = a[3], K = a[4], n = a[5];
    if (!std::strcmp(what, "ranges")) {  // at most n: count, kernel, and the kernel for that count
      const int c = gemm_split_count(wt, nt, M, N, K, n);
      std::printf("%d %d %d\n", c, gemm_rows_best(wt, nt, M, N, K, n),
                  gemm_rows_best(wt, nt, M, N, K, c));
    } else if (!std::strcmp(what, "rows")) {  // the few-row launch of a product in at most n ranges
      const RowsPlan p = rows_plan(wt, GEMV_STORE, M, N, K, kAddedOutside, n);
      std::printf("%d %d %d\n", p.tm, p.wn, p.nsplit);
    } else if (!std::strcmp(what, "merge")) {
      std::printf("%d\n", gemm_rows_merge_best(wt, nt, M, N, K));
    } else if (!std::strcmp(what, "tile") || !std::strcmp(what, "tileg")) {  // (g: SwiGLU)
      // bf16 weights, in n ranges: the shape, and every shape's time in ns
      const bool g = what[4] == 'g';
      std::printf("%d", tile_shape(nt, M, N, K, n, g));
      for (int s = 0; s < kTileShapes; ++s)
        std::printf(" %.0f", 1e3 * tile_time(s, g, nt, M, N, K, n));
      std::printf("\n");
    } else if (!std::strcmp(what, "fit") || !std::strcmp(what, "fitg")) {  // per tile: size, fit
      for (int s = 0; s < kTileShapes; ++s) {
        const Tile& t = tile_of(s, what[3] == 'g');
        std::printf("%d %d %d ", t.bm, t.bn, t.fit[nt - 1]);
      }
      std::printf("\n");
    } else {
      return 1;
    }
  }
  return 0;
}
