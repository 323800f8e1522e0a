// Host program of tests/test_scored_queries.py: reads "nw n_q" and the 2 * nw
// owner words of a workgroup per line, prints what scored_queries makes of
// them. Nothing of it runs on a GPU.
#include <cstdio>

#include "../paper_2606_26439_amd/csrc/fused_impl.h"

int main() {
  int nw;
  long long n_q;
  while (scanf("%d %lld", &nw, &n_q) == 2) {
    int64_t owners[32], a0 = 7, a1 = 7;
    for (int i = 0; i < 2 * nw; ++i) {
      long long v;
      if (scanf("%lld", &v) != 1) return 1;
      owners[i] = v;
    }
    const bool any = fused_detail::scored_queries(owners, nw, n_q, a0, a1);
    printf("%d %lld %lld\n", any ? 1 : 0, (long long)a0, (long long)a1);
  }
  return 0;
}
