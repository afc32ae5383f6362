// Host check of the rule that takes few test samples to one pass over the training rows: the pass where it
// was measured to be the faster way, tiles where it was not.
#include "few_rule.hpp"
#include <cstdio>
struct Case { int64_t k, per, d, m; bool pass; };
int main() {
  const Case cases[] = {
      // one problem: always the pass, up to 16 samples
      {1, 1000, 16, 1, true}, {1, 20000, 784, 16, true}, {1, 1000000, 301, 16, true}, {1, 1000, 16, 17, false},
      // small one-vs-one models, and one sample of any
      {3, 300, 16, 16, true}, {10, 100, 16, 16, true}, {64, 100, 100, 16, true}, {10, 300, 784, 4, true},
      {10, 6000, 784, 1, true}, {20, 3000, 784, 1, true}, {64, 500, 784, 1, true}, {3, 60000, 784, 4, true},
      // many pairs that share long rows
      {10, 300, 784, 5, false}, {10, 1000, 784, 4, false}, {10, 1000, 784, 16, false}, {10, 6000, 784, 2, false},
      {10, 6000, 784, 16, false}, {10, 6000, 128, 5, false}, {5, 2000, 300, 5, false}, {20, 3000, 784, 2, false},
      {30, 1000, 300, 2, false}, {64, 500, 784, 2, false}, {64, 500, 784, 16, false}, {3, 60000, 784, 12, false},
      {3, 300, 16, 17, false},
  };
  for (const Case &c : cases) {
    const int64_t problems = c.k == 1 ? 1 : c.k * (c.k - 1) / 2, n = c.k * c.per, rows = c.k == 1 ? n : (c.k - 1) * n;
    if (svmx::predict_few_pays(problems, rows, n, c.d, c.m) != c.pass) {
      printf("FAIL k=%lld per=%lld d=%lld m=%lld\n", (long long)c.k, (long long)c.per, (long long)c.d, (long long)c.m);
      return 1;
    }
  }
  printf("ok\n");
  return 0;
}
