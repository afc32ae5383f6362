// Host check that the split rows start on a 128-byte boundary and end inside their scratch, wherever the scratch
// starts.
#include "gram_split.hip"
#include <cstdio>
int main() {
  for (int64_t n : {1, 7, 128, 1001})
    for (int64_t d : {1, 32, 33, 784})
      for (uintptr_t off = 0; off < 512; off += 4) {
        const uintptr_t base = (uintptr_t)1 << 40;
        const svmx::SplitX s = svmx::split_views(reinterpret_cast<void *>(base + off), n, d);
        const uintptr_t rows = reinterpret_cast<uintptr_t>(s.rows), end = reinterpret_cast<uintptr_t>(s.nrm + n);
        if (rows % 128 || rows < base + off || end > base + off + (uintptr_t)svmx::gram_split_scratch_bytes(n, d) ||
            reinterpret_cast<uintptr_t>(s.scale) < rows + (uintptr_t)(4 * n * s.dp)) {
          printf("FAIL n=%lld d=%lld off=%llu\n", (long long)n, (long long)d, (unsigned long long)off);
          return 1;
        }
      }
  printf("ok\n");
  return 0;
}
