// half_face_scan.cpp -- TEST INFRASTRUCTURE: the loss kernel's walk over a range of half-faces, also one
// that ends at the most a mesh may have (2^31 - 1): every half-face once, nothing else read, and an
// end.  Exits non-zero on any failure.
#include <stdint.h>
#include <stdio.h>

#include <vector>

#include "rt_scan.h"

static int walk(int32_t h0, int32_t h1) {
  constexpr int THREADS = 256, B = 4;
  const int64_t n = (int64_t)h1 - h0;
  std::vector<int> seen((size_t)n, 0);
  for (uint32_t t = 0; t < THREADS; ++t) {
    int64_t batches = 0;
    bool ok = true;
    rt_scan_half_faces<THREADS, B>(h0, h1, t, [&](const uint32_t (&h)[B]) {
      if (++batches > n / (THREADS * B) + 1) {
        printf("thread %u does not end at [%d, %d)\n", t, h0, h1);
        __builtin_trap();
      }
      for (int b = 0; b < B; ++b) {
        const int64_t at = (int64_t)h[b] - h0;
        if (at < 0 || at >= n) ok = false;
        else if (b == 0 || h[b] != h[0]) ++seen[(size_t)at];
      }
    });
    if (!ok) {
      printf("thread %u leaves [%d, %d)\n", t, h0, h1);
      return 1;
    }
  }
  for (int64_t i = 0; i < n; ++i)
    if (seen[(size_t)i] != 1) {
      printf("half-face %lld of [%d, %d) taken %d times\n", (long long)(h0 + i), h0, h1, seen[(size_t)i]);
      return 1;
    }
  return 0;
}

int main() {
  int bad = 0;
  for (int32_t n : {0, 1, 255, 256, 257, 1023, 1024, 1025, 3000, 5121})
    for (int32_t h0 : {0, 12345, INT32_MAX - n - 1, INT32_MAX - n}) bad |= walk(h0, h0 + n);
  if (bad) return 1;
  printf("half-face scan OK\n");
  return 0;
}
