// mg_rule.cpp -- TEST INFRASTRUCTURE: the multigroup step's choice between the general one-kernel form
// and the separate launches for sets with antipodal pairs, against the faster of the two at measured
// sizes.  LDS as the launch computes it, at 300 half-faces of 16 cells and 600 of 32.
#include <stdio.h>

#include "rt_mg_rule.h"

int main() {
  const struct {
    int lanes, angles;
    size_t elem;
    int groups, n;
    double ratio;  // time of the separate launches over the one kernel's
  } seen[] = {
      {16, 5, 8, 5, 12, 2.07}, {16, 5, 8, 5, 48, 1.04}, {16, 5, 8, 6, 56, 1.08}, {16, 5, 8, 8, 48, 1.06}, {16, 5, 8, 8, 56, 1.09},
      {16, 5, 4, 9, 12, 2.11}, {16, 5, 4, 9, 56, 1.21}, {16, 5, 4, 12, 24, 1.35}, {16, 5, 4, 12, 32, 1.15}, {16, 5, 4, 12, 48, 0.98},
      {16, 5, 4, 12, 56, 0.95}, {16, 5, 4, 15, 32, 1.15}, {16, 5, 4, 15, 48, 0.97}, {16, 5, 4, 15, 56, 0.93}, {16, 3, 8, 8, 56, 1.11},
      {16, 3, 8, 10, 32, 1.08}, {16, 3, 8, 10, 40, 0.95}, {16, 3, 8, 10, 48, 0.91}, {16, 3, 8, 12, 56, 0.90}, {16, 3, 4, 16, 40, 1.11},
      {16, 3, 4, 16, 56, 1.01}, {8, 3, 8, 8, 56, 1.08}, {8, 3, 8, 10, 56, 1.08},
  };
  int bad = 0;
  for (const auto &s : seen) {
    const size_t cells = 256 / s.lanes, faces = cells == 16 ? 300 : 600;
    const size_t lds = (4 * s.elem + 4) * faces + 24 * s.groups * cells + s.elem * s.angles * 256 * (s.groups - 2);
    const bool one = rt_mg_general_step(s.lanes, s.angles, s.elem, (int64_t)s.n * s.n * s.n, lds, 163840);
    if (one != (s.ratio >= 1.0)) {
      printf("%d lanes, %d angles, %zu bytes, %d groups, %d^3: %s is taken at %.2f\n", s.lanes, s.angles, s.elem, s.groups, s.n,
             one ? "the one kernel" : "separate launches", s.ratio);
      ++bad;
    }
  }
  if (bad) return 1;
  printf("multigroup rule OK\n");
  return 0;
}
