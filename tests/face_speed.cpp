// face_speed.cpp -- TEST INFRASTRUCTURE: the speed of a face along the antipode of a direction, against
// the speed along that direction formed on its own and against 128-bit values.  Exits non-zero on any
// failure.
#include <stdint.h>
#include <stdio.h>

#include "rt_face_speed.h"

static uint64_t state = 88172645463325252ull;
static double uniform() {  // in [-1, 1)
  state ^= state << 13;
  state ^= state >> 7;
  state ^= state << 17;
  return (double)(int64_t)state * 0x1p-63;
}

int main() {
  double sum = 0.0, sum_anti = 0.0;
  for (int i = 0; i < 1000000; ++i) {
    const double ax = uniform(), ay = uniform(), az = uniform(), nb = 0.1 * uniform();
    const double x = uniform(), y = uniform(), z = uniform();
    const double g = rt_face_speed(ax, ay, az, nb, x, y, z);
    const double g2 = rt_antipode_speed(ax, ay, az, nb, x, y, z);
    if (g2 != rt_face_speed(ax, ay, az, nb, -x, -y, -z)) {
      printf("case %d: the antipode's speed is not the speed along it\n", i);
      return 1;
    }
    const __float128 dot = (__float128)ax * x + (__float128)ay * y + (__float128)az * z;
    const double e = (double)(g - (dot + nb)), e2 = (double)(g2 - (-dot + nb));
    sum += e * e;
    sum_anti += e2 * e2;
  }
  // the mean square errors of equal sums of a million terms agree to a fraction of a percent
  if (sum_anti > 1.02 * sum) {
    printf("mean square error %g of the antipode's speed, %g of the direction's\n", sum_anti, sum);
    return 1;
  }
  printf("face speed OK\n");
  return 0;
}
