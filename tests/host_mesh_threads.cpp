// host_mesh_threads.cpp -- TEST INFRASTRUCTURE: the host half of the mesh upload on a mesh large
// enough for a team of threads, its faces in shuffled order, against a plain serial
// recomputation; and which of several defects is reported.  Exits non-zero on any failure.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "rt_mesh_host.h"

static int failures = 0;
static void check(bool ok, const char *what) {
  if (!ok) {
    fprintf(stderr, "FAIL: %s\n", what);
    ++failures;
  }
}

int main() {
  const int n = 45;  // 91,125 cells (a last group of 53), 273,375 faces
  const int64_t N = (int64_t)n * n * n;
  const double h = 1.0 / n;
  struct Face {
    int32_t i, j;
    int axis;
    double area;
  };
  std::vector<Face> faces;
  for (int64_t c = 0; c < N; ++c)
    for (int ax = 0; ax < 3; ++ax) {
      int t[3] = {(int)(c % n), (int)(c / n % n), (int)(c / ((int64_t)n * n))};
      t[ax] = (t[ax] + 1) % n;
      const int32_t j = t[0] + n * (t[1] + n * t[2]);
      const int parts = (c * 7 + ax) % 11 == 0 ? 3 : 1;  // face counts vary
      for (int p = 0; p < parts; ++p) faces.push_back({(int32_t)c, j, ax, h * h / parts});
    }
  std::mt19937 rng(7);
  std::shuffle(faces.begin(), faces.end(), rng);
  const int64_t F = (int64_t)faces.size();
  std::vector<double> vol((size_t)N, h * h * h), area, normal, pos((size_t)(3 * N), 0.5);
  std::vector<int32_t> fc;
  std::vector<int8_t> shift((size_t)(3 * F), 0);
  for (const Face &f : faces) {
    fc.push_back(f.i);
    fc.push_back(f.j);
    area.push_back(f.area);
    for (int a = 0; a < 3; ++a) normal.push_back(a == f.axis ? 1.0 : 0.0);
  }
  auto build = [&](rt_host_mesh &m) {
    const rt_finite_check fin[] = {{pos.data(), 3 * N, "first"}, {pos.data(), 3 * N, "second"}};
    return rt_build_host_mesh(N, F, vol.data(), fc.data(), shift.data(), area.data(), normal.data(), m, fin, 2);
  };
  rt_host_mesh m;
  check(build(m).empty(), "a closed lattice is accepted");
  std::vector<std::vector<int32_t>> ref((size_t)N);
  for (int64_t f = 0; f < F; ++f) {
    ref[(size_t)fc[(size_t)(2 * f)]].push_back((int32_t)f);
    ref[(size_t)fc[(size_t)(2 * f + 1)]].push_back((int32_t)(-f - 1));
  }
  bool same = m.row_ptr[0] == 0;
  for (int64_t c = 0; c < N; ++c)
    same = same && std::vector<int32_t>(m.hf_face.begin() + m.row_ptr[(size_t)c], m.hf_face.begin() + m.row_ptr[(size_t)c + 1]) == ref[(size_t)c];
  check(same, "half-faces by cell, in input order");
  auto orders = [&](int cpb, const std::vector<uint8_t> &o, int32_t cap) {
    int32_t most = 0;
    bool ok = (int64_t)o.size() == N;
    for (int64_t c = 0; c < N && ok; c += cpb) {
      const int k = (int)std::min<int64_t>(cpb, N - c);
      std::vector<int> want((size_t)k);
      int32_t total = 0;
      for (int g = 0; g < k; ++g) {
        want[(size_t)g] = g;
        total += (int32_t)ref[(size_t)(c + g)].size();
      }
      most = std::max(most, total);
      std::stable_sort(want.begin(), want.end(), [&](int x, int y) { return ref[(size_t)(c + x)].size() < ref[(size_t)(c + y)].size(); });
      for (int g = 0; g < k; ++g) ok = ok && o[(size_t)(c + g)] == want[(size_t)g];
    }
    check(ok, "cells by face count");
    check(cap == most, "staging size");
  };
  orders(16, m.order16, m.hf_cap16);
  orders(32, m.order32, m.hf_cap32);
  orders(64, m.order64, m.hf_cap64);
  // the first of several defects is the one named, whichever thread finds it
  rt_host_mesh w;
  area[(size_t)(F - 5)] = -1.0;
  normal[(size_t)(3 * (F / 2))] = 2.0;
  check(build(w) == "face " + std::to_string(F / 2) + " normal is not unit", "the first bad face");
  vol[(size_t)(N - 1)] = 0.0;
  vol[(size_t)(N - 2)] = NAN;
  check(build(w) == "cell " + std::to_string(N - 2) + " has volume <= 0", "volumes before faces");
  pos[(size_t)(3 * N - 1)] = INFINITY;
  check(build(w) == "first has a non-finite entry (index " + std::to_string(3 * N - 1) + ")", "entries before volumes");
  if (failures) return 1;
  printf("host mesh threads OK\n");
  return 0;
}
