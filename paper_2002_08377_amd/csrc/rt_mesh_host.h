// Host half of the mesh upload (section 2: cells and faces of the tessellation): the
// checks of the input tessellation, the half-face index grouped by cell that every cell
// gathers its fluxes through, and the per-workgroup staging sizes and cell orders of the
// kernels.  Plain C++17 with no HIP, so that a host-only build can run it under sanitizers.
#pragma once

#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <atomic>
#include <new>
#include <string>
#include <thread>
#include <vector>

struct rt_host_mesh {
  std::vector<int32_t> row_ptr;  // [N+1]: half-faces of cell i are [row_ptr[i], row_ptr[i+1])
  std::vector<int32_t> hf_face;  // [2F]: face f for its first cell, -(f+1) for its second, in input order
  int32_t hf_cap16 = 0;          // most half-faces of any 16 / 32 / 64 consecutive cells
  int32_t hf_cap32 = 0;
  int32_t hf_cap64 = 0;
  // within every run of 16 / 32 / 64 consecutive cells, position g holds the offset of the
  // cell with the g-th smallest face count (a stable order), so each wave's cells pad alike
  std::vector<uint8_t> order16, order32, order64;
};

// An array of n doubles that must be finite, and what to call it.
struct rt_finite_check {
  const double *p;
  int64_t n;
  const char *what;
};

// A team of threads running one function, meeting at a barrier between its phases.  A mesh
// program re-tessellates between steps, so the upload is on its per-step path: at 64,000
// cells and 501,000 faces the checks and the index took 6.1 ms on one thread.  Small meshes
// stay on the calling thread (a team costs about 0.1 ms to start).
class rt_team {
 public:
  explicit rt_team(int64_t items) {
    const unsigned hw = std::thread::hardware_concurrency();
    const int64_t most = hw < 2 ? 1 : hw < 8 ? hw : 8;
    want_ = (int)std::max<int64_t>(1, std::min<int64_t>(most, items / 32768));
  }
  // fn(thread, threads) on every thread (at most wanted() of them); fn must not throw
  template <typename Fn> void run(Fn fn) {
    size_ = want_;
    std::vector<std::thread> others;
    std::atomic<int> go{0};
    try {
      others.reserve((size_t)want_);
      for (int t = 1; t < want_; ++t)
        others.emplace_back([&, t] {
          while (go.load(std::memory_order_acquire) == 0) std::this_thread::yield();
          if (t < size_) fn(t, size_);
        });
    } catch (...) {  // fewer threads than wanted
      size_ = 1 + (int)others.size();
    }
    go.store(1, std::memory_order_release);
    fn(0, size_);
    for (std::thread &o : others) o.join();
  }
  int wanted() const { return want_; }
  void meet() {
    const int phase = phase_.load(std::memory_order_acquire);
    if (here_.fetch_add(1, std::memory_order_acq_rel) + 1 == size_) {
      here_.store(0, std::memory_order_relaxed);
      phase_.store(phase + 1, std::memory_order_release);
    } else {
      while (phase_.load(std::memory_order_acquire) == phase) std::this_thread::yield();
    }
  }

 private:
  int want_ = 1, size_ = 1;
  std::atomic<int> here_{0}, phase_{0};
};

// Checks the tessellation and fills `out`.  Returns "" on success, else the reason (the
// first bad entry): a non-finite entry of `finite`, volume <= 0, face cells out of range or
// equal, area <= 0, non-unit normal, periodic shift outside {-1, 0, 1}, a cell whose faces do
// not close (|sum A n| > 1e-8 V^(2/3)).  N, F >= 1 and 2F < 2^31 are the caller's to check.
// The result does not depend on the number of threads.
inline std::string rt_build_host_mesh(int64_t N, int64_t F, const double *vol, const int32_t *face_cells,
                                      const int8_t *face_shift, const double *face_area, const double *face_normal,
                                      rt_host_mesh &out, const rt_finite_check *finite = nullptr, int n_finite = 0) {
  constexpr int64_t NONE = INT64_MAX;
  std::vector<std::atomic<int64_t>> bad_entry((size_t)n_finite);
  for (auto &b : bad_entry) b.store(NONE, std::memory_order_relaxed);
  std::atomic<int64_t> bad_vol{NONE}, bad_face{NONE}, bad_close{NONE};
  auto lower = [](std::atomic<int64_t> &a, int64_t v) {
    int64_t cur = a.load(std::memory_order_relaxed);
    while (v < cur && !a.compare_exchange_weak(cur, v, std::memory_order_relaxed)) {
    }
  };
  // why face f is refused, or null
  auto face_fault = [&](int64_t f) -> const char * {
    const int32_t i = face_cells[2 * f], j = face_cells[2 * f + 1];
    if (i < 0 || j < 0 || i >= N || j >= N || i == j) return "cells";
    const double A = face_area[f];
    if (!(A > 0.0) || !isfinite(A)) return "area";
    const double *n = &face_normal[3 * f];
    const double nn = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    if (!(fabs(nn - 1.0) < 1e-10)) return "normal";
    for (int c = 0; c < 3; ++c)
      if (face_shift[3 * f + c] < -1 || face_shift[3 * f + c] > 1) return "shift";
    return nullptr;
  };
  auto closure = [&](int64_t i) {
    double c[3] = {0.0, 0.0, 0.0};
    for (int32_t h = out.row_ptr[(size_t)i]; h < out.row_ptr[(size_t)i + 1]; ++h) {
      const int32_t code = out.hf_face[(size_t)h];
      const int64_t f = code >= 0 ? code : -(int64_t)code - 1;
      const double A = face_area[f], *n = &face_normal[3 * f];
      for (int d = 0; d < 3; ++d) c[d] += code >= 0 ? A * n[d] : -(A * n[d]);
    }
    return sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
  };
  out.row_ptr.assign((size_t)N + 1, 0);
  out.hf_face.resize(2 * (size_t)F);
  out.order16.resize((size_t)N);
  out.order32.resize((size_t)N);
  out.order64.resize((size_t)N);
  // per thread: its faces of each cell, then where it writes the next of them.  Threads take
  // consecutive faces, so a cell's faces come out in input order, and no two threads write to
  // one place (with one shared array of atomics the count and the fill took 1.3 of 2.6 ms at
  // 64,000 cells, and the cells had to be sorted afterwards).
  rt_team team(F);
  std::vector<std::vector<int32_t>> own((size_t)team.wanted());
  std::atomic<bool> no_memory{false};
  std::vector<int32_t> base((size_t)team.wanted() + 1, 0);
  std::atomic<int32_t> cap16{0}, cap32{0}, cap64{0};
  auto raise = [](std::atomic<int32_t> &a, int32_t v) {
    int32_t cur = a.load(std::memory_order_relaxed);
    while (v > cur && !a.compare_exchange_weak(cur, v, std::memory_order_relaxed)) {
    }
  };
  team.run([&](int t, int T) {
    // this thread's share of n items, a multiple of 64 at both ends
    auto from = [&](int64_t n) { return std::min(n, (n / T + 64) / 64 * 64 * (int64_t)t); };
    auto to = [&](int64_t n) { return t == T - 1 ? n : std::min(n, (n / T + 64) / 64 * 64 * (int64_t)(t + 1)); };
    try {
      own[(size_t)t].assign((size_t)N, 0);
    } catch (...) {
      no_memory = true;
    }
    int32_t *mine = own[(size_t)t].data();
    // 1. entries, volumes and faces; faces per cell
    for (int a = 0; a < n_finite; ++a)
      for (int64_t k = from(finite[a].n), e = to(finite[a].n); k < e; ++k)
        if (!isfinite(finite[a].p[k])) {
          lower(bad_entry[(size_t)a], k);
          break;
        }
    for (int64_t i = from(N), e = to(N); i < e; ++i)
      if (!(vol[i] > 0.0) || !isfinite(vol[i])) {
        lower(bad_vol, i);
        break;
      }
    for (int64_t f = from(F), e = no_memory ? 0 : to(F); f < e; ++f) {
      if (face_fault(f)) {
        lower(bad_face, f);
        break;
      }
      ++mine[face_cells[2 * f]];
      ++mine[face_cells[2 * f + 1]];
    }
    team.meet();
    if (no_memory || bad_vol != NONE || bad_face != NONE) return;
    // 2. half-faces grouped by cell
    {
      int32_t total = 0;
      for (int64_t i = from(N), e = to(N); i < e; ++i)
        for (int k = 0; k < T; ++k) total += own[(size_t)k][(size_t)i];
      base[(size_t)t + 1] = total;
    }
    team.meet();
    {
      int32_t at = 0;
      for (int k = 0; k <= t; ++k) at += base[(size_t)k];
      for (int64_t i = from(N), e = to(N); i < e; ++i) {
        out.row_ptr[(size_t)i] = at;
        for (int k = 0; k < T; ++k) {
          const int32_t n = own[(size_t)k][(size_t)i];
          own[(size_t)k][(size_t)i] = at;
          at += n;
        }
      }
      if (t == T - 1) out.row_ptr[(size_t)N] = at;
    }
    team.meet();
    for (int64_t f = from(F), e = to(F); f < e; ++f) {
      out.hf_face[(size_t)mine[face_cells[2 * f]]++] = (int32_t)f;
      out.hf_face[(size_t)mine[face_cells[2 * f + 1]]++] = (int32_t)(-f - 1);
    }
    team.meet();
    // 3. per 64 cells: closure, the staging sizes, and the cells by face count
    auto faces = [&](int64_t c) { return out.row_ptr[(size_t)c + 1] - out.row_ptr[(size_t)c]; };
    for (int64_t c0 = from(N), e = to(N); c0 < e; c0 += 64) {
      const int64_t c1 = std::min(c0 + 64, N);
      for (int64_t c = c0; c < c1; ++c)
        if (!(closure(c) <= 1e-8 * pow(vol[c], 2.0 / 3.0))) lower(bad_close, c);
      auto span = [&](int64_t b, int cpb) {
        return out.row_ptr[(size_t)std::min(b + cpb, N)] - out.row_ptr[(size_t)b];
      };
      raise(cap64, span(c0, 64));
      for (int64_t b = c0; b < c1; b += 32) raise(cap32, span(b, 32));
      for (int64_t b = c0; b < c1; b += 16) raise(cap16, span(b, 16));
      // runs of 16 by insertion, then pairs of runs merged (both keep equal counts in order)
      for (int64_t b = c0; b < c1; b += 16) {
        uint8_t *o = out.order16.data() + b;
        const int n = (int)std::min<int64_t>(16, N - b);
        for (int g = 0; g < n; ++g) {
          int k = g;
          for (; k > 0 && faces(b + o[k - 1]) > faces(b + g); --k) o[k] = o[k - 1];
          o[k] = (uint8_t)g;
        }
      }
      auto merge = [&](const std::vector<uint8_t> &in, std::vector<uint8_t> &ord, int cpb) {
        for (int64_t b = c0; b < c1; b += cpb) {
          const int n = (int)std::min<int64_t>(cpb, N - b), half = std::min(cpb / 2, n);
          int x = 0, y = half;
          for (int g = 0; g < n; ++g) {
            const int cx = x < half ? in[(size_t)(b + x)] : 0, cy = y < n ? half + in[(size_t)(b + y)] : 0;
            const bool first = y >= n || (x < half && faces(b + cx) <= faces(b + cy));
            ord[(size_t)(b + g)] = (uint8_t)(first ? cx : cy);
            if (first) ++x;
            else ++y;
          }
        }
      };
      merge(out.order16, out.order32, 32);
      merge(out.order32, out.order64, 64);
    }
  });
  if (no_memory) throw std::bad_alloc();
  char buf[256];
  for (int a = 0; a < n_finite; ++a)
    if (bad_entry[(size_t)a] != NONE) {
      snprintf(buf, sizeof buf, "%s has a non-finite entry (index %lld)", finite[a].what, (long long)bad_entry[(size_t)a]);
      return buf;
    }
  if (bad_vol != NONE) {
    snprintf(buf, sizeof buf, "cell %lld has volume <= 0", (long long)bad_vol);
    return buf;
  }
  if (bad_face != NONE) {
    const int64_t f = bad_face;
    const char why = *face_fault(f);
    if (why == 'c')
      snprintf(buf, sizeof buf, "face %lld has invalid cells (%d, %d)", (long long)f, face_cells[2 * f], face_cells[2 * f + 1]);
    else if (why == 'a')
      snprintf(buf, sizeof buf, "face %lld has area <= 0", (long long)f);
    else if (why == 'n')
      snprintf(buf, sizeof buf, "face %lld normal is not unit", (long long)f);
    else
      snprintf(buf, sizeof buf, "face %lld shift outside {-1,0,1}", (long long)f);
    return buf;
  }
  if (bad_close != NONE) {
    snprintf(buf, sizeof buf, "cell %lld is not closed: |sum A n| = %g", (long long)bad_close, closure(bad_close));
    return buf;
  }
  out.hf_cap16 = cap16;
  out.hf_cap32 = cap32;
  out.hf_cap64 = cap64;
  return std::string();
}
