// The walk of one thread of a workgroup over a range of half-faces, host and device alike.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define RT_HD __host__ __device__ __forceinline__
#else
#define RT_HD inline
#endif

// Calls batch(h) for the half-faces [h0, h1) of thread `t` of THREADS, B at a time, THREADS apart;
// slots past the end repeat the batch's first.  The indices are unsigned: a mesh may have up to
// 2^31 - 1 half-faces, and the step past the last of them (B THREADS further) has to stay above h1.
template <int THREADS, int B, typename Fn> RT_HD void rt_scan_half_faces(int32_t h0, int32_t h1, uint32_t t, Fn batch) {
  const uint32_t end = (uint32_t)h1;
  for (uint32_t h = (uint32_t)h0 + t; h < end; h += (uint32_t)(B * THREADS)) {
    uint32_t at[B];
#pragma unroll
    for (int b = 0; b < B; ++b) at[b] = h + (uint32_t)(b * THREADS) < end ? h + (uint32_t)(b * THREADS) : h;
    batch(at);
  }
}
