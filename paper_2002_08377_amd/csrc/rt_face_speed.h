// The speed of a face along a direction n: dt (cbar (A n_out).n - A (w~.n)_out), the charge leaving a
// cell through it per unit upwind intensity, with a = dt cbar A n_out and nb = -dt A (w~.n)_out.  Plain
// C++ so that the host can build it too.
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define RT_HD __host__ __device__ __forceinline__
#else
#include <math.h>
#define RT_HD inline
#endif

template <typename T> RT_HD T rt_face_speed(T ax, T ay, T az, T nb, T x, T y, T z) {
  return fma(az, z, fma(ay, y, fma(ax, x, nb)));
}

// The same along -n, by three multiply-adds of its own (2 nb - g would add the rounding of that difference
// to the rounding of g: half as much again in the mean square).
template <typename T> RT_HD T rt_antipode_speed(T ax, T ay, T az, T nb, T x, T y, T z) {
  return rt_face_speed(ax, ay, az, nb, -x, -y, -z);
}
