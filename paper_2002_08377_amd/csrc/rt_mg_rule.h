// Which kernel a multigroup step of a set with antipodal pairs takes where its paired layout does not
// fit (rows of the groups that wait in LDS, half of it at most): the one-kernel step in the general
// layout, or the separate launches in the paired one.  Host only.
#pragma once
#include <stddef.h>
#include <stdint.h>

// lanes per cell, angles per lane and LDS of the general layout; elem: bytes of an intensity.
//
// The one kernel is ahead wherever three of its workgroups fit in a CU, and on meshes of up to 32^3
// cells, which do not fill the chip (times of the separate launches over its: FP64 K = 80, 5 to 8
// groups 2.1 at 12^3, 1.2 at 32^3, 1.04 to 1.08 at 48^3; FP32 K = 80, 9 groups 2.1, 1.4, 1.25; 12 and 15
// groups 2.3, 1.15 and FP64 K = 48, 10 and 12 groups 2.3, 1.08 at 12^3 and 32^3).  With two workgroups per
// CU on larger meshes it is a matter of what a lane has in flight against what the separate launches
// do with the same set: at 48^3 and 56^3, FP64 K = 80 (5 angles per lane) 8 groups 1.06, 1.09; FP32 K = 48
// (3) 16 groups 1.11 at 40^3, 1.01; 8 lanes per cell, FP64 K = 24, 8 and 10 groups 1.08; but FP32
// K = 80 (5) 12 groups 0.98, 0.95, 15 groups 0.97, 0.93; FP64 K = 48 (3) 10 groups 0.91, 12 groups 0.91, 0.90.
static inline bool rt_mg_general_step(int lanes, int angles, size_t elem, int64_t cells, size_t lds, size_t lds_max) {
  if (cells <= 32768 || lds <= lds_max / 3 || lanes < 16) return true;
  return elem == 8 ? angles >= 5 : angles <= 3;
}
