// Limited linear reconstruction of every angle (section 2.2 item ii): the S10
// Voronoi gradient estimator
//   V_i grad phi_i = sum_faces [ (phi_j - phi_i) A c/d + (phi_i + phi_j) A n_out / 2 ]
// (c = face centroid minus the generators' midpoint, d = generator distance), gathered as
//   V_i grad phi_i = sum_faces phi_j e_f + phi_i b_i,
//   e_f = A c/d + A n_out / 2,  b_i = sum_faces (A n_out / 2 - A c/d)
// (the same sum regrouped; e_f and b_i are formed once per mesh in FP64), so each face
// costs three multiply-adds per angle instead of eleven operations;
// then the Barth-Jespersen factor alpha = min(1, (max - phi)/max_f delta_f,
// (min - phi)/min_f delta_f) over the extrapolations delta_f = grad.(r~_f - s_i),
// with max/min over the cell and its face neighbours.  Taking the largest and
// smallest delta and dividing once matches taking the minimum of the per-face
// ratios (division is monotone in the divisor; the reciprocal here is refined to
// within an ulp).
#include "rt_device.h"

namespace {

// The workgroup's cells are consecutive, so their half-faces form one contiguous range;
// its records (the neighbour's weight e_f, the extrapolation offset and the neighbour)
// are staged in LDS once and every lane group reads them from there.  Neighbour rows
// are gathered two faces per batch, all loads of a batch issued before any is used.
// Output: the limited gradient as [N][3][K] (PACKED false), or, for the PLM step's own
// stage 2, each cell and angle's face state (phi, alpha grad phi) in 16-byte parts (PACKED
// true; with split = K/2 the states of angles 0, 2, 4, ... first, then those of 1, 3, 5, ...).
// Bound by the address units of its gathers (FP64 64^3 x 80: 0.29 of 0.39 ms) and the bytes of its
// output; in a full layout (K = LPC APL) a neighbour's elements sit at compile-time
// offsets from one 64-bit multiply-add per face (two PLM steps at 64^3 x 80, FP64 2.63 -> 2.54
// ms).  Two or four consecutive angles per lane (fewer, wider gathers) spread its stores over
// more lines: FP64 2.59 ms with two, FP32 1.34 -> 1.42 with two and 1.79 with four.
template <typename T, int LPC, int APL, bool FULL, bool PACKED>
__global__ __launch_bounds__(RT_BLOCK) void k_gradient(int64_t N, int K, const int32_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ hf_nbr, const void *hf_gp,
                                                       const void *hf_rel, const void *cell_gb,
                                                       const double *__restrict__ vol0,
                                                       const T *__restrict__ I, T *__restrict__ G, int hf_cap,
                                                       int64_t nblk, int split, bool past_caches) {
  using V4 = typename rt_vec4<T>::type;
  constexpr int U = 2;
  constexpr int CPB = RT_BLOCK / LPC;
  extern __shared__ __align__(16) unsigned char rt_smem[];
  V4 *s_gp = (V4 *)rt_smem;        // [hf_cap]: e_f
  V4 *s_rel = s_gp + hf_cap;       // [hf_cap]: r~_f - s_i
  int32_t *s_nbr = (int32_t *)(s_rel + hf_cap);
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  const int64_t c0 = lb * CPB;
  const int64_t c1 = c0 + CPB < N ? c0 + CPB : N;
  const int H0 = row_ptr[c0];
  {
    const V4 *gp = (const V4 *)hf_gp;
    const V4 *rel = (const V4 *)hf_rel;
    const int nH = row_ptr[c1] - H0;  // <= hf_cap by construction
    for (int i = threadIdx.x; i < nH; i += RT_BLOCK) {
      s_gp[i] = gp[H0 + i];
      s_rel[i] = rel[2 * (H0 + i)];
      s_nbr[i] = hf_nbr[H0 + i];
    }
  }
  __syncthreads();
  const int64_t cell = c0 + threadIdx.x / LPC;
  if (cell >= N) return;
  const int l = threadIdx.x % LPC;
  int kk[APL];
  bool ok[APL];
  T s[APL], gx[APL], gy[APL], gz[APL], lo[APL], hi[APL];
  const int64_t row = cell * (int64_t)K;
  const V4 b = ((const V4 *)cell_gb)[cell];
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    const int k = l + LPC * q;
    ok[q] = FULL || k < K;
    kk[q] = ok[q] ? k : 0;
    s[q] = I[row + kk[q]];
    gx[q] = s[q] * b.x;
    gy[q] = s[q] * b.y;
    gz[q] = s[q] * b.z;
    lo[q] = hi[q] = s[q];
  }
  const int h0 = row_ptr[cell], h1 = row_ptr[cell + 1];
  for (int h = h0; h < h1; h += U) {
    // slots past the cell's last face repeat its first face with zero weights; they
    // leave the sums unchanged and re-read a neighbour already in the min/max
    uint32_t j[U];
    V4 e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool v = h + u < h1;
      const int i = (v ? h + u : h0) - H0;
      j[u] = (uint32_t)s_nbr[i];
      e[u] = s_gp[i];
      if (!v) e[u] = V4{T(0), T(0), T(0), T(0)};
    }
    T o[U][APL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T *n = (const T *)((const char *)I + (uint64_t)j[u] * (uint32_t)(K * sizeof(T)));
#pragma unroll
      for (int q = 0; q < APL; ++q) o[u][q] = FULL ? (n + l)[LPC * q] : n[kk[q]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < APL; ++q) {
        gx[q] += o[u][q] * e[u].x;
        gy[q] += o[u][q] * e[u].y;
        gz[q] += o[u][q] * e[u].z;
        lo[q] = fmin(lo[q], o[u][q]);
        hi[q] = fmax(hi[q], o[u][q]);
      }
  }
  const T iv = (T)rt_rcp(vol0[cell]);
  T dmax[APL], dmin[APL];
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    gx[q] *= iv;
    gy[q] *= iv;
    gz[q] *= iv;
    dmax[q] = dmin[q] = T(0);
  }
  for (int h = h0; h < h1; ++h) {
    const V4 r0 = s_rel[h - H0];
#pragma unroll
    for (int q = 0; q < APL; ++q) {
      const T dl = gx[q] * r0.x + gy[q] * r0.y + gz[q] * r0.z;
      dmax[q] = fmax(dmax[q], dl);
      dmin[q] = fmin(dmin[q], dl);
    }
  }
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    if (!ok[q]) continue;
    T al = T(1);
    if (dmax[q] > T(0)) al = fmin(al, (hi[q] - s[q]) * rt_rcp_refined(dmax[q]));
    if (dmin[q] < T(0)) al = fmin(al, (lo[q] - s[q]) * rt_rcp_refined(dmin[q]));
    const int k = kk[q];
    if constexpr (PACKED) {
      using S = rt_state<T>;
      // (asked in every FP64 layout: without the question 60^3 x 20 takes 983 us per two steps instead of 957)
      const int at = (FULL || sizeof(T) == 8) && split ? (k >> 1) + (k & 1 ? split : 0) : k;
      typename S::part *o = (typename S::part *)G + S::PARTS * cell * K + at;
      if (FULL && past_caches) S::template store<true>(o, K, s[q], al * gx[q], al * gy[q], al * gz[q]);
      else S::template store<false>(o, K, s[q], al * gx[q], al * gy[q], al * gz[q]);
    } else {
      G[(cell * 3 + 0) * K + k] = al * gx[q];
      G[(cell * 3 + 1) * K + k] = al * gy[q];
      G[(cell * 3 + 2) * K + k] = al * gz[q];
    }
  }
}

template <typename T, int LPC, int APL, bool FULL, bool PACKED>
hipError_t launch_one(const rt_mesh *m, int K, const void *I, void *G, int split, hipStream_t s) {
  using V4 = typename rt_vec4<T>::type;
  const int64_t cpb = RT_BLOCK / LPC;
  const int64_t nblk = (m->N + cpb - 1) / cpb;
  const void *gp = std::is_same<T, double>::value ? (const void *)m->hf_gp64 : (const void *)m->hf_gp32;
  const void *rel = std::is_same<T, double>::value ? (const void *)m->hf_rel64 : (const void *)m->hf_rel32;
  const void *gb = std::is_same<T, double>::value ? (const void *)m->gb64 : (const void *)m->gb32;
  const int cap = cpb == 16 ? m->hf_cap16 : m->hf_cap32;
  const size_t smem = (2 * sizeof(V4) + sizeof(int32_t)) * (size_t)cap;
  if (smem > (size_t)m->lds_max) return hipErrorInvalidConfiguration;
  // States that outgrow the 256 MB Infinity Cache (with half of it for the rest of the step)
  // are stored past the caches, to leave those to the gathered rows: 335 MB (FP32, 64^3 x 80)
  // 1.38 -> 1.36 ms per two PLM steps and 671 MB (FP64) 2.67 -> 2.63 ms; smaller ones are read
  // back from that cache: 85 MB (FP32, 48^3 x 48) 0.44 ms past the caches, 0.42 ms through them.
  const bool past_caches = PACKED && (int64_t)sizeof(V4) * m->N * K > (int64_t)128 << 20;
  hipLaunchKernelGGL((k_gradient<T, LPC, APL, FULL, PACKED>), dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK), smem,
                     s, m->N, K, m->row_ptr, m->hf_nbr, gp, rel, gb, m->vol0, (const T *)I, (T *)G, cap, nblk,
                     split, past_caches);
  return hipGetLastError();
}

template <typename T, int LPC, int APL, bool PACKED>
hipError_t launch(const rt_mesh *m, int K, const void *I, void *G, int split, hipStream_t s) {
  if (K == LPC * APL) return launch_one<T, LPC, APL, true, PACKED>(m, K, I, G, split, s);
  // Sets that stage 2 takes in pairs fill their lanes here: 8, 24 and 40 angles eight lanes (whose records
  // fit wherever stage 2's larger groups do), multiples of 16 sixteen.  So FP32 states are split in full layouts
  // only (two steps, FP32: 40^3 x 90 410 -> 403 us, 33^3 x 90 256 -> 250).
  if (split) return hipErrorInvalidValue;
  return launch_one<T, LPC, APL, false, PACKED>(m, K, I, G, 0, s);
}

template <typename T, bool PACKED>
hipError_t dispatch16(const rt_mesh *m, int K, const void *I, void *G, int split, hipStream_t s) {
  switch ((K + 15) / 16) {
    case 1: return launch<T, 16, 1, PACKED>(m, K, I, G, split, s);
    case 2: return launch<T, 16, 2, PACKED>(m, K, I, G, split, s);
    case 3: return launch<T, 16, 3, PACKED>(m, K, I, G, split, s);
    case 4: return launch<T, 16, 4, PACKED>(m, K, I, G, split, s);
    case 5: return launch<T, 16, 5, PACKED>(m, K, I, G, split, s);
    case 6: return launch<T, 16, 6, PACKED>(m, K, I, G, split, s);
    case 7: return launch<T, 16, 7, PACKED>(m, K, I, G, split, s);
    case 8: return launch<T, 16, 8, PACKED>(m, K, I, G, split, s);
  }
  return hipErrorInvalidValue;
}

// Small angle sets take 8 lanes per cell (32-cell workgroups); if their half-face
// records do not fit in LDS, 16 lanes (16-cell workgroups) halve the staging.
template <typename T, bool PACKED>
hipError_t dispatch(const rt_mesh *m, int K, const void *I, void *G, int split, hipStream_t s) {
  if (K % 16 == 0 || K > 64) return dispatch16<T, PACKED>(m, K, I, G, split, s);
  hipError_t e = hipErrorInvalidValue;
  switch ((K + 7) / 8) {
    case 1: e = launch<T, 8, 1, PACKED>(m, K, I, G, split, s); break;
    case 2: e = launch<T, 8, 2, PACKED>(m, K, I, G, split, s); break;
    case 3: e = launch<T, 8, 3, PACKED>(m, K, I, G, split, s); break;
    case 4: e = launch<T, 8, 4, PACKED>(m, K, I, G, split, s); break;
    case 5: e = launch<T, 8, 5, PACKED>(m, K, I, G, split, s); break;
    case 6: e = launch<T, 8, 6, PACKED>(m, K, I, G, split, s); break;
    case 7: e = launch<T, 8, 7, PACKED>(m, K, I, G, split, s); break;
    case 8: e = launch<T, 8, 8, PACKED>(m, K, I, G, split, s); break;
  }
  return e == hipErrorInvalidConfiguration ? dispatch16<T, PACKED>(m, K, I, G, split, s) : e;
}

}  // namespace

hipError_t rt_launch_gradient(const rt_mesh *m, int K, const void *I, void *grad, int dtype, bool packed, int split,
                              hipStream_t s) {
  if (packed)
    return dtype == RT_F32 ? dispatch<float, true>(m, K, I, grad, split, s)
                           : dispatch<double, true>(m, K, I, grad, split, s);
  return dtype == RT_F32 ? dispatch<float, false>(m, K, I, grad, 0, s) : dispatch<double, false>(m, K, I, grad, 0, s);
}
