// Grid reductions: conservation diagnostics (section 2.3.1) and the emergent-flux
// loss with its seed; and the per-cell angle moments (section 2.1), reduced over each
// cell's lanes only.  The lanes add their own terms over their cells, each workgroup
// reduces over its lanes, then one or two folds over the per-workgroup partials in a
// fixed order, so results are deterministic (no atomics).
#include <mutex>

#include "rt_device.h"
#include "rt_scan.h"

// Scratch of the loss that allocates nothing: the per-workgroup partial sums in its first
// RT_NOALLOC_PARTIALS doubles, the first fold in the last RT_BLOCK.  Each device holds
// its own copy for the life of the process.
static __device__ __align__(256) double rt_noalloc_scratch[RT_NOALLOC_PARTIALS + RT_BLOCK];

namespace {

constexpr int ND = RT_NDIAG;

// Reduction of NV values per thread over the workgroup, in a fixed order: the xor butterfly
// in each wave, then the four waves in turn.  Value i is a sum, or the minimum where bit i of
// `min_mask` is set; thread i of the first NV writes it to out[i].
template <int NV> __device__ __forceinline__ void block_reduce_store(const double (&v)[NV], unsigned min_mask, double *out) {
  __shared__ double sh[RT_BLOCK / 64][NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const bool is_min = (min_mask >> i) & 1u;
    double x = v[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double y = __shfl_xor(x, o, 64);
      x = is_min ? fmin(x, y) : x + y;
    }
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64][i] = x;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    const int i = threadIdx.x;
    const bool is_min = (min_mask >> i) & 1u;
    double acc = sh[0][i];
    for (int w = 1; w < RT_BLOCK / 64; ++w) acc = is_min ? fmin(acc, sh[w][i]) : acc + sh[w][i];
    out[i] = acc;
  }
}

// Conservation totals.  Bound by the one read of the intensities.  Every total is linear in
// them, so a lane adds its own angles' terms V W I and V W I n over all its cells and the lanes
// meet once, at the end of at most RT_DIAG_BLOCKS workgroups; four cells per lane are in
// flight at a time, and the gas totals are a second, coalesced sweep.  With one reduction
// per cell and one of ten values per 16 cells it took 198 us at 96^3 x 80 in FP32, now 80
// (4.2 TB/s; the read alone is 61 us at the rate of a copy).
#define RT_DIAG_BLOCKS 2048
#define RT_DIAG_CELLS 4
template <typename T, int LPC, int APL>
__global__ __launch_bounds__(RT_BLOCK) void k_diag(int64_t N, int K, const double *dirs, const double *W,
                                                   double c_red, double c_light, const T *I, const double *vol,
                                                   const double *etot, const double *mom, double *partial) {
  constexpr int CPB = RT_BLOCK / LPC, R = RT_DIAG_CELLS;
  const int l = threadIdx.x % LPC;
  rt_lane_angles<double, LPC, APL> ang;
  ang.load(dirs, W, K, l);
  double E = 0, Fx = 0, Fy = 0, Fz = 0, bad = 0;
  T mn = (T)INFINITY;
  for (int64_t c0 = (int64_t)blockIdx.x * (CPB * R); c0 < N; c0 += (int64_t)gridDim.x * (CPB * R)) {
    T x[R][APL];
    double V[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // past the last cell: that cell again
      const int64_t c = c0 + r * CPB + threadIdx.x / LPC, cell = c < N ? c : N - 1;
      V[r] = vol[cell];
#pragma unroll
      for (int q = 0; q < APL; ++q) x[r][q] = I[cell * (int64_t)K + ang.k[q]];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // what is read again (past the last cell, and angle 0 in a slot past K, the last of a lane)
      // is left out, not multiplied by zero: an infinite one would make the totals NaN
      if (c0 + r * CPB + threadIdx.x / LPC >= N) continue;
      double t = 0, tx = 0, ty = 0, tz = 0;
#pragma unroll
      for (int q = 0; q < APL; ++q) {
        const double wx = q + 1 < APL || ang.ok[q] ? ang.w[q] * (double)x[r][q] : 0.0;
        t += wx;
        tx += wx * ang.dx[q];
        ty += wx * ang.dy[q];
        tz += wx * ang.dz[q];
        mn = fmin(mn, x[r][q]);
      }
      E += V[r] * t;
      Fx += V[r] * tx;
      Fy += V[r] * ty;
      Fz += V[r] * tz;
      // a non-finite intensity leaves t non-finite, whatever its weight
      if (!isfinite(t))
        for (int q = 0; q < APL; ++q) bad += ang.ok[q] && !isfinite(x[r][q]);
    }
  }
  double eg = 0, mx = 0, my = 0, mz = 0;
  for (int64_t c = (int64_t)blockIdx.x * RT_BLOCK + threadIdx.x; c < N; c += (int64_t)gridDim.x * RT_BLOCK) {
    const double V = vol[c], e = etot[c], m0 = mom[3 * c], m1 = mom[3 * c + 1], m2 = mom[3 * c + 2];
    eg += V * e;
    mx += V * m0;
    my += V * m1;
    mz += V * m2;
    bad += !isfinite(e) + !isfinite(m0) + !isfinite(m1) + !isfinite(m2);
  }
  const double fp = 4.0 * RT_PI, f = fp / c_red;
  const double v[ND] = {eg, (c_light / c_red) * fp * E, mx, my, mz, f * Fx, f * Fy, f * Fz, (double)mn, bad};
  block_reduce_store<ND>(v, 1u << 8, partial + (int64_t)blockIdx.x * ND);
}

// Fold rows [blockIdx.x * chunk, +chunk) of an [nrows][NV] table into row blockIdx.x of
// `out`: thread t folds rows t, t + 256, ... of the chunk in order, then the workgroup
// reduction.  The chunking depends on nrows only, so results are deterministic.
template <int NV>
__global__ __launch_bounds__(RT_BLOCK) void k_fold(const double *partial, int64_t nrows, unsigned min_mask,
                                                   int64_t chunk, double *out) {
  const int64_t r0 = (int64_t)blockIdx.x * chunk;
  const int64_t r1 = r0 + chunk < nrows ? r0 + chunk : nrows;
  double acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = (min_mask >> i) & 1u ? INFINITY : 0.0;
  for (int64_t b = r0 + threadIdx.x; b < r1; b += RT_BLOCK)
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const double x = partial[b * NV + i];
      acc[i] = (min_mask >> i) & 1u ? fmin(acc[i], x) : acc[i] + x;
    }
  block_reduce_store<NV>(acc, min_mask, out + (int64_t)blockIdx.x * NV);
}

// One workgroup folds up to RT_FOLD_ROWS rows; more go through up to RT_BLOCK workgroups over
// contiguous chunks into `mid` ([RT_BLOCK][NV]) first (13,824 rows of one value: 15 us in one
// fold, 4.6 + 4.6 in two; 2048 rows of ten: 11 us in one).
#define RT_FOLD_ROWS (8 * RT_BLOCK)
template <int NV>
hipError_t reduce_partials(const double *partial, int64_t nrows, unsigned min_mask, double *mid, double *out,
                           hipStream_t s) {
  if (nrows > RT_FOLD_ROWS) {
    const int64_t chunk = (nrows + RT_BLOCK - 1) / RT_BLOCK;
    const int64_t g = (nrows + chunk - 1) / chunk;
    hipLaunchKernelGGL(k_fold<NV>, dim3((unsigned)g), dim3(RT_BLOCK), 0, s, partial, nrows, min_mask, chunk, mid);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    partial = mid;
    nrows = g;
  }
  hipLaunchKernelGGL(k_fold<NV>, dim3(1), dim3(RT_BLOCK), 0, s, partial, nrows, min_mask, nrows, out);
  return hipGetLastError();
}

// Loss: each (face, angle) belongs to its upwind cell (A n_out . n_k > 0), which adds
// u_f sigma 4 pi c W_k (A n_out . n_k) I to its partial loss and that coefficient to
// its seed; sigma = -1 on a face's second cell since n_out = -n_f there.
// A loss weights few faces (a plane's: 1% of the cells at 96^3), so what bounds it is finding
// them.  A workgroup of CELLS consecutive cells first reads the weights of its
// half-faces, one thread each (they are one contiguous range), marks the cells that have one
// and ends there when none has.  The lanes of a marked cell then read one face each, with its
// record, and take the weighted ones in face order.  With every lane of every cell reading
// all its faces it took 400 us at 96^3 x 80 with the caches cold, now 80 (its 55 MB of
// half-face ids and as much of weights: 24 us at the rate of a copy, 35 us without weights).
// A marked cell is a word in LDS that every finder sets: as bits of one word, set by atomics, their
// queue doubled the time where many faces have a weight (all of them, 12^3 x 24: 29 us with atomics,
// 13 without; 96^3 x 80 905 and 742).  CELLS is 64, or on meshes that leave fewer than
// RT_LOSS_BLOCKS workgroups of that size as many as the lanes take at once (16 or 32), so that these
// have no rounds over the marked cells (of 1024 workgroups the rounds are still the shorter:
// 33^3 x 37 21 us against 23, a tenth of the faces weighted).
#define RT_LOSS_CELLS 64
#define RT_LOSS_BLOCKS 256
template <typename T, int LPC, int APL, int CELLS>
__global__ __launch_bounds__(RT_BLOCK) void k_loss(int64_t N, int K, const int32_t *row_ptr, const int32_t *hf_face,
                                                   const double4 *hf_an, const double *dirs, const double *W,
                                                   double c_light, const T *I, const double *face_weight,
                                                   T *seed, double *partial, int64_t nblk) {
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  constexpr int CPB = RT_BLOCK / LPC;
  static_assert(CELLS <= 64, "one bit per cell");
  __shared__ int s_rows[CELLS + 1];
  __shared__ int s_mark[64];  // whether a cell has a weighted face
  const int64_t w0 = lb * CELLS;
  const int nc = (int)(N - w0 < CELLS ? N - w0 : CELLS);
  if (threadIdx.x <= nc) s_rows[threadIdx.x] = row_ptr[w0 + threadIdx.x];
  if (threadIdx.x < 64) s_mark[threadIdx.x] = 0;
  __syncthreads();
  {
    constexpr int B = 4;  // ids, then weights, fetched together
    rt_scan_half_faces<RT_BLOCK, B>(s_rows[0], s_rows[nc], threadIdx.x, [&](const uint32_t (&h)[B]) {
      int32_t fc[B];
      double u[B];
#pragma unroll
      for (int b = 0; b < B; ++b) fc[b] = hf_face[h[b]];
#pragma unroll
      for (int b = 0; b < B; ++b) u[b] = face_weight[fc[b] >= 0 ? fc[b] : -(int64_t)fc[b] - 1];
#pragma unroll
      for (int b = 0; b < B; ++b)
        if (u[b] != 0.0) {
          int c = 0, past = nc;  // rows[c] <= h[b] < rows[past]
          while (past - c > 1) {
            const int mid = (c + past) / 2;
            if ((uint32_t)s_rows[mid] <= h[b]) c = mid;
            else past = mid;
          }
          s_mark[c] = 1;  // every writer writes this
        }
    });
  }
  __syncthreads();
  const unsigned long long mark = __ballot(s_mark[threadIdx.x % 64] != 0);
  if (mark == 0) {
    if (threadIdx.x == 0) partial[lb] = 0.0;
    return;
  }
  const int l = threadIdx.x % LPC;
  rt_lane_angles<double, LPC, APL> ang;
  ang.load(dirs, W, K, l);
  const double fpc = 4.0 * RT_PI * c_light;
  double part = 0.0;
  const int marked = __popcll(mark);
  for (int i = threadIdx.x / LPC; i < marked; i += CPB) {
    unsigned long long m = mark;  // the i-th marked cell
    for (int k = 0; k < i; ++k) m &= m - 1;
    const int c = __ffsll(m) - 1;
    const int64_t cell = w0 + c, row = cell * (int64_t)K;
    double sd[APL], Iv[APL];
    for (int q = 0; q < APL; ++q) sd[q] = Iv[q] = 0.0;
    for (int q = 0; q < APL; ++q) Iv[q] = ang.ok[q] ? (double)I[row + ang.k[q]] : 0.0;
    const uint32_t h1 = s_rows[c + 1];  // unsigned, as in rt_scan_half_faces
    for (uint32_t hb = s_rows[c]; hb < h1; hb += LPC) {
      double u = 0.0;
      double4 an = {0.0, 0.0, 0.0, 0.0};
      if (hb + l < h1) {
        const int32_t fc = hf_face[hb + l];
        u = fc >= 0 ? face_weight[fc] : -face_weight[-(int64_t)fc - 1];
        if (u != 0.0) an = hf_an[hb + l];
      }
      // the cell's weighted faces among these, in order
      unsigned todo = (unsigned)(__ballot(u != 0.0) >> (threadIdx.x % 64 - l)) & ((1u << LPC) - 1u);
      while (todo) {
        const int b = __ffs(todo) - 1;
        todo &= todo - 1;
        const double sg = __shfl(u, b, LPC);
        const double rx = __shfl(an.x, b, LPC), ry = __shfl(an.y, b, LPC), rz = __shfl(an.z, b, LPC);
        for (int q = 0; q < APL; ++q) {
          const double m = rx * ang.dx[q] + ry * ang.dy[q] + rz * ang.dz[q];
          if (m > 0.0) {
            const double coef = sg * fpc * ang.w[q] * m;
            part += coef * Iv[q];
            sd[q] += coef;
          }
        }
      }
    }
    if (seed)
      for (int q = 0; q < APL; ++q)
        if (ang.ok[q] && sd[q] != 0.0) seed[row + ang.k[q]] = (T)((double)seed[row + ang.k[q]] + sd[q]);
  }
  const double v[1] = {part};
  block_reduce_store<1>(v, 0u, partial + lb);
}

// Angle moments of every cell (section 2.1): with intensities in energy-density units,
// E_r = 4 pi sum W I, F_r = 4 pi c sum W n I, P_r = 4 pi sum W n n I.  The LPC lanes of a
// cell sum their angles; the group sums (DPP) leave the totals in every lane, and lane c
// writes component c (two rounds when LPC = 8), so a cell's 80 bytes go out together.
// Each lane group takes RT_MOM_CELLS cells (CPB apart, so every round of a workgroup reads
// consecutive rows): the lane's directions and weights are loaded once for all of them,
// and all their intensity loads are issued before any is used.
#define RT_MOM_CELLS 4
template <typename T, int LPC, int APL>
__global__ __launch_bounds__(RT_BLOCK) void k_moments(int64_t N, int K, const double *dirs, const double *W,
                                                      double c_light, const T *I, double *out, int64_t nblk) {
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  constexpr int CPB = RT_BLOCK / LPC;
  constexpr int R = RT_MOM_CELLS;
  const int64_t c0 = lb * CPB * R + threadIdx.x / LPC;
  if (c0 >= N) return;  // whole lane groups
  const int l = threadIdx.x % LPC;
  rt_lane_angles<double, LPC, APL> ang;
  ang.load(dirs, W, K, l);
  T x[R][APL];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t cell = c0 + (int64_t)CPB * r;
#pragma unroll
    for (int q = 0; q < APL; ++q) x[r][q] = cell < N && ang.ok[q] ? I[cell * (int64_t)K + ang.k[q]] : T(0);
  }
  const double fourpi = 4.0 * RT_PI;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t cell = c0 + (int64_t)CPB * r;
    if (cell >= N) break;  // the same for all lanes of the group
    double m[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < APL; ++q) {
      const double wI = ang.w[q] * (double)x[r][q];
      const double nx = ang.dx[q], ny = ang.dy[q], nz = ang.dz[q];
      m[0] += wI;
      m[1] += wI * nx;
      m[2] += wI * ny;
      m[3] += wI * nz;
      m[4] += wI * nx * nx;
      m[5] += wI * ny * ny;
      m[6] += wI * nz * nz;
      m[7] += wI * nx * ny;
      m[8] += wI * nx * nz;
      m[9] += wI * ny * nz;
    }
    double v[10];
#pragma unroll
    for (int c = 0; c < 10; ++c) v[c] = rt_group_sum<LPC>(m[c]) * (c >= 1 && c <= 3 ? fourpi * c_light : fourpi);
#pragma unroll
    for (int b = 0; b < 10; b += LPC) {
      // lane l writes component b + l
      double o = v[b];
#pragma unroll
      for (int c = b + 1; c < b + LPC && c < 10; ++c)
        if (l == c - b) o = v[c];
      if (b + l < 10) out[10 * cell + b + l] = o;
    }
  }
}

// Angle moments with 16-byte row chunks: 4 lanes per cell, lane l reading chunks
// l, l + 4, ... (CPL of them) of its cell's row, so a wave's loads cover 16 rows 64 bytes
// at a time (the cheapest access pattern for these rows).  Each angle's (W, n) comes from
// LDS, where every lane at one position reads the same entry; the 4 lanes' moments are
// summed by DPP quad permutations.  Needs rows of whole 16-byte chunks, 16-byte aligned.
template <typename T, int CPL>
__global__ __launch_bounds__(RT_BLOCK) void k_moments16(int64_t N, int K, const double *dirs, const double *W,
                                                        double c_light, const T *I, double *out, int64_t nblk) {
  constexpr int EPC = 16 / sizeof(T);  // elements per chunk
  __shared__ double4 s_dw[RT_K_MAX];   // (W, n_x, n_y, n_z) per angle
  for (int k = threadIdx.x; k < K; k += RT_BLOCK) s_dw[k] = double4{W[k], dirs[3 * k], dirs[3 * k + 1], dirs[3 * k + 2]};
  __syncthreads();
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  const int64_t cell = lb * (RT_BLOCK / 4) + threadIdx.x / 4;
  if (cell >= N) return;  // whole lane groups
  const int l = threadIdx.x % 4;
  const int nch = K / EPC;  // chunks per row
  // the lane's chunks, all loads issued before any is used
  const char *row = (const char *)(I + cell * (int64_t)K);
  T x[CPL][EPC];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = l + 4 * c;
    if (ch < nch) {
      if constexpr (EPC == 4) {
        const float4 v = *(const float4 *)(row + 16 * ch);
        x[c][0] = v.x; x[c][1] = v.y; x[c][2] = v.z; x[c][3] = v.w;
      } else {
        const double2 v = *(const double2 *)(row + 16 * ch);
        x[c][0] = v.x; x[c][1] = v.y;
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPC; ++e) x[c][e] = T(0);
    }
  }
  double m[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = l + 4 * c;
    if (ch >= nch) continue;
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
      const double4 d = s_dw[EPC * ch + e];
      const double t = d.x * (double)x[c][e];
      const double tx = t * d.y, ty = t * d.z, tz = t * d.w;
      m[0] += t;
      m[1] += tx;
      m[2] += ty;
      m[3] += tz;
      m[4] += tx * d.y;
      m[5] += ty * d.z;
      m[6] += tz * d.w;
      m[7] += tx * d.z;
      m[8] += tx * d.w;
      m[9] += ty * d.w;
    }
  }
  const double fourpi = 4.0 * RT_PI;
  double v[10];
#pragma unroll
  for (int c = 0; c < 10; ++c) v[c] = rt_group_sum<4>(m[c]) * (c >= 1 && c <= 3 ? fourpi * c_light : fourpi);
  // lane l writes components l, l + 4 and (l < 2) l + 8
#pragma unroll
  for (int b = 0; b < 10; b += 4) {
    double o = v[b];
#pragma unroll
    for (int c = b + 1; c < b + 4 && c < 10; ++c)
      if (l == c - b) o = v[c];
    if (b + l < 10) out[10 * cell + b + l] = o;
  }
}

// The same moments for an antipodal set (pair kind 1: angle k's antipode at k + K/2; 2: at
// k + 1 for even k).  Each pair (k, k'), n_k' = -n_k and W_k' = W_k, adds W (I_k + I_k') to
// the energy and the pressure and W (I_k - I_k') n_k to the flux: one direction read and
// half the multiply-adds per angle.  Lane l of a cell's 4 takes chunks l, l + 4, ... of the
// first half of the row with their antipodes' chunks (kind 1), or whole chunks holding
// EPC / 2 pairs (kind 2).  Needs what the chunked kernel needs, and K / 2 a multiple of
// EPC for kind 1.
template <typename T, int CPL, int PAIRED>
__global__ __launch_bounds__(RT_BLOCK) void k_moments16p(int64_t N, int K, const double *dirs, const double *W,
                                                         double c_light, const T *I, double *out, int64_t nblk) {
  constexpr int EPC = 16 / sizeof(T);          // elements per chunk
  constexpr int PPC = PAIRED == 1 ? EPC : EPC / 2;  // pairs per chunk (kind 1: with its antipode chunk)
  __shared__ double4 s_dw[RT_K_MAX];           // (W, n_x, n_y, n_z) per angle
  for (int k = threadIdx.x; k < K; k += RT_BLOCK) s_dw[k] = double4{W[k], dirs[3 * k], dirs[3 * k + 1], dirs[3 * k + 2]};
  __syncthreads();
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  const int64_t cell = lb * (RT_BLOCK / 4) + threadIdx.x / 4;
  if (cell >= N) return;  // whole lane groups
  const int l = threadIdx.x % 4;
  const int nc = PAIRED == 1 ? K / (2 * EPC) : K / EPC;  // chunks the lanes walk
  const char *row = (const char *)(I + cell * (int64_t)K);
  T x[CPL][EPC], y[CPL][EPC];
  auto load = [&](T(&v)[EPC], int ch) {
    if constexpr (EPC == 4) {
      const float4 a = *(const float4 *)(row + 16 * ch);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    } else {
      const double2 a = *(const double2 *)(row + 16 * ch);
      v[0] = a.x; v[1] = a.y;
    }
  };
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = l + 4 * c;
    if (ch < nc) {
      load(x[c], ch);
      if (PAIRED == 1) load(y[c], ch + nc);
    }
  }
  double m[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int ch = l + 4 * c;
    if (ch >= nc) continue;
#pragma unroll
    for (int e = 0; e < PPC; ++e) {
      const double a = (double)(PAIRED == 1 ? x[c][e] : x[c][2 * e]);
      const double b = (double)(PAIRED == 1 ? y[c][e] : x[c][2 * e + 1]);
      const double4 d = s_dw[EPC * ch + (PAIRED == 1 ? e : 2 * e)];
      const double t = d.x * (a + b), u = d.x * (a - b);
      const double tx = t * d.y, ty = t * d.z, tz = t * d.w;
      m[0] += t;
      m[1] += u * d.y;
      m[2] += u * d.z;
      m[3] += u * d.w;
      m[4] += tx * d.y;
      m[5] += ty * d.z;
      m[6] += tz * d.w;
      m[7] += tx * d.z;
      m[8] += tx * d.w;
      m[9] += ty * d.w;
    }
  }
  const double fourpi = 4.0 * RT_PI;
  double v[10];
#pragma unroll
  for (int c = 0; c < 10; ++c) v[c] = rt_group_sum<4>(m[c]) * (c >= 1 && c <= 3 ? fourpi * c_light : fourpi);
  // lane l writes components l, l + 4 and (l < 2) l + 8
#pragma unroll
  for (int b = 0; b < 10; b += 4) {
    double o = v[b];
#pragma unroll
    for (int c = b + 1; c < b + 4 && c < 10; ++c)
      if (l == c - b) o = v[c];
    if (b + l < 10) out[10 * cell + b + l] = o;
  }
}

template <typename T, int CPL, int PAIRED>
hipError_t launch_moments16p(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light,
                             const void *I, double *out, hipStream_t s) {
  const int64_t nblk = (m->N + RT_BLOCK / 4 - 1) / (RT_BLOCK / 4);
  hipLaunchKernelGGL((k_moments16p<T, CPL, PAIRED>), dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK), 0, s, m->N,
                     K, dirs, W, c_light, (const T *)I, out, nblk);
  return hipGetLastError();
}

template <typename T, int PAIRED>
hipError_t dispatch_moments16p(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light,
                               const void *I, double *out, hipStream_t s) {
  constexpr int EPC = 16 / sizeof(T);
  const int nc = PAIRED == 1 ? K / (2 * EPC) : K / EPC;
  switch ((nc + 3) / 4) {  // chunks (kind 1: chunk pairs) per lane
    case 1: return launch_moments16p<T, 1, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 2: return launch_moments16p<T, 2, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 3: return launch_moments16p<T, 3, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 4: return launch_moments16p<T, 4, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 5: return launch_moments16p<T, 5, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 6: return launch_moments16p<T, 6, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 7: return launch_moments16p<T, 7, PAIRED>(m, K, dirs, W, c_light, I, out, s);
    case 8: return launch_moments16p<T, 8, PAIRED>(m, K, dirs, W, c_light, I, out, s);
  }
  return hipErrorInvalidValue;
}

template <typename T, int CPL>
hipError_t launch_moments16(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light,
                            const void *I, double *out, hipStream_t s) {
  const int64_t nblk = (m->N + RT_BLOCK / 4 - 1) / (RT_BLOCK / 4);
  hipLaunchKernelGGL((k_moments16<T, CPL>), dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK), 0, s, m->N, K, dirs,
                     W, c_light, (const T *)I, out, nblk);
  return hipGetLastError();
}

template <typename T, int LPC, int APL>
hipError_t launch_moments(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light, const void *I,
                          double *out, hipStream_t s) {
  const int64_t cpc = (int64_t)(RT_BLOCK / LPC) * RT_MOM_CELLS;  // cells per workgroup
  const int64_t nblk = (m->N + cpc - 1) / cpc;
  hipLaunchKernelGGL((k_moments<T, LPC, APL>), dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK), 0, s, m->N, K,
                     dirs, W, c_light, (const T *)I, out, nblk);
  return hipGetLastError();
}

template <typename T, int LPC, int APL>
hipError_t launch_diag(const rt_mesh *m, int K, const double *dirs, const double *W, double c_red, double c_light,
                       const void *I, const double *vol, const double *etot, const double *mom, double *out,
                       hipStream_t s) {
  constexpr int64_t cpb = RT_BLOCK / LPC * RT_DIAG_CELLS;
  const int64_t all = (m->N + cpb - 1) / cpb, g = all < RT_DIAG_BLOCKS ? all : RT_DIAG_BLOCKS;
  if (g > m->n_red_blocks) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_diag<T, LPC, APL>), dim3((unsigned)g), dim3(RT_BLOCK), 0, s, m->N, K, dirs, W, c_red, c_light,
                     (const T *)I, vol, etot, mom, m->red);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return reduce_partials<ND>(m->red, g, 1u << 8, m->red_mid, out, s);
}

// The loss into `partial` (one row per workgroup, at most `cap` rows), folded through `mid`
// ([RT_BLOCK] rows) into *loss.
template <typename T, int LPC, int APL>
hipError_t launch_loss(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light, const void *I,
                       const double *fw, double *loss, void *seed, double *partial, double *mid, int64_t cap,
                       hipStream_t s) {
  const int64_t wide = (m->N + RT_LOSS_CELLS - 1) / RT_LOSS_CELLS, cpb = RT_BLOCK / LPC;
  const int64_t nblk = wide < RT_LOSS_BLOCKS ? (m->N + cpb - 1) / cpb : wide;
  if (nblk > cap) return hipErrorInvalidValue;
  auto kernel = wide < RT_LOSS_BLOCKS ? k_loss<T, LPC, APL, RT_BLOCK / LPC> : k_loss<T, LPC, APL, RT_LOSS_CELLS>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK), 0, s, m->N, K, m->row_ptr, m->hf_face,
                     m->hf_an64, dirs, W, c_light, (const T *)I, fw, (T *)seed, partial, nblk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return reduce_partials<1>(partial, nblk, 0u, mid, loss, s);
}

#define RT_DISPATCH(FN, T, ...)                                   \
  do {                                                            \
    if (K % 16 == 0 || K > 64) {                                  \
      switch ((K + 15) / 16) {                                    \
        case 1: return FN<T, 16, 1>(__VA_ARGS__);                 \
        case 2: return FN<T, 16, 2>(__VA_ARGS__);                 \
        case 3: return FN<T, 16, 3>(__VA_ARGS__);                 \
        case 4: return FN<T, 16, 4>(__VA_ARGS__);                 \
        case 5: return FN<T, 16, 5>(__VA_ARGS__);                 \
        case 6: return FN<T, 16, 6>(__VA_ARGS__);                 \
        case 7: return FN<T, 16, 7>(__VA_ARGS__);                 \
        case 8: return FN<T, 16, 8>(__VA_ARGS__);                 \
      }                                                           \
    } else {                                                      \
      switch ((K + 7) / 8) {                                      \
        case 1: return FN<T, 8, 1>(__VA_ARGS__);                  \
        case 2: return FN<T, 8, 2>(__VA_ARGS__);                  \
        case 3: return FN<T, 8, 3>(__VA_ARGS__);                  \
        case 4: return FN<T, 8, 4>(__VA_ARGS__);                  \
        case 5: return FN<T, 8, 5>(__VA_ARGS__);                  \
        case 6: return FN<T, 8, 6>(__VA_ARGS__);                  \
        case 7: return FN<T, 8, 7>(__VA_ARGS__);                  \
        case 8: return FN<T, 8, 8>(__VA_ARGS__);                  \
      }                                                           \
    }                                                             \
    return hipErrorInvalidValue;                                  \
  } while (0)

template <typename T>
hipError_t diag_t(const rt_mesh *m, int K, const double *dirs, const double *W, double c_red, double c_light,
                  const void *I, const double *vol, const double *etot, const double *mom, double *out,
                  hipStream_t s) {
  RT_DISPATCH(launch_diag, T, m, K, dirs, W, c_red, c_light, I, vol, etot, mom, out, s);
}

template <typename T>
hipError_t moments_t(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light, const void *I,
                     double *out, int paired, hipStream_t s) {
  // rows of whole 16-byte chunks starting 16-byte aligned: the chunked kernel, 4 lanes per cell
  constexpr int EPC = 16 / sizeof(T);
  const bool chunked = K % EPC == 0 && ((uintptr_t)I & 15u) == 0;
  // antipodal sets whose pairs sit whole in the chunks (kind 2) or fill whole chunks in each
  // half of the row (kind 1): the paired form
  if (chunked && paired == 2 && EPC % 2 == 0 && K <= 32 * EPC)
    return dispatch_moments16p<T, 2>(m, K, dirs, W, c_light, I, out, s);
  if (chunked && paired == 1 && K % (2 * EPC) == 0 && K <= 64 * EPC)
    return dispatch_moments16p<T, 1>(m, K, dirs, W, c_light, I, out, s);
  if (chunked) {
    switch ((K / EPC + 3) / 4) {  // chunks per lane
      case 1: return launch_moments16<T, 1>(m, K, dirs, W, c_light, I, out, s);
      case 2: return launch_moments16<T, 2>(m, K, dirs, W, c_light, I, out, s);
      case 3: return launch_moments16<T, 3>(m, K, dirs, W, c_light, I, out, s);
      case 4: return launch_moments16<T, 4>(m, K, dirs, W, c_light, I, out, s);
      case 5: return launch_moments16<T, 5>(m, K, dirs, W, c_light, I, out, s);
      case 6: return launch_moments16<T, 6>(m, K, dirs, W, c_light, I, out, s);
      case 7: return launch_moments16<T, 7>(m, K, dirs, W, c_light, I, out, s);
      case 8: return launch_moments16<T, 8>(m, K, dirs, W, c_light, I, out, s);
      case 9: return launch_moments16<T, 9>(m, K, dirs, W, c_light, I, out, s);
      case 10: return launch_moments16<T, 10>(m, K, dirs, W, c_light, I, out, s);
      case 11: return launch_moments16<T, 11>(m, K, dirs, W, c_light, I, out, s);
      case 12: return launch_moments16<T, 12>(m, K, dirs, W, c_light, I, out, s);
      case 13: return launch_moments16<T, 13>(m, K, dirs, W, c_light, I, out, s);
      case 14: return launch_moments16<T, 14>(m, K, dirs, W, c_light, I, out, s);
      case 15: return launch_moments16<T, 15>(m, K, dirs, W, c_light, I, out, s);
      case 16: return launch_moments16<T, 16>(m, K, dirs, W, c_light, I, out, s);
    }
  }
  RT_DISPATCH(launch_moments, T, m, K, dirs, W, c_light, I, out, s);
}

template <typename T>
hipError_t loss_t(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light, const void *I,
                  const double *fw, double *loss, void *seed, double *partial, double *mid, int64_t cap,
                  hipStream_t s) {
  RT_DISPATCH(launch_loss, T, m, K, dirs, W, c_light, I, fw, loss, seed, partial, mid, cap, s);
}

// Device address of the scratch on each device, looked up once per device with that
// device current (host code must never use the array's own name as a device pointer).
std::mutex g_scratch_mu;
double *g_scratch_ptr[RT_MAX_DEVICES] = {};

hipError_t noalloc_scratch(int device, double **out) {
  if (device < 0 || device >= RT_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(rt_noalloc_scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = (double *)p;
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

}  // namespace

hipError_t rt_launch_diagnostics(const rt_mesh *m, int K, const double *dirs, const double *W, double c_red,
                                 double c_light, const void *I, const double *vol, const double *etot,
                                 const double *mom, double *out_dev, int dtype, hipStream_t s) {
  return dtype == RT_F32 ? diag_t<float>(m, K, dirs, W, c_red, c_light, I, vol, etot, mom, out_dev, s)
                         : diag_t<double>(m, K, dirs, W, c_red, c_light, I, vol, etot, mom, out_dev, s);
}

hipError_t rt_launch_flux_loss(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light,
                               const void *I, const double *face_weight, double *loss, void *seed, int dtype,
                               hipStream_t s) {
  return dtype == RT_F32
             ? loss_t<float>(m, K, dirs, W, c_light, I, face_weight, loss, seed, m->red, m->red_mid, m->n_red_blocks, s)
             : loss_t<double>(m, K, dirs, W, c_light, I, face_weight, loss, seed, m->red, m->red_mid, m->n_red_blocks,
                              s);
}

hipError_t rt_launch_flux_loss_noalloc(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light,
                                       const void *I, const double *face_weight, double *loss, void *seed, int dtype,
                                       hipStream_t s) {
  double *scratch = nullptr;
  const hipError_t e = noalloc_scratch(m->device, &scratch);
  if (e != hipSuccess) return e;
  double *mid = scratch + RT_NOALLOC_PARTIALS;
  return dtype == RT_F32
             ? loss_t<float>(m, K, dirs, W, c_light, I, face_weight, loss, seed, scratch, mid, RT_NOALLOC_PARTIALS, s)
             : loss_t<double>(m, K, dirs, W, c_light, I, face_weight, loss, seed, scratch, mid, RT_NOALLOC_PARTIALS,
                              s);
}

hipError_t rt_launch_moments(const rt_mesh *m, int K, const double *dirs, const double *W, double c_light,
                             const void *I, double *out, int dtype, int paired, hipStream_t s) {
  return dtype == RT_F32 ? moments_t<float>(m, K, dirs, W, c_light, I, out, paired, s)
                         : moments_t<double>(m, K, dirs, W, c_light, I, out, paired, s);
}
