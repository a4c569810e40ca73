// The radiation step kernel: transport (section 2.2) and the implicit source
// update (section 2.3) of one cell per group of LPC lanes, each lane holding APL
// angles.  One pass reads the cell's intensity row, gathers the neighbour rows of
// its faces through the half-face index (no atomics), updates the charges, runs the
// source on the transported row while it is in registers, and writes the row once.
#include "rt_face_speed.h"
#include "rt_source_vjp.h"
#include "rt_step_common.h"

namespace {

// Faces gathered per batch: all their neighbour-row loads are issued before any is
// used, so one memory round trip serves U faces.  At 128^3 x 80: two faces measured ~2%
// faster than four in FP32.  The FP64 form with antipodes side by side ran 5% faster with
// three (1.91 against 2.00 ms) at two waves per SIMD; since its source holds fewer values
// (three waves) two are faster again: 1.85 ms, against 2.45 ms with three.
// PLM stage 2 holds four values per gathered state, and of a pair gathers one: one face at a
// time at 8 to 12 angles per lane (two cost a wave per SIMD: 64^3 x 80 step, FP32 0.69 against
// 0.70 ms, FP64 1.34 against 1.72), two at 4 and 6 (one: 48^3 x 24, FP32 0.138 against 0.142),
// four at 2 (two: 40^3 x 8, FP32 0.062 against 0.064 ms); without pairs two (one: 48^3 x 37,
// FP32 0.196 against 0.202 ms, FP64 0.37 against 0.48).  Grids of a few rounds wait more than they
// gather, and take two faces in FP32 (rt_states).
template <typename T, int APL, int PAIRED, int STATES> struct rt_batch {
  static constexpr int U = 2;
  static constexpr int PLM = !PAIRED || STATES == 2 || (STATES == 1 && sizeof(T) == 4 && APL > 2) ? 2
                             : APL > 6 ? 1 : APL > 2 ? 2 : 4;
};

// Which states of an antipodal pair PLM stage 2 gathers from a neighbour: 0 the one that enters,
// and behind it the other where both do; 1 the same, the other fetched along with the first;
// 2 both.  The fewest fetches and registers (0) are the fastest on large grids; on small ones the
// wait for a second fetch behind the first, or for one face after the other, is longer than the
// fetches take, the more so the more pairs enter whole.  Two PLM steps in FP32, faces at 1e-3 / 1e-2
// of the light speed, speed relative to the kernel that gathered both states of every pair, two
// faces at a time, before they were stored in 16-byte parts:
//   K = 80  12^3: (0) .97 / .91 (1) 1.00 / .98 (2) 1.00 / 1.00   32^3: 1.01 / .95, 1.07 / 1.05, 1.02 / 1.02
//           48^3: 1.09 / 1.04, 1.08 / 1.05, 1.03 / 1.03          64^3: 1.07 / 1.03, 1.06 / 1.04, 1.01 / 1.01
//   K = 48  12^3: (0) 1.00 / .96 (1) .99 / .98 (2) 1.03 / 1.04   32^3: 1.08 / 1.07, 1.03 / 1.02, 1.02 / 1.02
//   K = 24  12^3: (0) 1.00 / .96 (1) .99 / .98 (2) 1.03 / 1.03   64^3: 1.02 / .98, 1.01 / 1.00, 1.00 / 1.00
// With four lanes per cell a wave holds twice the faces, and (0) nearly always fetches twice.
// FP64 K = 80, antipodes side by side, 12^3: (0) 1.04 / .96 (1) 1.04 / .99, 20^3: 1.03 / .98, 1.02 / 1.00,
// 24^3: 1.10 / 1.06, 1.06 / 1.05; K/2 apart 12^3: 1.32 / 1.24, 1.27 / 1.21; (2) spills.
template <typename T> constexpr int rt_states(int lpc, int apl, int paired, int64_t nblk) {
  const int64_t per_cu = (nblk + 255) / 256;  // workgroups
  if (sizeof(T) == 8) return paired == 2 && (apl == 8 || apl == 10) && per_cu <= 1 ? 1 : 0;
  if (per_cu <= (apl >= 8 ? 1 : 2)) return 2;
  return lpc == 4 || (apl >= 8 && per_cu <= 10) ? 1 : 0;
}

// Rows (of whole lines: rows of part lines take longer past the caches, 48^3 x 37 FP32 0.22 ms
// against 0.20) that PLM stage 2 reads and writes past the caches, to leave those to the gathered
// states: on meshes of more than RT_PAST_CELLS cells, or with more than RT_PAST_BYTES of rows.  On
// smaller ones the next half step, which gathers each row about 16 times, finds more of them in the
// caches.  Two PLM steps, past the caches or through them: FP32 K = 80, 32^3 0.192 or 0.190 ms, 40^3
// 0.315 or 0.310, 48^3 0.538 or 0.549; K = 48, 32^3 0.139 or 0.137, 40^3 0.232 or 0.226, 48^3 0.369 or
// 0.379; FP64 K = 80, 32^3 0.317 or 0.310, 48^3 1.080 or 1.088, 64^3 2.486 or 2.502; K = 48, 40^3 0.379 or
// 0.385.  A kernel of its own: chosen inside one, the branch cost small grids 1 to 2%.
#define RT_PAST_CELLS 81920
#define RT_PAST_BYTES (22 << 20)
template <typename T, int LPC, int APL, bool FULL> constexpr bool rt_whole_lines() {
  return FULL && LPC * APL * sizeof(T) % 64 == 0;
}

// MODE 0: source only (in place); 1: upwind transport (+ source); 2: reconstructed
// transport of PLM stage 2 (+ source); 3: the transpose of upwind transport (the
// adjoint: input mu = lam*/V' per cell and angle, output lam_i = V_i mu_i - sum over the
// faces the cell is upwind of, g > 0, of g (mu_i - mu_j)); 4: the transpose of step
// n + 1 followed, in registers, by the reverse of the source of step n (output lam*/V'
// of step n, so consecutive launches chain the reverse of a run of steps without
// storing dL/dI in between); 5: the reverse of the source of step n alone (input dL/dI
// of its output, read from the cell's own row only).  Separate instantiations keep each
// one's registers to what its own code needs.
//
// The cells of a workgroup are consecutive, so their half-faces form one contiguous
// range; it is staged in LDS (dynamic size: the largest range of any workgroup,
// found at upload) and the face loops read their records from there.
// Occupancy target: the FP64 PLM stage 2 is held to two waves per SIMD (10 angles per lane: 248
// registers; unpaired forms of 6 to 8 angles and 12 paired spill 16 to 44), except the form of
// small grids, which have one (held to two it spills 30 values: 12^3 x 80, two steps 93 us, now 88).
// Everything else keeps the compiler's choice.
template <typename T, int MODE, int STATES> struct rt_step_waves {
  static constexpr int value = MODE == 2 && sizeof(T) == 8 && STATES == 0 ? 2 : 1;
};
template <typename T, int LPC, int APL, int MODE, bool FULL, int PAIRED, int STATES = 0, bool PAST = false>
__global__ __launch_bounds__(RT_BLOCK) __attribute__((amdgpu_waves_per_eu(rt_step_waves<T, MODE, STATES>::value))) void
k_step(rt_step_args a, int64_t nblk) {
  using V4 = typename rt_vec4<T>::type;
  // Runs of two pairs per lane (fewer, wider gathers): at 128^3 x 80 upwind, FP32 with
  // antipodes side by side 1.30 -> 1.18 ms and FP64 with antipodes K/2 on 2.35 -> 2.04 ms
  // (the other two forms within 3%).  PLM stage 2 gathers 16-byte parts of states and keeps
  // one pair per slot.
  using Ang = rt_step_angles<T, LPC, APL, FULL, PAIRED, MODE != 2>;
  constexpr bool FACES = MODE >= 1 && MODE <= 4;  // the modes that read face records
  constexpr bool TRANSPOSE = MODE == 3 || MODE == 4;
  constexpr int P = Ang::P;
  constexpr int U = rt_batch<T, APL, PAIRED, STATES>::U;
  constexpr int CPB = RT_BLOCK / LPC;
  extern __shared__ __align__(16) unsigned char rt_smem[];
  V4 *s_an = (V4 *)rt_smem;
  V4 *s_rel = s_an + a.hf_cap;
  int32_t *s_nbr = (int32_t *)(s_an + (MODE == 2 ? 3 : 1) * a.hf_cap);
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;  // whole padding workgroup
  const int64_t c0 = lb * CPB;
  const int g = threadIdx.x / LPC;
  const bool live = c0 + g < a.N;
  const int64_t cell = live ? c0 + a.wg_order[c0 + g] : c0;
  const int l = threadIdx.x % LPC;
  const int K = a.K;
  int H0 = 0;
  if (FACES) {
    const V4 *an = (const V4 *)a.hf_an;
    const V4 *rel = (const V4 *)a.hf_rel;
    const int64_t c1 = c0 + CPB < a.N ? c0 + CPB : a.N;
    H0 = a.row_ptr[c0];
    const int nH = a.row_ptr[c1] - H0;  // <= hf_cap by construction
    for (int i = threadIdx.x; i < nH; i += RT_BLOCK) {
      s_nbr[i] = a.hf_nbr[H0 + i];
      s_an[i] = an[H0 + i];
      if (MODE == 2) {
        s_rel[2 * i] = rel[2 * (H0 + i)];
        s_rel[2 * i + 1] = rel[2 * (H0 + i) + 1];
      }
    }
    __syncthreads();
  }
  if (!live) return;
  Ang ang;
  ang.load(a.dirs, a.W, K, l);

  const T *Iin = (const T *)a.I_in;
  const int64_t row = cell * (int64_t)K;
  // the lane's base pointers into row 0 (its first angle, and its lone pair's angle)
  const int k_single = Ang::SINGLE ? ang.k[P - 1] : ang.k[0];
  const T *Iin_lane = Iin + ang.k[0], *Iin_single = Iin + k_single;
  T Ic[APL];
  ang.template read_lane<PAST>(Iin_lane + row, Iin_single + row, Ic);

  double Vnew = 0.0, Vstart = 0.0;
  // the start-of-step volume: the reverse modes take it from the forward step's tape
  const double *tape = a.src_tape ? a.src_tape + RT_SRC_TAPE * cell : nullptr;
  const bool vol_from_tape = MODE >= 4 || (MODE == 3 && tape);
  if (MODE == 5) Vnew = rt_vol_next(tape[RT_TAPE_V], a.dt, a.D[cell]);
  if (FACES) {
    // ---- transport: charges V I minus the upwind charge through every face -------------
    const double Vn = vol_from_tape ? tape[RT_TAPE_V] : a.vol_in[cell];
    Vstart = Vn;
    const double dV = a.dt * a.D[cell];
    Vnew = rt_vol_next(Vn, a.dt, a.D[cell]);  // the end-of-step volume
    // the charge through the faces is accumulated apart from V I (the transpose adds V mu,
    // with V the start-of-step volume of the step it transposes: step n + 1 in mode 4)
    T acc[APL];
#pragma unroll
    for (int q = 0; q < APL; ++q) acc[q] = TRANSPOSE ? (T)(MODE == 4 ? Vnew : Vn) * Ic[q] : T(0);
    const T sc = (T)(a.dt * a.c_red), sd = (T)a.dt;
    const int h0 = a.row_ptr[cell], h1 = a.row_ptr[cell + 1];
    // a neighbour's row is one multiply-add away from the lane's base pointers
    const uint32_t row_bytes = (uint32_t)(K * sizeof(T));
    if (MODE == 1 || TRANSPOSE) {
      for (int h = h0; h < h1; h += U) {
        // batch metadata; slots past the cell's last face reuse face h0 with a zero record
        uint32_t j[U];
        V4 r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool v = h + u < h1;
          const int i = (v ? h + u : h0) - H0;
          j[u] = (uint32_t)s_nbr[i];
          r[u] = s_an[i];
          if (!v) r[u] = V4{T(0), T(0), T(0), T(0)};
        }
        T xn[U][APL];
#pragma unroll
        for (int u = 0; u < U; ++u)
          ang.read_lane(ang.lane_row(Iin_lane, j[u], row_bytes), ang.lane_row(Iin_single, j[u], row_bytes), xn[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // g = dt (cbar (A n_out).n_k - A (w~.n)_out): charge leaving per unit upwind intensity,
          // as three fused multiply-adds from -dt A (w~.n)_out.  Every operand of the face's
          // other side is negated exactly, so both sides get bitwise opposite g (conservation).
          const T ax = sc * r[u].x, ay = sc * r[u].y, az = sc * r[u].z, nb = -(sd * r[u].w);
          const T m2b = nb + nb;  // -2 dt A (w~.n)_out, exact
#pragma unroll
          for (int q = 0; q < P; ++q) {
            const T g = fma(az, ang.z[q], fma(ay, ang.y[q], fma(ax, ang.x[q], nb)));
            if constexpr (MODE == 1) {
              acc[q] -= g * (g > T(0) ? Ic[q] : xn[u][q]);
            } else {
              acc[q] -= g > T(0) ? g * (Ic[q] - xn[u][q]) : T(0);
            }
            if (PAIRED) {
              const T g2 = m2b - g;  // the antipodal angle: -(dot) - b
              if constexpr (MODE == 1) {
                acc[q + P] -= g2 * (g2 > T(0) ? Ic[q + P] : xn[u][q + P]);
              } else {
                acc[q + P] -= g2 > T(0) ? g2 * (Ic[q + P] - xn[u][q + P]) : T(0);
              }
            }
          }
        }
      }
    } else {
      // reconstructed face states of the half-step intensities (PLM stage 2).  Of an antipodal
      // pair only the direction that enters through a face needs the neighbour's state, so one
      // state per pair is gathered, chosen by the sign of the face speed, and the second where
      // both enter.  The kernel is bound by its gathers: their address units are busy 68% of the
      // time in either precision, and the L2 lines behind them add to it: 64^3 x 80 step with antipodes K/2
      // apart, FP64 1.64 -> 1.25 ms, side by side 1.38 -> 1.24; FP32 0.74 -> 0.69 and 0.71 -> 0.65.
      // Faces at a third of the light speed, where many pairs enter whole: FP32 0.323 -> 0.324 ms
      // (48^3 x 80), FP64 0.72 -> 0.61.  Small grids wait for each face in turn: rt_states.
      using S = rt_state<T>;
      const int KK = FULL ? LPC * APL : K;
      // a pair's states are K/2 apart in either order of the angles, so that lanes which pick the
      // same side read whole lines (two PLM steps with antipodes side by side, their states beside
      // each other: FP32 1.370 -> 1.344 ms, FP64 2.574 -> 2.504)
      const typename S::part *states = (const typename S::part *)a.states + (PAIRED ? l : ang.k[0]);
      const uint32_t state_row = (uint32_t)(K * sizeof(V4));
      auto of = [&](uint32_t c) { return (const typename S::part *)((const char *)states + (uint64_t)c * state_row); };
      auto at = [&](int q) { return FULL ? LPC * q : ang.k[q] - ang.k[0]; };
      V4 own[APL];
#pragma unroll
      for (int q = 0; q < APL; ++q) own[q] = S::load(of((uint32_t)cell) + at(q), KK);
      constexpr int UP = rt_batch<T, APL, PAIRED, STATES>::PLM;
      for (int h = h0; h < h1; h += UP) {
        uint32_t j[UP];
        V4 r[UP], r0[UP], r1[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) {
          const bool v = h + u < h1;
          const int i = (v ? h + u : h0) - H0;
          j[u] = (uint32_t)s_nbr[i];
          r[u] = s_an[i];
          r0[u] = s_rel[2 * i];
          r1[u] = s_rel[2 * i + 1];
          if (!v) r[u] = V4{T(0), T(0), T(0), T(0)};
        }
        T g[UP][P], m2b[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) {
          const T ax = sc * r[u].x, ay = sc * r[u].y, az = sc * r[u].z, nb = -(sd * r[u].w);
          m2b[u] = nb + nb;
#pragma unroll
          for (int q = 0; q < P; ++q) g[u][q] = rt_face_speed(ax, ay, az, nb, ang.x[q], ang.y[q], ang.z[q]);
        }
        // The antipode's speed: in FP64 with no rounding on top of that of g; in FP32 as in the upwind loop,
        // written out where it is used (through a call the 12-angle form loses a wave per SIMD).
        constexpr bool FP64 = sizeof(T) == 8;
        T g2d[UP][P];
        if (FP64)
#pragma unroll
          for (int u = 0; u < UP; ++u)
#pragma unroll
            for (int q = 0; q < P; ++q)
              g2d[u][q] = rt_antipode_speed<T>(sc * r[u].x, sc * r[u].y, sc * r[u].z, -(sd * r[u].w), ang.x[q],
                                               ang.y[q], ang.z[q]);
        V4 x[UP][P], x2[UP][P];  // x2: set, and used, where a pair's other state is needed
        bool more[UP];           // a face fast enough that both directions of a pair enter through it
#pragma unroll
        for (int u = 0; u < UP; ++u) {
          const typename S::part *n = of(j[u]), *across = n + LPC * P;
          more[u] = false;
#pragma unroll
          for (int q = 0; q < P; ++q) {
            const bool in = g[u][q] < T(0), in2 = (FP64 ? g2d[u][q] : m2b[u] - g[u][q]) < T(0);
            x[u][q] = S::load((PAIRED && STATES < 2 && !in ? across : n) + at(q), KK);
            if (PAIRED && STATES == 2) x2[u][q] = S::load(across + at(q), KK);
            more[u] |= PAIRED && in && in2;
          }
          if (PAIRED && STATES == 1 && more[u]) {
#pragma unroll
            for (int q = 0; q < P; ++q)
              if (g[u][q] < T(0) && (FP64 ? g2d[u][q] : m2b[u] - g[u][q]) < T(0)) x2[u][q] = S::load(across + at(q), KK);
          }
        }
#pragma unroll
        for (int u = 0; u < UP; ++u) {
          // the states of the face's two sides
          auto here = [&](const V4 &o) { return o.x + o.y * r0[u].x + o.z * r0[u].y + o.w * r0[u].z; };
          auto there = [&](const V4 &o) { return o.x + o.y * r0[u].w + o.z * r1[u].x + o.w * r1[u].y; };
          // In forms 1 and 2 both are formed before one is taken: a select between expressions becomes
          // a branch around the fetches behind them (0.82 of the speed in form 2)
          auto upwind = [&](bool in, T n, const V4 &o) {
            if constexpr (STATES == 0) return in ? n : here(o);
            const T f = here(o);
            return in ? n : f;
          };
#pragma unroll
          for (int q = 0; q < P; ++q) {
            const T n = there(x[u][q]);
            if constexpr (!PAIRED && !FP64) {
              // the speed formed here, behind the fetches, instead of held across them (two steps, K = 51:
              // 48^3 500 -> 490 us, 33^3 205 -> 200; K = 61, 40^3 319 -> 314; FP64, K = 90, 24^3 2% slower)
              const T gu = rt_face_speed(sc * r[u].x, sc * r[u].y, sc * r[u].z, -(sd * r[u].w), ang.x[q], ang.y[q],
                                         ang.z[q]);
              const T f = here(own[q]);
              acc[q] -= gu * (gu < T(0) ? n : f);
              continue;
            }
            const bool in = g[u][q] < T(0);
            acc[q] -= g[u][q] * upwind(in, n, own[q]);
            if (PAIRED) {
              const T g2 = FP64 ? g2d[u][q] : m2b[u] - g[u][q];
              const T n2 = STATES == 2 ? there(x2[u][q]) : n;
              const bool in2 = g2 < T(0), both = STATES < 2 && in && in2;
              const T to = acc[q + P] - g2 * upwind(in2, n2, own[q + P]);
              acc[q + P] = both ? acc[q + P] : to;
            }
          }
          if (PAIRED && STATES < 2 && more[u]) {
#pragma unroll
            for (int q = 0; q < P; ++q) {
              const T g2 = FP64 ? g2d[u][q] : m2b[u] - g[u][q];
              if (g[u][q] < T(0) && g2 < T(0))
                acc[q + P] -= g2 * there(STATES == 1 ? x2[u][q] : S::load(of(j[u]) + at(q + P), KK));
            }
          }
        }
      }
    }
    if constexpr (TRANSPOSE) {
#pragma unroll
      for (int q = 0; q < APL; ++q) Ic[q] = acc[q];
    } else {
      // I' = I (V/V') + (charge through the faces)/V'.  The ratio V/V' = 1 - dt D/V' is
      // formed in FP64, so on a still mesh it is exactly one: the stored intensities then
      // carry no per-cell rounding of V that would repeat, with one sign, every step.
      const double iV = rt_rcp(Vnew);
      const T cr = (T)(1.0 - dV * iV), ci = (T)iV;
#pragma unroll
      for (int q = 0; q < APL; ++q) Ic[q] = Ic[q] * cr + acc[q] * ci;
    }
    if constexpr (MODE == 1) {
      if (a.I_star_out) {
        T *o = (T *)a.I_star_out + row;
        ang.write_lane(o + ang.k[0], o + k_single, Ic);
      }
    }
  }

  if constexpr (MODE <= 2) {
    if (a.do_source) rt_source_cell<T, LPC, APL>(a, ang, cell, l, Ic);
  }
  if constexpr (MODE >= 4) {
    // Ic holds dL/dI^{n+1} of the cell; the reverse of the source of step n turns it into
    // dL/dI* / V' (V' = Vnew, the end-of-step volume of step n), reading the step's output
    T Io[APL];
    const T *In = (const T *)a.I_next + row;
    ang.read_lane(In + ang.k[0], In + k_single, Io);
    rt_source_vjp_cell<T, LPC, APL>(a, ang, cell, l, Io, Ic, Vnew);
  }

  {
    T *o = (T *)a.I_out + row;
    ang.template write_lane<PAST>(o + ang.k[0], o + k_single, Ic);
  }
  if ((MODE == 1 || MODE == 2) && l == 0 && a.vol_out) a.vol_out[cell] = Vnew;
  if (MODE == 1 && l == 0 && a.src_tape_out) a.src_tape_out[RT_SRC_TAPE * cell + RT_TAPE_V] = Vstart;
}

size_t rt_step_lds(int mode, size_t v4, int hf_cap) {
  const bool faces = mode >= 1 && mode <= 4;
  return faces ? ((mode == 2 ? 3 : 1) * v4 + sizeof(int32_t)) * (size_t)hf_cap : 0;
}

template <typename T, int LPC, int APL, bool FULL, int PAIRED>
hipError_t launch_plm(const rt_step_args &a, int64_t nblk, dim3 grid, size_t smem, hipStream_t s) {
  const dim3 block(RT_BLOCK);
  const bool past = rt_whole_lines<T, LPC, APL, FULL>() &&
                    (a.N > RT_PAST_CELLS || (int64_t)sizeof(T) * a.N * a.K > RT_PAST_BYTES);
  const int states = PAIRED ? rt_states<T>(LPC, APL, PAIRED, nblk) : 0;
  // only the forms rt_states can choose for this layout are built
  constexpr bool BOTH = PAIRED && sizeof(T) == 4;
  constexpr bool AHEAD = PAIRED && (sizeof(T) == 4 ? APL >= 8 || LPC == 4 : PAIRED == 2 && (APL == 8 || APL == 10));
  constexpr bool BEHIND = !PAIRED || sizeof(T) == 8 || LPC == 8;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, smem, s, a, nblk);
    return hipGetLastError();
  };
  if constexpr (BOTH)
    if (states == 2) return launch(k_step<T, LPC, APL, 2, FULL, PAIRED, 2>);
  if constexpr (AHEAD)
    if (states == 1) return launch(k_step<T, LPC, APL, 2, FULL, PAIRED, 1>);
  if constexpr (BEHIND)
    if (states == 0 && !past) return launch(k_step<T, LPC, APL, 2, FULL, PAIRED>);
  if constexpr (rt_whole_lines<T, LPC, APL, FULL>())
    if (states == 0 && past) return launch(k_step<T, LPC, APL, 2, FULL, PAIRED, 0, true>);
  return hipErrorInvalidValue;
}

// Staging needs (records per half-face) x (half-faces of the largest range of the
// workgroup's cells) bytes of LDS; a layout that would need more than a workgroup may
// use (160 KiB on gfx950) is refused with hipErrorInvalidConfiguration (the dispatch then
// tries the general layout, whose 16-cell workgroups the upload checked to fit).
template <typename T, int LPC, int APL, bool FULL, int PAIRED>
hipError_t launch_mode(const rt_step_args &args, hipStream_t s) {
  using V4 = typename rt_vec4<T>::type;
  rt_step_args a = args;
  a.hf_cap = LPC == 16 ? a.hf_cap16 : LPC == 8 ? a.hf_cap32 : a.hf_cap64;
  a.wg_order = LPC == 16 ? a.wg_order16 : LPC == 8 ? a.wg_order32 : a.wg_order64;
  const int64_t cpb = RT_BLOCK / LPC;
  const int64_t nblk = (a.N + cpb - 1) / cpb;
  const dim3 grid((unsigned)rt_grid_for(nblk)), block(RT_BLOCK);
  const size_t smem = rt_step_lds(a.do_transport, sizeof(V4), a.hf_cap);
  if (smem > (size_t)a.lds_max) return hipErrorInvalidConfiguration;
  switch (a.do_transport) {
    case 0: hipLaunchKernelGGL((k_step<T, LPC, APL, 0, FULL, PAIRED>), grid, block, smem, s, a, nblk); break;
    case 1: hipLaunchKernelGGL((k_step<T, LPC, APL, 1, FULL, PAIRED>), grid, block, smem, s, a, nblk); break;
    case 2: return launch_plm<T, LPC, APL, FULL, PAIRED>(a, nblk, grid, smem, s);
    case 3: hipLaunchKernelGGL((k_step<T, LPC, APL, 3, FULL, PAIRED>), grid, block, smem, s, a, nblk); break;
    case 4: hipLaunchKernelGGL((k_step<T, LPC, APL, 4, FULL, PAIRED>), grid, block, smem, s, a, nblk); break;
    case 5: hipLaunchKernelGGL((k_step<T, LPC, APL, 5, FULL, PAIRED>), grid, block, smem, s, a, nblk); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, int LPC, int APL> hipError_t launch(const rt_step_args &a, hipStream_t s) {
  return a.K == LPC * APL ? launch_mode<T, LPC, APL, true, 0>(a, s)
                          : launch_mode<T, LPC, APL, false, 0>(a, s);
}

template <typename T, int PAIRED> hipError_t dispatch_paired(const rt_step_args &a, hipStream_t s) {
  switch (rt_paired_lanes(a.K)) {  // 0 (no paired layout for K) matches no case
    case 0x0802: return launch_mode<T, 8, 2, true, PAIRED>(a, s);
    case 0x0804: return launch_mode<T, 8, 4, true, PAIRED>(a, s);
    case 0x0806: return launch_mode<T, 8, 6, true, PAIRED>(a, s);
    case 0x0808: return launch_mode<T, 8, 8, true, PAIRED>(a, s);
    case 0x080a: return launch_mode<T, 8, 10, true, PAIRED>(a, s);
    case 0x080c: return launch_mode<T, 8, 12, true, PAIRED>(a, s);
    case 0x0402: return launch_mode<T, 4, 2, true, PAIRED>(a, s);
    case 0x0406: return launch_mode<T, 4, 6, true, PAIRED>(a, s);
    case 0x040a: return launch_mode<T, 4, 10, true, PAIRED>(a, s);
  }
  return hipErrorInvalidConfiguration;
}

template <typename T> hipError_t dispatch_general16(const rt_step_args &a, hipStream_t s) {
  switch ((a.K + 15) / 16) {
    case 1: return launch<T, 16, 1>(a, s);
    case 2: return launch<T, 16, 2>(a, s);
    case 3: return launch<T, 16, 3>(a, s);
    case 4: return launch<T, 16, 4>(a, s);
    case 5: return launch<T, 16, 5>(a, s);
    case 6: return launch<T, 16, 6>(a, s);
    case 7: return launch<T, 16, 7>(a, s);
    case 8: return launch<T, 16, 8>(a, s);
  }
  return hipErrorInvalidValue;
}

// The general layout for K; when 8 lanes per cell (32-cell workgroups) cannot stage their
// face records, 16 lanes (16-cell workgroups, which the upload checked to fit) serve K.
template <typename T> hipError_t dispatch_general(const rt_step_args &a, hipStream_t s) {
  const int lanes = rt_step_lanes(a.K, 0);
  if ((lanes >> 8) == 16) return dispatch_general16<T>(a, s);
  hipError_t e = hipErrorInvalidValue;
  switch (lanes) {
    case 0x0801: e = launch<T, 8, 1>(a, s); break;
    case 0x0802: e = launch<T, 8, 2>(a, s); break;
    case 0x0803: e = launch<T, 8, 3>(a, s); break;
    case 0x0804: e = launch<T, 8, 4>(a, s); break;
    case 0x0805: e = launch<T, 8, 5>(a, s); break;
    case 0x0806: e = launch<T, 8, 6>(a, s); break;
    case 0x0807: e = launch<T, 8, 7>(a, s); break;
    case 0x0808: e = launch<T, 8, 8>(a, s); break;
  }
  return e == hipErrorInvalidConfiguration ? dispatch_general16<T>(a, s) : e;
}

// Antipodal sets take the paired kernel when it has a lane layout for K and its staging
// fits in LDS; everything else (and that fallback) the general kernel.
template <typename T> hipError_t dispatch(const rt_step_args &a, hipStream_t s) {
  if (a.paired) {
    const hipError_t e = a.paired == 2 ? dispatch_paired<T, 2>(a, s) : dispatch_paired<T, 1>(a, s);
    if (e != hipErrorInvalidConfiguration) return e;
  }
  return dispatch_general<T>(a, s);
}

}  // namespace

bool rt_plm_pairs(const rt_step_args &a, int dtype) {
  const int lanes = a.paired ? rt_paired_lanes(a.K) : 0;
  const size_t v4 = dtype == RT_F32 ? sizeof(float4) : sizeof(double4);
  return lanes && rt_step_lds(2, v4, (lanes >> 8) == 8 ? a.hf_cap32 : a.hf_cap64) <= (size_t)a.lds_max;
}

hipError_t rt_launch_step(const rt_step_args &a, int dtype, hipStream_t s) {
  return dtype == RT_F32 ? dispatch<float>(a, s) : dispatch<double>(a, s);
}
