// Implicit source update with temperature-dependent opacities (section 2.3: the
// temperature equation solved by Newton-Raphson iteration), one cell per group of LPC
// lanes.  kP(T) = kP0 (T/T_ref)^bP, kJ(T) = kJ0 (T/T_ref)^bJ at T^{n+1}; ks constant.
// With J~ eliminated the temperature equation is
//   f(T) = rho cv (T - T^n) + dt c rho [kP a T^4 S1 - 4 pi kJ SI] / D,
// whose comoving sums depend on T through chi = kJ(T) + ks; every evaluation sums the
// angles again (S1, SG, SI and their chi-derivatives) and reduces over the lanes, so
// all lanes of a cell take the same steps.  The bracket's far end is found from T^n
// (doubling upward while f < 0, halving downward while f > 0); Newton steps start at T^n,
// the bracket's near end from the first step on, and are kept inside [T^n, hi] (or
// [lo, T^n]; bisection when a step leaves it) until a step changes T by at most 1e-14 T, or is
// short enough that the next would (such a step is taken as it is); at most 200 evaluations,
// about 5 in practice.  Where f
// has several roots this gives the first met from T^n in the direction of f's sign.
// Per-angle arithmetic is FP64 in both precision forms; the update and the bookkeeping
// are those of the grey source.
#include "rt_step_common.h"

namespace {

struct kT_eval {
  double kP, kJ, S1, SG, SI, D, f, fp;
};

// x^b for b = half2 / 2 with a whole |half2| <= 40 (the same for every thread), x > 0 (or 0 with
// b > 0), by repeated squaring of x, its reciprocal or its reciprocal root, each value carried with its
// rounding error (p + pl, x + xl): within an ulp.  Squaring plain doubles doubles their errors each
// time, |b| + 3 ulp in all, where exp(b ln x) is within |b ln x| + 2, which is less near x = 1.
__device__ __forceinline__ double rt_half_power(double x, int half2) {
  const double x0 = x;
  unsigned m = half2 < 0 ? -half2 : half2;
  if (m == 0) return 1.0;
  double xl = 0.0, p, pl;
  if (m & 1u) {
    double s = __builtin_amdgcn_rsq(x);
    double e = fma(-(x * s), s, 1.0);
    s = fma(s * e, fma(0.375, e, 0.5), s);
    const double h = x * s, hl = fma(x, s, -h);  // h: the root
    e = fma(-hl, s, fma(-h, s, 1.0));
    const double sl = 0.5 * s * e;
    if (half2 < 0) {
      p = s;
      pl = sl;
      const double q = s * s;
      xl = fma(s, s, -q) + 2.0 * s * sl;
      x = q;
    } else {
      p = h;
      pl = fma(x, sl, hl);
    }
    m >>= 1;
  } else {
    if (half2 < 0) {
      const double r = rt_rcp(x);
      xl = fma(-x, r, 1.0) * r;
      x = r;
    }
    for (m >>= 1; !(m & 1u); m >>= 1) {
      const double q = x * x;
      xl = fma(x, x, -q) + 2.0 * x * xl;
      x = q;
    }
    p = x;
    pl = xl;
    m >>= 1;
    if (m) {
      const double q = x * x;
      xl = fma(x, x, -q) + 2.0 * x * xl;
      x = q;
    }
  }
  while (m > 1u) {
    if (m & 1u) {
      const double q = p * x;
      pl = fma(p, x, -q) + fma(p, xl, pl * x);
      p = q;
    }
    m >>= 1;
    const double q = x * x;
    xl = fma(x, x, -q) + 2.0 * x * xl;
    x = q;
  }
  if (m == 0) x = 1.0, xl = 0.0;
  const double v = fma(p, x, fma(p, xl, pl * x));
  if (half2 > 0 && x0 == 0.0) return 0.0;
  return v == v ? v : p * x;  // an overflow leaves no remainder
}

// What bounds the kernel is FP64 vector issue: about five evaluations per cell, each over all
// angles, so an evaluation is written for few instructions.  With u = y chi every sum is a
// combination of the five sums over r'^2, r' = (1 + u) r:  with e = 1 / (1 + u),
// 1 / r' = e + u e Gamma, so  sum Wt r = e (e P0 + u e P1),  sum Wt Gamma r = e (e P1 + u e P2)
// and likewise for SI, and the chi-derivatives are -e^2 P1, -e^2 P2, -e^2 Q1: sums of positive
// terms, no cancellation, and r' of order one keeps the squares in range for any u.  A power
// law with a whole or half-whole exponent is a few multiplications instead of log and exp.
// The directions and weights come from LDS (read by every lane before and after the
// iteration).  64^3 x 80, exponent -3.5, FP32, kernel alone, when each was made: 272 -> 175 us (the
// sums and powers alone 240; one evaluation fewer at either end of the iteration 187; three waves per
// SIMD the rest).  At 128^3 x 80 1.14 ms with plain powers, 1.15 with powers that round once.
// HALF: both exponents are whole or half-whole numbers (rt_half_power).
//
// Waves per SIMD the register use is held to: three where the spill stays within a few values (4 to 11
// here, at 10 angles per lane in pairs and at 8 without), against 196 to 228 registers and two waves.
// Steps of unpaired sets at 8 angles per lane, three waves and two: 40^3 x 120 FP32 121 and 146 us,
// FP64 134 and 150; 40^3 x 61 75 and 86, 76 and 84; 24^3 x 61 the same.  log and exp take 30 registers
// more, and there three waves spill 50 (64^3 x 80 step, FP32: 411 against 370 us).
template <int APL, int PAIRED, bool HALF> struct rt_kT_waves {
  static constexpr int value = HALF && (!PAIRED || APL <= 10) ? 3 : PAIRED && APL > 10 ? 1 : 2;
};
// The update of one cell.  row: its incoming intensities, .first(ang, q) before the iteration and
// .again(ang, q) after it, and .store(ang, out) for the updated ones.
template <typename T, int LPC, int APL, bool HALF, typename Ang, typename Row>
__device__ __forceinline__ void rt_kT_cell(const rt_kT_args &a, const double *s_dir, const double *s_w, int64_t cell,
                                           int l, const Row &row) {
  const int K = a.K;
  Ang ang;
  ang.load(s_dir, s_w, K, l);

  const double rho = a.rho[cell];
  const double m0 = a.mom[3 * cell], m1 = a.mom[3 * cell + 1], m2 = a.mom[3 * cell + 2];
  const double Eg = a.etot[cell];
  const double c = a.c_light, fourpi = 4.0 * RT_PI;
  // reciprocals (within an ulp) and products instead of FP64 divisions
  const double irho = rt_rcp(rho), ic = rt_rcp(c);
  const double vx = m0 * irho, vy = m1 * irho, vz = m2 * irho;
  const double gam = rsqrt(1.0 - (vx * vx + vy * vy + vz * vz) * (ic * ic));
  double Gm[APL], Wt[APL], WI[APL];  // Gamma, W~ and W~ I~
  double norm = 0.0;
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    const double I0 = (double)row.first(ang, q);
    const double vn = vx * ang.dx(q) + vy * ang.dy(q) + vz * ang.dz(q);
    Gm[q] = gam * (1.0 - vn * ic);
    const double iG = rt_rcp(Gm[q]);
    Wt[q] = ang.wt(q) * (iG * iG);
    WI[q] = ang.wt(q) * (Gm[q] * Gm[q]) * I0;  // W Gamma^-2 Gamma^4 I
    norm += Wt[q];
  }
  norm = rt_group_sum<LPC>(norm);
  const double inorm = rt_rcp(norm);
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    Wt[q] *= inorm;
    WI[q] *= inorm;
  }
  const double y = a.dt * a.c_red * rho;
  const double rcv = rho * a.cv;
  const double Tn = (Eg - 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) * irho) * rt_rcp(rcv);
  const double iTref = rt_rcp(a.T_ref);
  const double kJ0 = a.kJ0[cell], ks = a.ks[cell];
  // Gas with less total than kinetic energy has no temperature.  The logarithm makes such a cell
  // NaN, which the diagnostics count; multiplication would not (x^2 of a negative x is as good as
  // any), so there the opacity is made NaN here.  At T = 0 only two rising laws have a value.
  const bool cold = HALF && (Tn < 0.0 || (Tn == 0.0 && (a.bP2 <= 0 || a.bJ2 <= 0)));
  const double kP0 = cold ? NAN : a.kP0[cell];

  auto evaluate = [&](double Tq) {
    kT_eval e;
    const double x = Tq * iTref;
    double pP, pJ;
    if constexpr (HALF) {
      pP = rt_half_power(x, a.bP2);
      pJ = a.bJ2 == a.bP2 ? pP : rt_half_power(x, a.bJ2);
    } else {
      // (T/T_ref)^b as exp(b ln(T/T_ref)): within (|b ln(T/T_ref)| + 2) ulp, and far cheaper
      // than pow (whose code alone, even on a branch not taken, costs this kernel registers).
      // The error stays below the Newton stopping tolerance (1e-14 T) while |b ln| < ~40;
      // beyond that the bracketed iteration still ends, through its bisection steps.
      const double lt = log(x);
      pP = exp(a.bP * lt);
      pJ = a.bJ == a.bP ? pP : exp(a.bJ * lt);
    }
    e.kP = kP0 * pP;
    e.kJ = kJ0 * pJ;
    const double u = y * (e.kJ + ks);
    const double ie = rt_rcp(1.0 + u), ue = u * ie;
    double P0 = 0, P1 = 0, P2 = 0, Q0 = 0, Q1 = 0;
#pragma unroll
    for (int q = 0; q < APL; ++q) {
      const double r = rt_rcp(fma(ue, Gm[q], ie));
      const double r2 = r * r;
      const double w = Wt[q] * r2, wG = w * Gm[q], wI = WI[q] * r2;
      P0 += w;
      P1 += wG;
      P2 = fma(wG, Gm[q], P2);
      Q0 += wI;
      Q1 = fma(wI, Gm[q], Q1);
    }
    P0 = rt_group_sum<LPC>(P0);
    P1 = rt_group_sum<LPC>(P1);
    P2 = rt_group_sum<LPC>(P2);
    Q0 = rt_group_sum<LPC>(Q0);
    Q1 = rt_group_sum<LPC>(Q1);
    e.S1 = ie * fma(ue, P1, ie * P0);
    e.SG = ie * fma(ue, P2, ie * P1);
    e.SI = ie * fma(ue, Q1, ie * Q0);
    e.D = e.S1 + y * e.kJ * e.SG;
    const double T3 = Tq * Tq * Tq, T4 = T3 * Tq;
    const double Nn = e.kP * a.a_rad * T4 * e.S1 - fourpi * e.kJ * e.SI;
    const double iD = rt_rcp(e.D), iTq = rt_rcp(Tq);
    e.f = rcv * (Tq - Tn) + a.dt * c * rho * Nn * iD;
    const double dkP = a.bP * e.kP * iTq, dkJ = a.bJ * e.kJ * iTq;
    const double dr = -y * dkJ * (ie * ie);
    const double dS1 = dr * P1, dSG = dr * P2, dSI = dr * Q1;
    const double dD = dS1 + y * (dkJ * e.SG + e.kJ * dSG);
    const double dN = dkP * a.a_rad * T4 * e.S1 + e.kP * a.a_rad * 4.0 * T3 * e.S1 + e.kP * a.a_rad * T4 * dS1 -
                      fourpi * (dkJ * e.SI + e.kJ * dSI);
    e.fp = rcv + a.dt * c * rho * (dN * e.D - Nn * dD) * (iD * iD);
    return e;
  };

  // Safeguarded Newton from T^n, one loop with a single evaluation site.  The bracket's far end
  // is the first of 2 T^n, 4 T^n, ... with f >= 0 (f(T^n) < 0; else of T^n / 2, ... with f <= 0),
  // but it is only looked for (modes 1 and 2) once a step would leave the first interval
  // (`open`): steps that stay inside it are the same whatever the far end is, and its
  // evaluation is one of about six.  A step is the last when it is at most 1e-14 T, or when it is
  // at most 1e-8 T and the step after it, about step^3 / previous^2 by quadratic convergence
  // (both of them Newton steps), would be at most 2e-17 T.  The estimate alone does not do: after
  // a long step the second can be small by accident (100,000 cells far from equilibrium, law
  // -3.5: errors of T up to 1e-12, with the bound on the step 3e-16 as with 1e-14 T alone, at
  // 8.27 evaluations on average against 8.97).
  // The search for the far end keeps nothing of the evaluation at the current T: it is done
  // again there when the end is found (held through the loop it cost a fifth of the registers).
  double Tq = Tn, lo = Tn, hi = Tn, x = Tn, prev = 0.0;
  int mode = 0;  // 0: at T^n; 1: doubling hi; 2: halving lo; 3: Newton
  bool open = false, up = false, done = false;
  kT_eval e;
  for (int nev = 1;; ++nev) {
    e = evaluate(x);
    const bool neg = e.f < 0.0, pos = e.f > 0.0;
    if (mode == 1 || mode == 2) {
      const bool on = nev < 200 && (up ? neg : pos);
      hi = up && on ? 2.0 * hi : hi;
      lo = !up && on ? 0.5 * lo : lo;
      mode = on ? mode : 3;
      done = nev >= 200;
      x = !on ? Tq : up ? hi : lo;
      continue;
    }
    Tq = x;
    if (done || nev >= 200 || e.f == 0.0) break;
    if (mode == 0) {
      mode = 3;
      up = neg;
      open = neg || pos;
      hi = neg ? 2.0 * Tn : hi;
      lo = pos ? 0.5 * Tn : lo;
    }
    lo = neg ? Tq : lo;
    hi = neg ? hi : Tq;
    open = open && up == neg;
    double Tx = Tq - e.f * rt_rcp(e.fp);
    const double step = fabs(Tx - Tq);
    const bool in = Tx > lo && Tx < hi;
    // a step within the tolerance has converged and is taken as it is; a larger one that
    // leaves the bracket is replaced by bisection
    done = step <= 1e-14 * Tq;
    if (!done && !in && open) {
      open = false;
      mode = up ? 1 : 2;
      x = up ? hi : lo;
      continue;
    }
    x = done || in ? Tx : 0.5 * (lo + hi);
    done = done || (in && step <= 1e-8 * Tq && step * step * step <= 2e-17 * Tq * (prev * prev));
    prev = in ? step : 0.0;
  }

  // The directions and weights are needed before the iteration and after it, not in it: read
  // them again here (through an offset the compiler cannot prove zero, so it does not keep
  // the first copy live through the iteration) instead of holding them in registers.
  int again = 0;
  asm volatile("" : "+s"(again));
  ang.load(s_dir + again, s_w + again, K, l);
  const double T4 = Tq * Tq * Tq * Tq;
  const double planck = a.a_rad * T4 * (1.0 / fourpi);
  const double Jc = (e.SI + y * e.kP * e.SG * planck) * rt_rcp(e.D);
  const double yS = y * (e.kP * planck + ks * Jc), yc = y * (e.kJ + ks);
  double dE = 0, dFx = 0, dFy = 0, dFz = 0;
  T out[APL];
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    // I' = (Gamma^4 I + y Gamma S) r / Gamma^4 = r (I + y S / Gamma^3), the incoming value
    // read again rather than held through the iteration
    const double I0 = (double)row.again(ang, q);
    const double iG = rt_rcp(Gm[q]);
    out[q] = (T)((I0 + yS * (iG * iG * iG)) * rt_rcp(1.0 + yc * Gm[q]));
    const double wd = ang.wt(q) * (I0 - (double)out[q]);
    dE += wd;
    dFx += wd * ang.dx(q);
    dFy += wd * ang.dy(q);
    dFz += wd * ang.dz(q);
  }
  row.store(ang, out);
  dE = rt_group_sum<LPC>(dE);
  dFx = rt_group_sum<LPC>(dFx);
  dFy = rt_group_sum<LPC>(dFy);
  dFz = rt_group_sum<LPC>(dFz);
  if (l == 0) {
    a.etot[cell] = Eg + a.e_gain * dE;
    a.mom[3 * cell] = m0 + a.m_gain * dFx;
    a.mom[3 * cell + 1] = m1 + a.m_gain * dFy;
    a.mom[3 * cell + 2] = m2 + a.m_gain * dFz;
    if (a.T_out) a.T_out[cell] = Tq;
  }
}

__device__ __forceinline__ void rt_kT_stage_angles(const rt_kT_args &a, double *s_dir, double *s_w) {
  for (int i = threadIdx.x; i < 3 * a.K; i += RT_BLOCK) s_dir[i] = a.dirs[i];
  for (int i = threadIdx.x; i < a.K; i += RT_BLOCK) s_w[i] = a.W[i];
}

template <typename T, int LPC, int APL, bool FULL, int PAIRED, bool HALF>
__global__ __launch_bounds__(RT_BLOCK) __attribute__((amdgpu_waves_per_eu(rt_kT_waves<APL, PAIRED, HALF>::value))) void
k_source_kT(rt_kT_args a, int64_t nblk) {
  using Ang = rt_step_angles<double, LPC, APL, FULL, PAIRED>;
  constexpr int CPB = RT_BLOCK / LPC;
  __shared__ double s_dir[3 * RT_K_MAX], s_w[RT_K_MAX];
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;  // whole workgroup
  rt_kT_stage_angles(a, s_dir, s_w);
  __syncthreads();
  const int64_t cell = lb * CPB + threadIdx.x / LPC;
  if (cell >= a.N) return;
  struct Row {
    T *I;
    __device__ __forceinline__ T first(const Ang &ang, int q) const { return I[ang.k[q]]; }
    __device__ __forceinline__ T again(const Ang &ang, int q) const { return I[ang.k[q]]; }
    __device__ __forceinline__ void store(const Ang &ang, const T (&v)[APL]) const {
#pragma unroll
      for (int q = 0; q < APL; ++q)
        if (ang.ok[q]) I[ang.k[q]] = v[q];
    }
  };
  rt_kT_cell<T, LPC, APL, HALF, Ang>(a, s_dir, s_w, cell, threadIdx.x % LPC, Row{(T *)a.I + cell * (int64_t)a.K});
}

// The step: upwind transport into registers, then the source.  As two launches the transported
// intensities were written, read twice and written again, and the transport (bound by its
// gathers) and the source (bound by FP64 issue) each left the other's unit idle.  The
// transported values wait in LDS, in words of the lane's own, through the iteration.
// A call at 64^3 x 80, exponent -3.5, FP32, its state reset included: 310 -> 274 us when it was made,
// 269 now.  FP64 rows of 10 angles per lane take two waves per SIMD (198 registers), measured at K = 80:
// 24^3 26.5 us against 28.7 with three, 48^3 131 against 128, 64^3 322 against 360.
template <typename T, int APL, int PAIRED, bool HALF> struct rt_kT_step_waves {
  static constexpr int value = sizeof(T) == 8 && PAIRED && APL == 10 ? 2 : rt_kT_waves<APL, PAIRED, HALF>::value;
};
template <typename T, int LPC, int APL, bool FULL, int PAIRED, bool HALF>
__global__ __launch_bounds__(RT_BLOCK)
__attribute__((amdgpu_waves_per_eu(rt_kT_step_waves<T, APL, PAIRED, HALF>::value))) void
k_step_kT(rt_step_args t, rt_kT_args a, int64_t nblk) {
  using V4 = typename rt_vec4<T>::type;
  using AngT = rt_step_angles<T, LPC, APL, FULL, PAIRED, true>;
  using Ang = rt_step_angles<double, LPC, APL, FULL, PAIRED, true>;  // the same slots
  constexpr int CPB = RT_BLOCK / LPC;
  __shared__ double s_dir[3 * RT_K_MAX], s_w[RT_K_MAX];
  __shared__ T s_rows[APL * RT_BLOCK];
  extern __shared__ __align__(16) unsigned char rt_smem[];
  V4 *s_an = (V4 *)rt_smem;
  int32_t *s_nbr = (int32_t *)(s_an + t.hf_cap);
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;  // whole workgroup
  const int64_t c0 = lb * CPB, c1 = c0 + CPB < t.N ? c0 + CPB : t.N;
  const int g = threadIdx.x / LPC, l = threadIdx.x % LPC;
  const bool live = c0 + g < t.N;
  const int64_t cell = live ? c0 + t.wg_order[c0 + g] : c0;
  const int H0 = t.row_ptr[c0];
  {
    const V4 *an = (const V4 *)t.hf_an;
    const int nH = t.row_ptr[c1] - H0;  // <= hf_cap by construction
    for (int i = threadIdx.x; i < nH; i += RT_BLOCK) {
      s_nbr[i] = t.hf_nbr[H0 + i];
      s_an[i] = an[H0 + i];
    }
  }
  rt_kT_stage_angles(a, s_dir, s_w);
  __syncthreads();
  if (!live) return;
  T I[1][APL];
  {
    AngT ang;
    ang.load(t.dirs, t.W, t.K, l);
    const int k_single = AngT::SINGLE ? ang.k[AngT::P - 1] : ang.k[0];
    const double dD = t.D[cell];
    const double Vnew = rt_vol_next(t.vol_in[cell], t.dt, dD);
    const double iV = rt_rcp(Vnew);
    const int h0 = t.row_ptr[cell] - H0, nh = t.row_ptr[cell + 1] - H0 - h0;
    rt_upwind_sweep<T, LPC, APL, 1>(t, ang, 0, cell, (const T *)t.I_in, k_single, s_nbr + h0, s_an + h0, nh,
                                    (T)(1.0 - t.dt * dD * iV), (T)iV, I);
    if (l == 0) t.vol_out[cell] = Vnew;
  }
  T *own = s_rows + threadIdx.x;
#pragma unroll
  for (int q = 0; q < APL; ++q) own[q * RT_BLOCK] = I[0][q];
  struct Row {
    const T *own;
    T *out;
    __device__ __forceinline__ T first(const Ang &, int q) const { return own[q * RT_BLOCK]; }
    __device__ __forceinline__ T again(const Ang &, int q) const { return own[q * RT_BLOCK]; }
    __device__ __forceinline__ void store(const Ang &ang, const T (&v)[APL]) const {
#pragma unroll
      for (int q = 0; q < APL; ++q)
        if (ang.ok[q]) out[ang.k[q]] = v[q];
    }
  };
  rt_kT_cell<T, LPC, APL, HALF, Ang>(a, s_dir, s_w, cell, l, Row{own, (T *)t.I_out + cell * (int64_t)t.K});
}

rt_kT_args with_powers(rt_kT_args a, bool &half) {
  a.bP2 = (int)(2.0 * a.bP);
  a.bJ2 = (int)(2.0 * a.bJ);
  half = a.bP2 == 2.0 * a.bP && a.bJ2 == 2.0 * a.bJ;
  return a;
}

struct rt_source_only {
  rt_kT_args a;
  int K() const { return a.K; }
  int paired() const { return a.paired; }
  template <typename T, int LPC, int APL, bool FULL, int PAIRED> hipError_t run(hipStream_t s) const {
    bool half;
    const rt_kT_args b = with_powers(a, half);
    const int64_t cpb = RT_BLOCK / LPC;
    const int64_t nblk = (b.N + cpb - 1) / cpb;
    const dim3 grid((unsigned)rt_grid_for(nblk)), block(RT_BLOCK);
    if (half) hipLaunchKernelGGL((k_source_kT<T, LPC, APL, FULL, PAIRED, true>), grid, block, 0, s, b, nblk);
    else hipLaunchKernelGGL((k_source_kT<T, LPC, APL, FULL, PAIRED, false>), grid, block, 0, s, b, nblk);
    return hipGetLastError();
  }
};

// hipErrorInvalidConfiguration: the paired layout does not fit and the general one is tried (on
// meshes of 50 to 200 faces per cell 1.0 to 1.4 times as fast as the separate launches in the
// paired layout), or that does not either and the step takes its separate launches.
struct rt_whole_step {
  rt_step_args t;
  rt_kT_args a;
  int K() const { return a.K; }
  int paired() const { return a.paired; }
  template <typename T, int LPC, int APL, bool FULL, int PAIRED> hipError_t run(hipStream_t s) const {
    bool half;
    const rt_kT_args b = with_powers(a, half);
    rt_step_args u = t;
    u.hf_cap = LPC == 16 ? t.hf_cap16 : LPC == 8 ? t.hf_cap32 : t.hf_cap64;
    u.wg_order = LPC == 16 ? t.wg_order16 : LPC == 8 ? t.wg_order32 : t.wg_order64;
    const int64_t cpb = RT_BLOCK / LPC;
    const int64_t nblk = (b.N + cpb - 1) / cpb;
    const dim3 grid((unsigned)rt_grid_for(nblk)), block(RT_BLOCK);
    const size_t smem = (sizeof(typename rt_vec4<T>::type) + sizeof(int32_t)) * (size_t)u.hf_cap;
    const size_t fixed = sizeof(double) * 4 * RT_K_MAX + sizeof(T) * APL * RT_BLOCK;
    // two workgroups per CU at least, as the separate launches have at the same face counts
    if (smem + fixed > (size_t)t.lds_max / 2) return hipErrorInvalidConfiguration;
    if (half) hipLaunchKernelGGL((k_step_kT<T, LPC, APL, FULL, PAIRED, true>), grid, block, smem, s, u, b, nblk);
    else hipLaunchKernelGGL((k_step_kT<T, LPC, APL, FULL, PAIRED, false>), grid, block, smem, s, u, b, nblk);
    return hipGetLastError();
  }
};

// OP is the launch to make in the layout chosen: the source alone, or the step.
template <typename T, int PAIRED, typename OP> hipError_t dispatch_paired(const OP &op, hipStream_t s) {
  switch (rt_paired_lanes(op.K())) {  // 0 (no paired layout for K) matches no case
    case 0x0802: return op.template run<T, 8, 2, true, PAIRED>(s);
    case 0x0804: return op.template run<T, 8, 4, true, PAIRED>(s);
    case 0x0806: return op.template run<T, 8, 6, true, PAIRED>(s);
    case 0x0808: return op.template run<T, 8, 8, true, PAIRED>(s);
    case 0x080a: return op.template run<T, 8, 10, true, PAIRED>(s);
    case 0x080c: return op.template run<T, 8, 12, true, PAIRED>(s);
    case 0x0402: return op.template run<T, 4, 2, true, PAIRED>(s);
    case 0x0406: return op.template run<T, 4, 6, true, PAIRED>(s);
    case 0x040a: return op.template run<T, 4, 10, true, PAIRED>(s);
  }
  return hipErrorInvalidConfiguration;
}

// Antipodal sets with a paired layout put 4 or 8 lanes on a cell (more cells per wave, so the
// per-cell scalar work of each evaluation is shared by fewer lanes); others the general one.
template <typename T, typename OP> hipError_t dispatch(const OP &op, hipStream_t s) {
  if (op.paired()) {
    const hipError_t e = op.paired() == 2 ? dispatch_paired<T, 2>(op, s) : dispatch_paired<T, 1>(op, s);
    if (e != hipErrorInvalidConfiguration) return e;
  }
  switch (rt_step_lanes(op.K(), 0)) {
    case 0x1001: return op.template run<T, 16, 1, false, 0>(s);
    case 0x1002: return op.template run<T, 16, 2, false, 0>(s);
    case 0x1003: return op.template run<T, 16, 3, false, 0>(s);
    case 0x1004: return op.template run<T, 16, 4, false, 0>(s);
    case 0x1005: return op.template run<T, 16, 5, false, 0>(s);
    case 0x1006: return op.template run<T, 16, 6, false, 0>(s);
    case 0x1007: return op.template run<T, 16, 7, false, 0>(s);
    case 0x1008: return op.template run<T, 16, 8, false, 0>(s);
    case 0x0801: return op.template run<T, 8, 1, false, 0>(s);
    case 0x0802: return op.template run<T, 8, 2, false, 0>(s);
    case 0x0803: return op.template run<T, 8, 3, false, 0>(s);
    case 0x0804: return op.template run<T, 8, 4, false, 0>(s);
    case 0x0805: return op.template run<T, 8, 5, false, 0>(s);
    case 0x0806: return op.template run<T, 8, 6, false, 0>(s);
    case 0x0807: return op.template run<T, 8, 7, false, 0>(s);
    case 0x0808: return op.template run<T, 8, 8, false, 0>(s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t rt_launch_source_kT(const rt_kT_args &a, int dtype, hipStream_t s) {
  const rt_source_only op{a};
  return dtype == RT_F32 ? dispatch<float>(op, s) : dispatch<double>(op, s);
}

hipError_t rt_launch_step_kT(const rt_step_args &t, const rt_kT_args &a, int dtype, hipStream_t s) {
  const rt_whole_step op{t, a};
  return dtype == RT_F32 ? dispatch<float>(op, s) : dispatch<double>(op, s);
}
