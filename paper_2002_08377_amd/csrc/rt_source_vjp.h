// Reverse of the implicit source update (section 2.3) of one cell held by a group of LPC
// lanes, in the step kernel's lane layouts, for the fused adjoint modes of the step kernel.
//
// Forward (per cell, with Gamma_k = gamma (1 - v.n_k / c), weights W_k):
//   comoving intensity I0_k = Gamma_k^4 I*_k, Wt_k = W_k Gamma_k^-2 / sum_j W_j Gamma_j^-2,
//   r_k = 1 / (1 + y chi Gamma_k), sums S1 = sum Wt r, SG = sum Wt Gamma r, SI = sum Wt I0 r,
//   the temperature root of A T^4 + B T = C (eq. 33 form; A, C from the sums, B = rho cv),
//   source S = kP a T^4 / 4 pi + ks J, per angle I'_k = (I0_k + y Gamma_k S) r_k Gamma_k^-4,
//   then the gas takes the radiation energy and momentum the update removed (eqs. 35-36).
// The taped forward step stores each cell's 1/sum W Gamma^-2, S1, SG, SI, 1/D and T^{n+1}
// (D = S1 + y kJ SG) with its start-of-step volume and momentum, so the reverse needs no
// sums, no root and no gas state of its own; through the root
// it uses the implicit function theorem, dT = -(T^4 dA + T dB - dC) / (4 A T^3 + B).
//
// The intensities the reverse reads are the step's output I' (which the recompute of a
// segment keeps anyway, one buffer per step) rather than the transported I*: the update
// inverts to Gamma^4 I* + y Gamma S = I' Gamma^4 / r, so the forward need not store I*.
//
// Per-angle arithmetic runs in the intensities' type T, sums over angles and per-cell
// values in FP64, as in the forward source.  On return lam holds dL/dI* divided by the
// cell's end-of-step volume V', the input of the transpose of the upwind charge update.
#pragma once

#include "rt_device.h"

template <typename T, int LPC, int APL, typename Ang>
__device__ __forceinline__ void rt_source_vjp_cell(const rt_step_args &a, const Ang &ang, int64_t cell, int l,
                                                   const T (&Io)[APL], T (&lam)[APL], double Vp) {
  constexpr int P = Ang::P;
  constexpr bool PAIRED = Ang::PAIRED_LAYOUT;
  const double rho = a.rho[cell];
  const double kP = a.kP[cell], kJ = a.kJ[cell], ks = a.ks[cell];
  const double *tp = a.src_tape + RT_SRC_TAPE * cell;
  const double m0 = tp[RT_TAPE_M], m1 = tp[RT_TAPE_M + 1], m2 = tp[RT_TAPE_M + 2];
  const double iQ = tp[RT_TAPE_IQ], S1 = tp[RT_TAPE_S1], SG = tp[RT_TAPE_SG], SI = tp[RT_TAPE_SI];
  const double iD = tp[RT_TAPE_ID], Tq = tp[RT_TAPE_T];
  const double c = a.c_light, ic = a.inv_c, dt = a.dt;
  const double irho = rt_rcp(rho);
  const double vx = m0 * irho, vy = m1 * irho, vz = m2 * irho;
  const double gam = rsqrt(1.0 - (vx * vx + vy * vy + vz * vz) * (ic * ic));
  const double y = dt * a.c_red * rho;
  const double chi = kJ + ks;
  const double rcv = rho * a.cv;
  const double T3 = Tq * Tq * Tq, T4 = T3 * Tq;
  const double planck = a.a_4pi * T4;
  const double Jc = (SI + y * kP * SG * planck) * iD;
  const double Ssrc = kP * planck + ks * Jc;
  const double fourpi = 4.0 * RT_PI;
  const double Aq = dt * c * rho * kP * a.a_rad * S1 * iD;

  const T tg = (T)gam, tvx = (T)(vx * ic), tvy = (T)(vy * ic), tvz = (T)(vz * ic);
  const T ychiA = (T)(y * chi), ySA = (T)(y * Ssrc), iQA = (T)iQ;
  // the gas bookkeeping hands I* - I' to the gas: the energy and momentum adjoints reach
  // each angle as 4 pi W (c lamE + n.lamM) / cbar
  const double lEp = a.lamE[cell];
  const double lmp0 = a.lamM[3 * cell], lmp1 = a.lamM[3 * cell + 1], lmp2 = a.lamM[3 * cell + 2];
  const T clE = (T)(c * lEp), lm0 = (T)lmp0, lm1 = (T)lmp1, lm2 = (T)lmp2, mg = (T)a.m_gain;

  // The reverse is bound by vector issue behind the transpose of transport, at the three waves
  // per SIMD its kept values leave, so the three passes over the angles are written in what
  // survives of the forward quantities (FP32, 80 angles: 1566 -> 1276 instructions; gradient of
  // 16 steps at 96^3 x 80 in FP32 23.2 -> 22.8 ms, of 20 steps at 32^3 x 48 in FP64 1.21 ->
  // 1.18 ms; held to four waves it spills 45 registers and takes 28.5 ms).  With X = I' Gamma^4 / r
  // and R0 = r Gamma^4 I* = I' Gamma^4 - y S Gamma r:
  //   ell = dL/dI' net of the bookkeeping,  dL/dS = y sum ell r Gamma^-3,
  //   zr = r (lS1 + lSG Gamma + lSI Gamma^4 I*) = r (lS1 + lSG Gamma) + lSI R0    (dL/dWt),
  //   dL/d(1/r) = -(ell I' r + zr Wt r),
  //   dL/dGamma = -3 y S ell r Gamma^-4 + Wt (lSG r + (4 lSI R0 - 2 (zr - sum zr Wt)) / Gamma)
  //               + y chi dL/d(1/r),
  //   dL/dI* = bookkeeping + r (ell + lSI W Gamma^2 / sum W Gamma^-2),
  // where the two terms -+4 ell I' / Gamma of dL/dGamma have cancelled exactly.  R0 itself
  // cancels where a cell is optically thick, to the rounding of I' (as the forward's own r
  // scales every use of Gamma^4 I*).
  // Between the passes a lane keeps only I', ell, gamma v.n / c per direction, and 1 / Gamma
  // and r per slot; each pass rebuilds the other quantities from them.  Empty register
  // barriers on the kept values make the rebuild real: without them the compiler holds
  // every intermediate across the group sums, at the cost of a wave per SIMD.
  constexpr int H = PAIRED ? 2 : 1;  // slots per stored direction
  T gv[P], iGk[APL], rk[APL];
  auto gamma = [&](int q, int h) { return h ? tg + gv[q] : tg - gv[q]; };  // the antipode has direction -n
  auto through = [&](int q, int h, T nl) { return (T)ang.wt(q) * mg * (h ? clE - nl : clE + nl); };

  // ---- first pass: dL/dI' net of the bookkeeping, and dL/dS ------------------------------
  double lS = 0.0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    gv[q] = tg * (tvx * ang.dx(q) + tvy * ang.dy(q) + tvz * ang.dz(q));
    const T nl = ang.dx(q) * lm0 + ang.dy(q) * lm1 + ang.dz(q) * lm2;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int s = q + h * P;
      const T G = gamma(q, h);
      iGk[s] = rt_rcp(G);
      rk[s] = rt_rcp(T(1) + ychiA * G);
      // a slot past K (general layout) holds no angle: its weight is zero, and so must be
      // its adjoint, whatever the slot's row entry holds
      lam[s] = (ang.ok[s] ? lam[s] : T(0)) - through(q, h, nl);
      lS += (double)(lam[s] * rk[s] * (iGk[s] * iGk[s] * iGk[s]));
    }
  }
  lS = y * rt_group_sum<LPC>(lS);

  // ---- per cell: S -> J, T -> the root's A and C -> the sums, kappas, gas state ----------
  double lkP = lS * planck, lkJ = 0.0;
  double lplanck = lS * kP;
  const double lJc = lS * ks;
  double lSI = lJc * iD;
  lkP += lJc * y * SG * planck * iD;
  double lSG = lJc * y * kP * planck * iD;
  lplanck += lJc * y * kP * SG * iD;
  double lD = -lJc * Jc * iD;
  const double lT = lplanck * a.a_rad * T3 * (4.0 / fourpi);
  const double iFp = rt_rcp(4.0 * Aq * T3 + rcv);
  const double lA = -lT * T4 * iFp;
  const double lC = lT * iFp;
  lkP += lA * dt * c * rho * a.a_rad * S1 * iD;
  double lS1 = lA * dt * c * rho * kP * a.a_rad * iD;
  lD -= lA * Aq * iD;
  // C = rho cv T^n + dt c rho 4 pi kJ SI / D, with T^n = (E_g - |m|^2 / 2 rho) / (rho cv):
  // dL/dE_g gains lC and dL/dm gains -lC v
  lkJ += lC * dt * c * rho * fourpi * SI * iD;
  lSI += lC * dt * c * rho * fourpi * kJ * iD;
  lD -= lC * dt * c * rho * fourpi * kJ * SI * (iD * iD);
  lS1 += lD;
  lkJ += lD * y * SG;
  lSG += lD * y * kJ;
  const T lS1A = (T)lS1, lSGA = (T)lSG, lSIA = (T)lSI;

  // per slot: R0, Wt, zr and -dL/d(1/r)
  struct Bw {
    T G, R0, Wt, zr, lden;
  };
  auto bw = [&](int q, int h) {
    const int s = q + h * P;
    const T r = rk[s], iG = iGk[s];
    Bw b;
    b.G = gamma(q, h);
    const T G2 = b.G * b.G;
    b.R0 = Io[s] * (G2 * G2) - ySA * b.G * r;
    b.Wt = (T)ang.wt(q) * iQA * (iG * iG);
    b.zr = r * (lS1A + lSGA * b.G) + lSIA * b.R0;
    b.lden = lam[s] * Io[s] * r + b.zr * b.Wt * r;
    return b;
  };

  // ---- second pass: dL/dchi through r and the weights' normalisation ---------------------
#pragma unroll
  for (int q = 0; q < P; ++q) asm volatile("" : "+v"(gv[q]));
#pragma unroll
  for (int q = 0; q < APL; ++q) asm volatile("" : "+v"(iGk[q]), "+v"(rk[q]));
  double lchi = 0.0, sw = 0.0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const Bw b = bw(q, h);
      lchi += (double)(b.lden * b.G);
      sw += (double)(b.zr * b.Wt);
    }
  }
  lchi = -y * rt_group_sum<LPC>(lchi);
  sw = rt_group_sum<LPC>(sw);
  lkJ += lchi;

  // ---- third pass: Gamma through gamma and v, and dL/dI* ----------------------------------
#pragma unroll
  for (int q = 0; q < P; ++q) asm volatile("" : "+v"(gv[q]));
#pragma unroll
  for (int q = 0; q < APL; ++q) asm volatile("" : "+v"(iGk[q]), "+v"(rk[q]));
  const T swA = (T)sw, y3S = T(3) * ySA, lSI4 = T(4) * lSIA;
  double lgam = 0.0, lvx = 0.0, lvy = 0.0, lvz = 0.0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const T nl = ang.dx(q) * lm0 + ang.dy(q) * lm1 + ang.dz(q) * lm2;
    double gs = 0.0;  // sum of -+dL/dGamma over the slots
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int s = q + h * P;
      const Bw b = bw(q, h);
      const T ell = lam[s], r = rk[s], iG = iGk[s], iG2 = iG * iG;
      const T lg = b.Wt * (lSGA * r + iG * (lSI4 * b.R0 - T(2) * (b.zr - swA))) - y3S * (ell * r * (iG2 * iG2)) -
                   ychiA * b.lden;
      lam[s] = through(q, h, nl) + r * (ell + lSIA * ((T)ang.wt(q) * iQA * (b.G * b.G)));
      lgam += (double)(lg * b.G);
      gs += (double)(h == 0 ? -lg : lg);
    }
    lvx += gs * (double)ang.dx(q);
    lvy += gs * (double)ang.dy(q);
    lvz += gs * (double)ang.dz(q);
  }
  // Gamma = gamma (1 -+ v.n / c): dGamma/dgamma = Gamma / gamma, dGamma/dv = -+ gamma n / c
  const double glc = gam * ic;
  lgam = rt_group_sum<LPC>(lgam) * rt_rcp(gam);
  lvx = rt_group_sum<LPC>(lvx) * glc;
  lvy = rt_group_sum<LPC>(lvy) * glc;
  lvz = rt_group_sum<LPC>(lvz) * glc;
  const T iVp = (T)rt_rcp(Vp);
#pragma unroll
  for (int q = 0; q < APL; ++q) lam[q] *= iVp;
  if (l == 0) {
    // v = m / rho and gamma(v): dL/dm = (dL/dv + dL/dgamma gamma^3 v / c^2) / rho
    const double g3 = gam * gam * gam * (ic * ic);
    a.lamE[cell] = lEp + lC;
    a.lamM[3 * cell] = lmp0 - lC * vx + (lvx + lgam * g3 * vx) * irho;
    a.lamM[3 * cell + 1] = lmp1 - lC * vy + (lvy + lgam * g3 * vy) * irho;
    a.lamM[3 * cell + 2] = lmp2 - lC * vz + (lvz + lgam * g3 * vz) * irho;
    if (a.dkP) a.dkP[cell] += lkP;
    if (a.dkJ) a.dkJ[cell] += lkJ;
  }
}
