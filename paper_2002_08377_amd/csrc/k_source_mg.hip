// Multigroup implicit source update, and the step around it (section 2.3 with frequency groups coupled only
// through the gas temperature).  Intensities are group-major, I[g][N][K]; opacities
// kP, kJ, ks are [g][N]; group g carries the weight Wg[g] in the moments and the gas
// equation.  One cell per group of LPC lanes, each lane holding APL angles:
//  pass 1, per group: the comoving sums S1, SG, SI (the weights W~ and Gamma are the
//    same for every group), reduced over the lanes and kept in LDS; they add
//    Wg kP S1 / D and Wg kJ SI / D to the quartic's coefficients;
//  the temperature: A T^4 + B T - C = 0 in FP64, as in the grey update;
//  pass 2, per group: the row is read again and updated, I' = I r + (r / Gamma^3) y S_g
//    with S_g = kP_g a T^4/4pi + ks_g J~_g, and the radiation energy and momentum lost
//    by the stored values (weighted by Wg) go to the gas.
#include "rt_mg_rule.h"
#include "rt_step_common.h"

namespace {

template <typename T, int LPC, int APL, bool FULL, int PAIRED>
__global__ __launch_bounds__(RT_BLOCK) void k_source_mg(rt_mg_args a, int64_t nblk) {
  using Ang = rt_step_angles<T, LPC, APL, FULL, PAIRED>;
  constexpr int P = Ang::P;
  constexpr int CPB = RT_BLOCK / LPC;
  extern __shared__ __align__(16) unsigned char rt_smem[];
  double *s_grp = (double *)rt_smem;  // [CPB][G][4]: S1, SG, SI, 1/D
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  const int g = threadIdx.x / LPC;
  const int64_t cell = lb * CPB + g;
  if (cell >= a.N) return;
  const int l = threadIdx.x % LPC;
  const int K = a.K, G = a.G;
  const int64_t N = a.N;
  Ang ang;
  ang.load(a.dirs, a.W, K, l);
  double *sg = s_grp + (int64_t)g * G * 4;

  const double rho = a.rho[cell];
  const double m0 = a.mom[3 * cell], m1 = a.mom[3 * cell + 1], m2 = a.mom[3 * cell + 2];
  const double Eg = a.etot[cell];
  const double irho = rt_rcp(rho);
  const double vx = m0 * irho, vy = m1 * irho, vz = m2 * irho;
  const double ic = a.inv_c;
  const double gam = rsqrt(1.0 - (vx * vx + vy * vy + vz * vz) * (ic * ic));
  const double y = a.dt * a.c_red * rho;
  const T tg = (T)gam, tvx = (T)(vx * ic), tvy = (T)(vy * ic), tvz = (T)(vz * ic);
  // group-independent per angle: Gamma and 1/Gamma^2 (the comoving weight W / Gamma^2 is
  // formed again where it is used, which holds fewer registers than keeping it)
  T Gm[APL], iG2[APL];
  double sQ = 0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const T vn = tvx * ang.x[q] + tvy * ang.y[q] + tvz * ang.z[q];
    Gm[q] = tg * (T(1) - vn);
    if (PAIRED) Gm[q + P] = tg * (T(1) + vn);
  }
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    const T iG = rt_rcp(Gm[q]);
    iG2[q] = iG * iG;
    sQ += ang.wt(q) * (double)iG2[q];
  }
  sQ = rt_group_sum<LPC>(sQ);
  const double iQ = rt_rcp(sQ);

  // A group's row (and in the FP64 form its opacities) is loaded one group ahead in both
  // passes, so that its memory latency overlaps the previous group's arithmetic.  The FP32
  // form loads the opacities at the top of each group instead: held ahead, their registers
  // would cost a wave per SIMD (174 registers against 160; 1.82 against 1.70 ms at 128^3 x 80,
  // 4 groups), while the FP64 form is 3% faster with them ahead.
  constexpr bool KAPPA_AHEAD = sizeof(T) == 8;
  struct grp {
    T I[APL];
    double kJ, ks, kP;
  };
  auto fetch = [&](int j, grp &o) {
    const int64_t gc = (int64_t)j * N + cell;
    const T *Ir = (const T *)a.I + gc * K;
#pragma unroll
    for (int q = 0; q < APL; ++q) o.I[q] = Ir[ang.k[q]];
    if constexpr (KAPPA_AHEAD) {
      o.kJ = a.kJ[gc];
      o.ks = a.ks[gc];
      o.kP = a.kP[gc];
    }
  };
  auto kappa = [&](int j, const grp &g, double &kJ, double &ks, double &kP) {
    if constexpr (KAPPA_AHEAD) {
      kJ = g.kJ;
      ks = g.ks;
      kP = g.kP;
    } else {
      const int64_t gc = (int64_t)j * N + cell;
      kJ = a.kJ[gc];
      ks = a.ks[gc];
      kP = a.kP[gc];
    }
  };

  // pass 1: per-group comoving sums and the quartic's coefficients
  double Asum = 0, Csum = 0;
  grp cur, nxt;
  fetch(0, cur);
  nxt = cur;  // defined when the last group rotates it in
  for (int j = 0; j < G; ++j) {
    if (j + 1 < G) fetch(j + 1, nxt);
    double kJ, ks, kP;
    kappa(j, cur, kJ, ks, kP);
    const T tyc = (T)(y * (kJ + ks));
    double s1 = 0, sG = 0, sI = 0;
#pragma unroll
    for (int q = 0; q < APL; ++q) {
      const T I = cur.I[q];
      const T r = rt_rcp(T(1) + tyc * Gm[q]);
      const T G2 = Gm[q] * Gm[q];
      const double qk = ang.wt(q) * (double)iG2[q];
      s1 += qk * (double)r;
      sG += qk * (double)(Gm[q] * r);
      sI += qk * (double)(G2 * G2 * I * r);
    }
    s1 = rt_group_sum<LPC>(s1) * iQ;
    sG = rt_group_sum<LPC>(sG) * iQ;
    sI = rt_group_sum<LPC>(sI) * iQ;
    const double iD = rt_rcp(s1 + y * kJ * sG);
    Asum += a.Wg[j] * kP * s1 * iD;
    Csum += a.Wg[j] * kJ * sI * iD;
    if (l == 0) {
      sg[4 * j] = s1;
      sg[4 * j + 1] = sG;
      sg[4 * j + 2] = sI;
      sg[4 * j + 3] = iD;
    }
    cur = nxt;
  }
  const double rcv = rho * a.cv;
  const double Tn = (Eg - 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) * irho) * rt_rcp(rcv);
  const double fourpi = 4.0 * RT_PI;
  const double Aq = a.dt * a.c_light * rho * a.a_rad * Asum;
  const double Cq = rcv * Tn + a.dt * a.c_light * rho * fourpi * Csum;
  const double Tnew = rt_quartic_root_from(Aq, rcv, Cq, Tn);
  const double T4 = Tnew * Tnew * Tnew * Tnew;
  const double planck = a.a_4pi * T4;
  // lane 0's LDS writes are read by the group's other lanes (same wave): release them to the
  // wave, meet, then acquire
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // pass 2: per group, update the row and book the energy and momentum handed over
  double dE = 0, dFx = 0, dFy = 0, dFz = 0;
  fetch(0, cur);
  nxt = cur;
  for (int j = 0; j < G; ++j) {
    // the next group's row is another array than this group's, so reading it ahead of
    // this group's stores is safe
    if (j + 1 < G) fetch(j + 1, nxt);
    T *Ir = (T *)a.I + ((int64_t)j * N + cell) * K;
    double kJ, ks, kP;
    kappa(j, cur, kJ, ks, kP);
    const T tyc = (T)(y * (kJ + ks));
    const double Jc = (sg[4 * j + 2] + y * kP * sg[4 * j + 1] * planck) * sg[4 * j + 3];
    const T ySrc = (T)(y * (kP * planck + ks * Jc));
    const double wg = a.Wg[j];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      auto upd = [&](int qq) -> double {
        const T I0 = cur.I[qq];
        const T r = rt_rcp(T(1) + tyc * Gm[qq]);
        const T out = I0 * r + r * iG2[qq] * rt_rcp(Gm[qq]) * ySrc;
        if (ang.ok[qq]) Ir[ang.k[qq]] = out;
        return wg * ang.wt(qq) * ((double)I0 - (double)out);
      };
      double wd = upd(q);
      dE += wd;
      if (PAIRED) {
        const double wd2 = upd(q + P);
        dE += wd2;
        wd -= wd2;  // the antipode's direction is -n
      }
      dFx += wd * (double)ang.x[q];
      dFy += wd * (double)ang.y[q];
      dFz += wd * (double)ang.z[q];
    }
    cur = nxt;
  }
  dE = rt_group_sum<LPC>(dE);
  dFx = rt_group_sum<LPC>(dFx);
  dFy = rt_group_sum<LPC>(dFy);
  dFz = rt_group_sum<LPC>(dFz);
  if (l == 0) {
    a.etot[cell] = Eg + a.e_gain * dE;
    a.mom[3 * cell] = m0 + a.m_gain * dFx;
    a.mom[3 * cell + 1] = m1 + a.m_gain * dFy;
    a.mom[3 * cell + 2] = m2 + a.m_gain * dFz;
    if (a.T_out) a.T_out[cell] = Tnew;
  }
}

// The whole multigroup step in one kernel: every group's upwind transport, then the source.
// As one transport launch per group and the source kernel behind them, a step at 64^3 x 80 with
// 4 groups in FP32 spent 0.21 of 0.80 ms reading the transported rows twice and writing them a
// second time, and each transport staged the face records and formed the face speeds again.
// Here JG groups share a sweep over the faces (their speeds, records and upwind tests are the
// same), each group's transported row is summed on the spot, and the rows wait for the
// temperature where the lane left them: the last sweep's in registers, the others in LDS, in
// words of the lane's own (no other lane reads them).  A call, its state reset included: 0.80 ->
// 0.59 ms (FP32); FP64 at 48^3 x 80 0.53 -> 0.38, 12^3 x 24 43 -> 27 us.  Bound now by the gathers and the vector
// issue of the faces, at three waves per SIMD (FP32; held to four it spills and takes 0.69 ms).
// groups whose rows wait in LDS: all but the last sweep's two (a lone group's waits there)
__host__ __device__ constexpr int rt_mg_rows(int G) { return G > 2 ? G - 2 : G == 1 ? 1 : 0; }

template <typename T, int LPC, int APL, bool FULL, int PAIRED>
__global__ __launch_bounds__(RT_BLOCK) void k_step_mg(rt_step_args a, rt_mg_args m, int64_t nblk, bool past_caches) {
  using Ang = rt_step_angles<T, LPC, APL, FULL, PAIRED, true>;
  using V4 = typename rt_vec4<T>::type;
  constexpr int P = Ang::P;
  constexpr int CPB = RT_BLOCK / LPC;
  constexpr int JG = 2;
  constexpr bool NT = FULL && LPC * APL * sizeof(T) % 64 == 0;  // rows of whole lines
  extern __shared__ __align__(16) unsigned char rt_smem[];
  const int G = m.G;
  V4 *s_an = (V4 *)rt_smem;
  double *s_grp = (double *)(s_an + a.hf_cap);  // [CPB][G][3]: what the update needs of a group
  T *s_rows = (T *)(s_grp + CPB * G * 3);       // [rt_mg_rows][APL][RT_BLOCK]: a lane's transported values
  int32_t *s_nbr = (int32_t *)(s_rows + rt_mg_rows(G) * APL * RT_BLOCK);
  const int64_t lb = rt_logical_block(nblk);
  if (lb < 0) return;
  const int64_t c0 = lb * CPB;
  const int64_t c1 = c0 + CPB < a.N ? c0 + CPB : a.N;
  const int g = threadIdx.x / LPC;
  const bool live = c0 + g < a.N;
  const int64_t cell = live ? c0 + a.wg_order[c0 + g] : c0;
  const int l = threadIdx.x % LPC;
  const int H0 = a.row_ptr[c0];
  {
    const V4 *an = (const V4 *)a.hf_an;
    const int nH = a.row_ptr[c1] - H0;  // <= hf_cap by construction
    for (int i = threadIdx.x; i < nH; i += RT_BLOCK) {
      s_nbr[i] = a.hf_nbr[H0 + i];
      s_an[i] = an[H0 + i];
    }
  }
  __syncthreads();
  if (!live) return;
  Ang ang;
  ang.load(a.dirs, a.W, a.K, l);
  const int k_single = Ang::SINGLE ? ang.k[P - 1] : ang.k[0];
  const int64_t slab = a.N * (int64_t)a.K;
  double *sg = s_grp + g * G * 3;
  T *rows = s_rows + threadIdx.x;

  const double Vn = a.vol_in[cell];
  const double dV = a.dt * a.D[cell];
  const double Vnew = rt_vol_next(Vn, a.dt, a.D[cell]);
  const double iV = rt_rcp(Vnew);
  const T cr = (T)(1.0 - dV * iV), ci = (T)iV;  // as in the single-group step
  const int h0 = a.row_ptr[cell] - H0, nh = a.row_ptr[cell + 1] - H0 - h0;

  const double rho = m.rho[cell];
  const double m0 = m.mom[3 * cell], m1 = m.mom[3 * cell + 1], m2 = m.mom[3 * cell + 2];
  const double irho = rt_rcp(rho);
  const double vx = m0 * irho, vy = m1 * irho, vz = m2 * irho;
  const double ic = m.inv_c;
  const double gam = rsqrt(1.0 - (vx * vx + vy * vy + vz * vz) * (ic * ic));
  const double y = m.dt * m.c_red * rho;
  const T tg = (T)gam, tvx = (T)(vx * ic), tvy = (T)(vy * ic), tvz = (T)(vz * ic);
  T vn[P];  // Gamma = tg (1 -+ vn)
#pragma unroll
  for (int q = 0; q < P; ++q) vn[q] = tvx * ang.x[q] + tvy * ang.y[q] + tvz * ang.z[q];
  auto gamma = [&](int q) { return q < P ? tg * (T(1) - vn[q]) : tg * (T(1) + vn[q % P]); };

  double sQ = 0;
#pragma unroll
  for (int q = 0; q < APL; ++q) {
    const T iG = rt_rcp(gamma(q));
    sQ += ang.wt(q) * (double)(iG * iG);
  }
  const double iQ = rt_rcp(rt_group_sum<LPC>(sQ));

  // one group's comoving sums, kept for the update, and its part of the quartic's coefficients
  double Asum = 0, Csum = 0;
  struct kappas {
    double J, s, P;
  };
  auto kappa = [&](int j) {
    const int64_t gc = (int64_t)j * a.N + cell;
    return kappas{m.kJ[gc], m.ks[gc], m.kP[gc]};
  };
  auto sums = [&](int j, const kappas &k, const T (&I)[APL]) {
    const double kJ = k.J, ks = k.s, kP = k.P;
    const T tyc = (T)(y * (kJ + ks));
#pragma unroll
    for (int q = 0; q < P; ++q) asm volatile("" : "+v"(vn[q]));  // formed again for each group, not held
    double s1 = 0, sG = 0, sI = 0;
#pragma unroll
    for (int q = 0; q < APL; ++q) {
      const T Gm = gamma(q);
      const T iG = rt_rcp(Gm);
      const T r = rt_rcp(T(1) + tyc * Gm);
      const T G2 = Gm * Gm;
      const double qk = ang.wt(q) * (double)(iG * iG);
      s1 += qk * (double)r;
      sG += qk * (double)(Gm * r);
      sI += qk * (double)(G2 * G2 * I[q] * r);
    }
    s1 = rt_group_sum<LPC>(s1) * iQ;
    sG = rt_group_sum<LPC>(sG) * iQ;
    sI = rt_group_sum<LPC>(sI) * iQ;
    const double iD = rt_rcp(s1 + y * kJ * sG);
    Asum += m.Wg[j] * kP * s1 * iD;
    Csum += m.Wg[j] * kJ * sI * iD;
    if (l == 0) {
      // y S = y (kP a T^4 / 4 pi + ks J~), J~ = (SI + y kP SG a T^4 / 4 pi) / D
      sg[3 * j] = y * (kJ + ks);
      sg[3 * j + 1] = y * kP * (1.0 + y * ks * sG * iD);
      sg[3 * j + 2] = y * ks * sI * iD;
    }
  };

  const T *Iin = (const T *)a.I_in;
  const int32_t *nbr = s_nbr + h0;
  const V4 *an = s_an + h0;
  int j = 0;
  if (G % JG) {  // (JG = 2) an odd group first, so that the last sweep is a full one
    T I[1][APL];
    const kappas k = kappa(0);
    rt_upwind_sweep<T, LPC, APL, 1>(a, ang, slab, cell, Iin, k_single, nbr, an, nh, cr, ci, I);
    sums(0, k, I[0]);
#pragma unroll
    for (int q = 0; q < APL; ++q) rows[q * RT_BLOCK] = I[0][q];
    j = 1;
  }
  T last[JG][APL];
  for (; j < G; j += JG) {
    kappas k[JG];  // behind the sweep their latency would show: 0.63 against 0.61 ms (64^3 x 80, 4 groups)
#pragma unroll
    for (int i = 0; i < JG; ++i) k[i] = kappa(j + i);
    rt_upwind_sweep<T, LPC, APL, JG>(a, ang, slab, cell, Iin + j * slab, k_single, nbr, an, nh, cr, ci, last);
#pragma unroll
    for (int i = 0; i < JG; ++i) sums(j + i, k[i], last[i]);
    if (j + JG < G) {
#pragma unroll
      for (int i = 0; i < JG; ++i)
#pragma unroll
        for (int q = 0; q < APL; ++q) rows[((j + i) * APL + q) * RT_BLOCK] = last[i][q];
    }
  }
  if (l == 0) a.vol_out[cell] = Vnew;

  const double Eg = m.etot[cell];
  const double rcv = rho * m.cv;
  const double Tn = (Eg - 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) * irho) * rt_rcp(rcv);
  const double fourpi = 4.0 * RT_PI;
  const double Aq = m.dt * m.c_light * rho * m.a_rad * Asum;
  const double Cq = rcv * Tn + m.dt * m.c_light * rho * fourpi * Csum;
  const double Tnew = rt_quartic_root_from(Aq, rcv, Cq, Tn);
  const double T4 = Tnew * Tnew * Tnew * Tnew;
  const double planck = m.a_4pi * T4;
  // lane 0's LDS writes are read by the group's other lanes (same wave): release them to the
  // wave, meet, then acquire
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  double dE = 0, dFx = 0, dFy = 0, dFz = 0;
  auto update = [&](int jj, T (&I)[APL]) {
    const T tyc = (T)sg[3 * jj];
    const T ySrc = (T)(sg[3 * jj + 1] * planck + sg[3 * jj + 2]);
    const double wg = m.Wg[jj];
#pragma unroll
    for (int q = 0; q < P; ++q) asm volatile("" : "+v"(vn[q]));
#pragma unroll
    for (int q = 0; q < P; ++q) {
      auto upd = [&](int qq) -> double {
        const T Gm = gamma(qq);
        const T iG = rt_rcp(Gm);
        const T r = rt_rcp(T(1) + tyc * Gm);
        const T out = I[qq] * r + r * (iG * iG) * iG * ySrc;
        const double wd = wg * ang.wt(qq) * ((double)I[qq] - (double)out);
        I[qq] = out;
        return wd;
      };
      double wd = upd(q);
      dE += wd;
      if (PAIRED) {
        const double wd2 = upd(q + P);
        dE += wd2;
        wd -= wd2;  // the antipode's direction is -n
      }
      dFx += wd * (double)ang.x[q];
      dFy += wd * (double)ang.y[q];
      dFz += wd * (double)ang.z[q];
    }
    T *o = (T *)a.I_out + jj * slab + cell * a.K;
    if (NT && past_caches) ang.template write_lane<true>(o + ang.k[0], o + k_single, I);
    else ang.write_lane(o + ang.k[0], o + k_single, I);
  };
  if (G >= JG) {
#pragma unroll
    for (int i = 0; i < JG; ++i) update(G - JG + i, last[i]);
  }
  for (int jj = 0; jj < (G < JG ? G : G - JG); ++jj) {
    T I[APL];
#pragma unroll
    for (int q = 0; q < APL; ++q) I[q] = rows[(jj * APL + q) * RT_BLOCK];
    update(jj, I);
  }
  dE = rt_group_sum<LPC>(dE);
  dFx = rt_group_sum<LPC>(dFx);
  dFy = rt_group_sum<LPC>(dFy);
  dFz = rt_group_sum<LPC>(dFz);
  if (l == 0) {
    m.etot[cell] = Eg + m.e_gain * dE;
    m.mom[3 * cell] = m0 + m.m_gain * dFx;
    m.mom[3 * cell + 1] = m1 + m.m_gain * dFy;
    m.mom[3 * cell + 2] = m2 + m.m_gain * dFz;
    if (m.T_out) m.T_out[cell] = Tnew;
  }
}

// Both kernels go through one list of layouts: OP is the launch to make in the layout chosen.
struct rt_source_only {
  rt_mg_args a;
  int K() const { return a.K; }
  int paired() const { return a.paired; }
  template <typename T, int LPC, int APL, bool FULL, int PAIRED> hipError_t run(hipStream_t s) const {
    const int64_t cpb = RT_BLOCK / LPC;
    const int64_t nblk = (a.N + cpb - 1) / cpb;
    const size_t smem = sizeof(double) * 4 * (size_t)a.G * cpb;
    if (smem > 65536) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_source_mg<T, LPC, APL, FULL, PAIRED>), dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK),
                       smem, s, a, nblk);
    return hipGetLastError();
  }
};

// hipErrorInvalidConfiguration: the paired layout does not fit and the general one is tried, or
// that does not either (or is the slower one, rt_mg_rule.h) and the step takes its separate launches.
struct rt_whole_step {
  rt_step_args a;
  rt_mg_args m;
  int K() const { return a.K; }
  int paired() const { return a.paired; }
  template <typename T, int LPC, int APL, bool FULL, int PAIRED> hipError_t run(hipStream_t s) const {
    constexpr int64_t cpb = RT_BLOCK / LPC;
    rt_step_args b = a;
    b.hf_cap = LPC == 16 ? a.hf_cap16 : LPC == 8 ? a.hf_cap32 : a.hf_cap64;
    b.wg_order = LPC == 16 ? a.wg_order16 : LPC == 8 ? a.wg_order32 : a.wg_order64;
    const size_t rows = rt_mg_rows(m.G);
    const size_t smem = (sizeof(typename rt_vec4<T>::type) + sizeof(int32_t)) * (size_t)b.hf_cap +
                        sizeof(double) * 3 * (size_t)m.G * cpb + sizeof(T) * APL * RT_BLOCK * rows;
    // Two workgroups per CU at least.  One (FP32, 16 groups, 40^3 x 80) took 1.30 ms where the
    // separate launches take 0.83; two are still ahead of them (FP64, 4 groups, 48^3 x 80: 0.40
    // against 0.53 ms; FP32, 8 groups: 0.52 against 0.70).
    if (smem > (size_t)a.lds_max / 2) return hipErrorInvalidConfiguration;
    // a set that has a paired layout, whose rows did not fit in it
    if (!PAIRED && a.paired && rt_paired_lanes(a.K) &&
        !rt_mg_general_step(LPC, APL, sizeof(T), a.N, smem, (size_t)a.lds_max))
      return hipErrorInvalidConfiguration;
    // An output that outgrows the Infinity Cache is stored past the caches, to leave them to the
    // gathered rows (kernel alone, 335 MB: 0.615 -> 0.602 ms; 8 groups, 283 MB: 0.553 -> 0.515).
    const bool past_caches = (int64_t)sizeof(T) * m.G * a.N * a.K > (int64_t)128 << 20;
    const int64_t nblk = (a.N + cpb - 1) / cpb;
    hipLaunchKernelGGL((k_step_mg<T, LPC, APL, FULL, PAIRED>), dim3((unsigned)rt_grid_for(nblk)), dim3(RT_BLOCK),
                       smem, s, b, m, nblk, past_caches);
    return hipGetLastError();
  }
};

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

hipError_t rt_launch_source_mg(const rt_mg_args &a, int dtype, hipStream_t s) {
  const rt_source_only op{a};
  return dtype == RT_F32 ? dispatch<float>(op, s) : dispatch<double>(op, s);
}

hipError_t rt_launch_step_mg(const rt_step_args &a, const rt_mg_args &m, int dtype, hipStream_t s) {
  const rt_whole_step op{a, m};
  return dtype == RT_F32 ? dispatch<float>(op, s) : dispatch<double>(op, s);
}
