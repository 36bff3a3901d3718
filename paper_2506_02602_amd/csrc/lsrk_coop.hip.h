// Cooperative integration: G lanes of one wave advance one cell together.
//
// Used for the tail of a flow step -- the few stiff cells still stepping
// after the rest have finished -- where one cell per lane leaves the chip
// nearly idle and the step latency of a single lane bounds the whole call.
// Splitting one cell's right-hand side over G lanes cuts that latency.
//
// What bounds it: latency.  A wave is often alone on its SIMD, where a
// dependent FP64 operation takes 9.5 cycles (independent ones 5), a scalar
// move of a literal 8 and an LDS round trip 70-130, so the step is kept short
// in dependent operations: ln T of a stage from the step's start (log_near), the
// T-only part of k_r's exponent formed beside k_f's, thermo rows in registers,
// sums in several chains, the controller's factor from reciprocal square roots.  A lone wave's step of the 9-species mechanism
// takes 4.2 us (4.5 with the literals loaded where they are used, 5.3 without
// any of these), about 200 instructions a stage; the 1024 x 1024 front 1.69 ->
// 1.39 ms.
//
// Lane roles within a group (gl = lane index in the group, 0..G-1):
//   every lane      holds T and its stage registers (replicated: every lane
//                   computes the same dT/dt from the same sums);
//   species lane    k = gl < N: holds Y_k and its stage registers, evaluates
//                   species k's concentration and NASA-7 thermo (paper
//                   Eq. 10) and sums its production rate;
//   reaction lane   j = gl + r G < J: reaction j's forward and reverse rates
//                   and rate of progress (paper Eq. 15-16).
// Lanes without a species or reaction evaluate a clamped duplicate and
// discard it, so the rate law runs without divergent branches and the
// forward-rate exponentials overlap the thermo.  The rate law is the one of
// the unrolled per-lane RHS, read from the mechanism's generated tables.
// Values pass between lanes through the group's LDS area; every sum over
// species is taken by every lane in the same order, so all lanes of a group
// hold the same bits and the step-control decisions (paper Eq. 22) are
// uniform within the group.
#pragma once

#include <hip/hip_runtime.h>

#include "lsrk.hip.h"

namespace chemgpu {

__device__ __forceinline__ void coop_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS scratch of one group (doubles): concentrations c[N+1] (c[N] = 1, the
// pad of the species lists), g/RT g[N+1] (g[N] = 0), c_k (cp_k/R - 1) d[N],
// rates of progress q[J], per-species terms w[N] of the energy and error
// sums, and one discard slot per lane of the group: a lane without a
// species or reaction stores there instead of branching around the store.
template <class M>
struct CoopScratch {
  static constexpr int N = M::NS;
  static constexpr int SC = 0, SG = N + 1, SD = 2 * (N + 1), SQ = SD + N, SW = SQ + M::Coop::J;
  static constexpr int SX = (SW + N + 1) & ~1;  // one slot per lane for discarded stores
  static constexpr int SIZE = (SX + M::Coop::G + 1) & ~1;
};

// Groups of G lanes never straddle a wave: a wave holds floor(64 / G) of
// them and its remaining lanes (64 mod G) stay idle.
template <int G>
struct CoopWave {
  static_assert(G >= 1 && G <= 64, "a group fits in one wave");
  static constexpr int GPW = 64 / G;  // groups per wave
};

// LDS pointers keep their address space: the group's base then is one opaque
// register, and every access an offset from it.
typedef __attribute__((address_space(3))) double lds_double;

// v[0] + ... + v[N-1] in three interleaved partial sums.
template <int N>
__device__ __forceinline__ double coop_sum(const lds_double* v) {
  double p[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < N; ++k) p[k % 3] = k < 3 ? v[k] : p[k % 3] + v[k];
  return (p[0] + p[1]) + p[2];
}

template <class M>
struct CoopCtx {
  const double* D;  // the mechanism's double table, in LDS
  const double* E;  // 2^(j/64), j = 0..63 (kExp2Frac), in LDS
  const int* I;     // its int table, in LDS
  lds_double* s;    // this group's scratch
  int gl;
  NearConsts k;
};

// A lane's own table entries (its reaction, its species' production list,
// its reaction's third-body row, its species' thermo row), read into
// registers when they fit (one reaction per lane and short lists); otherwise
// read from LDS at each evaluation.  The thermo row is the one of the range
// the species' last temperature sat in: a wave reads it again when a lane
// changes range.
template <class M, int G>
struct CoopLane {
  using C = typename M::Coop;
  static constexpr int R = (C::J + G - 1) / G;
  static constexpr bool PRE = R == 1 && C::L <= 16 && M::NS <= 16;
  double lna, bexp, ear, dnu, lnpr;
  double gnu[PRE ? C::MG : 1];
  int gk[PRE ? C::MG : 1], ri[PRE ? C::MR : 1], pi[PRE ? C::MR : 1];
  int tb;
  double one, eff[PRE ? M::NS : 1];
  double slnu[PRE ? C::L : 1];
  int slj[PRE ? C::L : 1];
  double th[PRE ? C::TH_ROW : 1], tmid, invw, wmol;
  bool lo;
  const double* throw_lo;  // the species' low-range row (LDS); high: N rows further

  __device__ __forceinline__ void load_thermo(bool l) {
    if constexpr (PRE) {
      lo = l;
      const double* t = throw_lo + (l ? 0 : M::NS * C::TH_ROW);
#pragma unroll
      for (int q = 0; q < C::TH_ROW; ++q) th[q] = t[q];
    }
  }

  __device__ __forceinline__ void load(const double* D, const int* I, int gl) {
    if constexpr (PRE) {
      constexpr int N = M::NS;
      const int j = min(gl, C::J - 1);
      const int k = min(gl, N - 1);
      lna = D[C::O_LNA + j];
      bexp = D[C::O_BEXP + j];
      ear = D[C::O_EAR + j];
      dnu = D[C::O_DNU + j];
      lnpr = D[C::O_LNPR + j];
#pragma unroll
      for (int q = 0; q < C::MG; ++q) {
        gnu[q] = D[C::O_GNU + j * C::MG + q];
        gk[q] = I[C::O_GK + j * C::MG + q];
      }
#pragma unroll
      for (int q = 0; q < C::MR; ++q) {
        ri[q] = I[C::O_RI + j * C::MR + q];
        pi[q] = I[C::O_PI + j * C::MR + q];
      }
      tb = I[C::O_TB + j];
      one = D[C::O_TBONE + j];
#pragma unroll
      for (int kk = 0; kk < N; ++kk) eff[kk] = D[C::O_TBEFF + tb * N + kk];
#pragma unroll
      for (int l = 0; l < C::L; ++l) {
        slnu[l] = D[C::O_SLNU + k * C::L + l];
        slj[l] = I[C::O_SLJ + k * C::L + l];
      }
      tmid = D[C::O_TMID + k];
      invw = D[C::O_INVW + k];
      wmol = D[C::O_WK + k];
      throw_lo = D + C::O_TH + k * C::TH_ROW;
      load_thermo(false);
    }
  }
};

// f(T, Y): returns this lane's dY_k/dt (0 for lanes past N) and, on every
// lane, dT/dt in fT.  lnT: ln T (see log_near).
template <class M, int G>
__device__ __forceinline__ double coop_rhs(double Yk, double T, double lnT, double rho,
                                           double inv_rho, const CoopCtx<M>& x,
                                           CoopLane<M, G>& ln, double& fT) {
  using C = typename M::Coop;
  using S = CoopScratch<M>;
  using L = CoopLane<M, G>;
  constexpr int N = M::NS;
  constexpr int R = L::R;
  constexpr bool PRE = L::PRE;
  static_assert(N <= G, "one lane per species");
  lds_double* const s = x.s;
  const double* D = x.D;
  const int* I = x.I;
  const int gl = x.gl;
  const bool sl = gl < N;
  const int k = sl ? gl : N - 1;
  const double invT = rcp_nr(T);
  const double omlnT = 1.0 - lnT;
  // species k: concentration and thermo
  const double c = Yk * (rho * (PRE ? ln.invw : D[C::O_INVW + k]));
  const bool lo = T < (PRE ? ln.tmid : D[C::O_TMID + k]);
  if constexpr (PRE) {
    if (__any(lo != ln.lo)) ln.load_thermo(lo);
  }
  const double* th = PRE ? ln.th : D + C::O_TH + (lo ? 0 : N * C::TH_ROW) + k * C::TH_ROW;
  const double T2 = T * T;
  const double gp = fma(T2, fma(th[10], T, th[9]), fma(th[8], T, th[7]));
  const double gk = fma(th[6], omlnT, fma(th[5], invT, -th[11])) - T * gp;
  const double dk = c * fma(T2, fma(th[16], T2, fma(th[15], T, th[14])), fma(th[13], T, th[12]));
  {
    // lanes past N store into their own discard slot: no branch
    const int o = sl ? k : S::SX - S::SC + gl;
    s[S::SC + o] = c;
    s[(sl ? S::SG + k : S::SX + gl)] = gk;
    s[(sl ? S::SD + k : S::SX + gl)] = dk;
  }
  coop_sync();
  // The exchanges' latency (a wave is often alone on its SIMD) is covered by
  // what does not depend on them: the values are read right behind the
  // stores (a wave's LDS accesses stay in order) and the forward rates come
  // before their first use; likewise below.
  double gv[PRE ? C::MG : 1], cv[PRE ? 2 * C::MR : 1];
  if constexpr (PRE) {
#pragma unroll
    for (int q = 0; q < C::MG; ++q) gv[q] = s[S::SG + ln.gk[q]];
#pragma unroll
    for (int q = 0; q < C::MR; ++q) {
      cv[q] = s[S::SC + ln.ri[q]];
      cv[C::MR + q] = s[S::SC + ln.pi[q]];
    }
  }
  double kf[R], lkr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = min(gl + r * G, C::J - 1);
    const double lkf = fma(PRE ? ln.bexp : D[C::O_BEXP + j], lnT,
                           fma(PRE ? -ln.ear : -D[C::O_EAR + j], invT, PRE ? ln.lna : D[C::O_LNA + j]));
    kf[r] = exp_coop(lkf, x.E, x.k);
    lkr[r] = lkf + fma(PRE ? ln.dnu : D[C::O_DNU + j], lnT, PRE ? ln.lnpr : D[C::O_LNPR + j]);
  }
  const double hm1 = fma(T2, fma(th[4], T2, fma(th[3], T, th[2])), fma(th[1], T, th[0])) + th[5] * invT;
  // reactions: reverse rates, rates of progress
  double rden = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j0 = gl + r * G;
    const int j = min(j0, C::J - 1);
    // two chains over the reaction's net stoichiometry
    double dg0 = 0.0, dg1 = 0.0, cf, cr;
    if constexpr (PRE) {
#pragma unroll
      for (int q = 0; q < C::MG; ++q) {
        double& acc = (q & 1) ? dg1 : dg0;
        acc = fma(ln.gnu[q], gv[q], acc);
      }
      cf = cv[0];
      cr = cv[C::MR];
#pragma unroll
      for (int q = 1; q < C::MR; ++q) { cf *= cv[q]; cr *= cv[C::MR + q]; }
    } else {
#pragma unroll
      for (int q = 0; q < C::MG; ++q) {
        double& acc = (q & 1) ? dg1 : dg0;
        acc = fma(D[C::O_GNU + j * C::MG + q], s[S::SG + I[C::O_GK + j * C::MG + q]], acc);
      }
      cf = s[S::SC + I[C::O_RI + j * C::MR]];
      cr = s[S::SC + I[C::O_PI + j * C::MR]];
#pragma unroll
      for (int q = 1; q < C::MR; ++q) {
        cf *= s[S::SC + I[C::O_RI + j * C::MR + q]];
        cr *= s[S::SC + I[C::O_PI + j * C::MR + q]];
      }
    }
    const double kr = exp_coop(lkr[r] + (dg0 + dg1), x.E, x.k);
    // [M], or 1 + 0 without a third body
    const int row = PRE ? 0 : I[C::O_TB + j];
    double mt0 = PRE ? ln.one : D[C::O_TBONE + j], mt1 = 0.0;
#pragma unroll
    for (int kk = 0; kk < N; ++kk) {
      double& acc = (kk & 1) ? mt1 : mt0;
      acc = fma(PRE ? ln.eff[kk] : D[C::O_TBEFF + row * N + kk], s[S::SC + kk], acc);
    }
    const double mt = mt0 + mt1;
    // sum_k c_k (cp_k/R - 1), the same order on every lane
    if (r == 0) rden = -T * rcp_nr(coop_sum<N>(s + S::SD));
    s[j0 < C::J ? S::SQ + j : S::SX + gl] = mt * (kf[r] * cf - kr * cr);
  }
  if constexpr (PRE) asm volatile("" : "+v"(rden));
  coop_sync();
  // species k: production rate (four partial sums)
  double wk[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int l = 0; l < C::L; ++l) {
    const double v = PRE ? ln.slnu[l] : D[C::O_SLNU + k * C::L + l];
    wk[l & 3] = fma(v, s[S::SQ + (PRE ? ln.slj[l] : I[C::O_SLJ + k * C::L + l])], wk[l & 3]);
  }
  const double w = (wk[0] + wk[1]) + (wk[2] + wk[3]);
  s[sl ? S::SW + k : S::SX + gl] = hm1 * w;
  coop_sync();
  fT = rden * coop_sum<N>(s + S::SW);
  return sl ? w * ((PRE ? ln.wmol : D[C::O_WK + k]) * inv_rho) : 0.0;
}

// One step of size h (paper Eq. 21).  (uT, uk): the state at the start of
// the step (T on every lane, Y_k on species lanes); (XT, Xk) receive the new
// state.  Returns the group's squared WRMS error (the same on every lane).
template <class M, int G>
__device__ __forceinline__ double coop_step(double uT, double uk, double rho, double inv_rho,
                                            double h, double& XT, double& Xk, const Control& c,
                                            const CoopCtx<M>& x, CoopLane<M, G>& ln) {
  using S = CoopScratch<M>;
  constexpr int N = M::NS, N1 = N + 1;
  // (ready here: the compiler would form the remainder where the stages use it,
  // a lone step 4 % longer)
  LogParts ln0 = log_checked_parts<M>(uT, 1.02);
  asm volatile("" : "+v"(ln0.hi), "+v"(ln0.lo));
  const double r0 = rcp_nr(uT);
  double UT = uT, Uk = uk, ET = 0.0, Ek = 0.0;
  XT = uT;
  Xk = uk;
  auto stage = [&](int s) {
    double FT;
    const double Fk = coop_rhs<M, G>(Uk, UT, s == 0 ? ln0.hi : log_near<M>(UT, uT, ln0, r0, x.k),
                                     rho, inv_rho, x, ln, FT);
    const double bs = s == 0 ? LS_B[0] : s == 1 ? LS_B[1] : s == 2 ? LS_B[2] : s == 3 ? LS_B[3] : LS_B[4];
    const double bhs = s == 0 ? LS_BH[0] : s == 1 ? LS_BH[1] : s == 2 ? LS_BH[2] : s == 3 ? LS_BH[3] : LS_BH[4];
    const double as = s == 0 ? LS_A[0] : s == 1 ? LS_A[1] : s == 2 ? LS_A[2] : s == 3 ? LS_A[3] : 0.0;
    const double eh = (bs - bhs) * h;
    ET += eh * FT;
    Ek += eh * Fk;
    if (s < 4) {
      const double ah = as * h, bah = (bs - as) * h;
      UT = XT + ah * FT;
      XT = UT + bah * FT;
      Uk = Xk + ah * Fk;
      Xk = Uk + bah * Fk;
    } else {
      const double bh = bs * h;
      XT = XT + bh * FT;
      Xk = Xk + bh * Fk;
    }
  };
  if constexpr (CoopLane<M, G>::PRE) {
    // small mechanisms: the five stages unrolled (coefficients become
    // immediates, the loop's selects and branches go away: ~15 % fewer
    // instructions, still two waves per SIMD)
#pragma unroll
    for (int s = 0; s < 5; ++s) stage(s);
  } else {
    // large ones stay rolled: unrolled they would drop to one wave per SIMD
#pragma unroll 1
    for (int s = 0; s < 5; ++s) stage(s);
  }
  const double wT = ET * rcp_nr(c.rtol * fabs(uT) + c.atol);
  const double wk = Ek * rcp_nr(c.rtol * fabs(uk) + c.atol);
  coop_sync();
  x.s[x.gl < N ? S::SW + x.gl : S::SX + x.gl] = wk * wk;
  coop_sync();
  return fma(wT, wT, coop_sum<N>(x.s + S::SW)) * (1.0 / N1);
}

// One attempted step towards dt (same control as `advance`): returns
// CELL_RUNNING or the cell's final code.
template <class M, int G>
__device__ __forceinline__ int coop_try_step(double& uT, double& uk, double rho, double inv_rho,
                                             double dt, double& t, double& h, int& nacc,
                                             int& nrej, const Control& c, const CoopCtx<M>& x,
                                             CoopLane<M, G>& ln) {
  bool last = false;
  double hh = h;
  if (hh >= dt - t) { hh = dt - t; last = true; }
  double XT, Xk;
  const double err = coop_step<M, G>(uT, uk, rho, inv_rho, hh, XT, Xk, c, x, ln);
  const double fac = step_factor_sq(err);
  if (err <= 1.0) {
    uT = XT;
    uk = Xk;
    ++nacc;
    if (last) { h = hh * fac; return CELL_OK; }
    t = t + hh;
  } else {
    ++nrej;
  }
  h = hh * fac;
  if (nacc + nrej >= c.max_steps) return CELL_MAXSTEPS;
  if (h < 1e-14 * dt) return CELL_H_UNDERFLOW;
  return CELL_RUNNING;
}

}  // namespace chemgpu
