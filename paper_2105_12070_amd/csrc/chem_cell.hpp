// Device solver for one cell per wavefront (N <= NP <= 64).
//
// Layout: lane i owns component i of every state-sized vector (lane 0 = T,
// lane 1+k = Y_k) and row i of the iteration matrix M = I/(gamma h) - J, held
// in NP registers.  Reaction-level work runs one reaction per lane in rounds
// of 64; species-level work runs one species per lane.  The Jacobian is
// assembled in the wave's LDS workspace, rows owned by lanes, so its
// accumulation is deterministic.
#pragma once
#include "chem_common.hpp"

namespace chem {

struct MechView {
  MechDims d;
  const double* lnA;      // LDS
  const double* b;        // LDS
  const double* th;       // LDS
  const uint64_t* sp;     // LDS: reactant slots in bytes 0..2, products 3..5, n_reac byte 6, n_prod byte 7
  const double* W;        // LDS
  const double* iW;       // LDS
  const int32_t* cptr;    // LDS [K+1]
  const uint32_t* cent;   // LDS [L] (r << 8) | (uint8)nu
  const int32_t* tbp;     // LDS [R - R0 + 1]
  const int32_t* tbs;     // LDS third-body species
  const double* tbd;      // LDS efficiency - 1
  const double* troe;     // LDS [R - R1][8]
  const double* nasa;     // global [K][16]
  const uint32_t* jsched; // global [jit][64] species-scatter schedule: (r << 16) | (k << 8) | (uint8)nu
  int jit;
};

__device__ inline MechView make_view(const uint8_t* lds, const IntArgs& a) {
  MechView m;
  m.d = a.d;
  m.lnA = (const double*)(lds + a.d.o_lnA);
  m.b = (const double*)(lds + a.d.o_b);
  m.th = (const double*)(lds + a.d.o_th);
  m.sp = (const uint64_t*)(lds + a.d.o_sp);
  m.W = (const double*)(lds + a.d.o_W);
  m.iW = (const double*)(lds + a.d.o_iW);
  m.cptr = (const int32_t*)(lds + a.d.o_cptr);
  m.cent = (const uint32_t*)(lds + a.d.o_cent);
  m.tbp = (const int32_t*)(lds + a.d.o_tbp);
  m.tbs = (const int32_t*)(lds + a.d.o_tbs);
  m.tbd = (const double*)(lds + a.d.o_tbd);
  m.troe = (const double*)(lds + a.d.o_troe);
  m.nasa = a.nasa;
  m.jsched = a.jsched;
  m.jit = a.jsched_it;
  return m;
}

// Per-wave LDS workspace.
struct CellWs {
  double* J;    // [N][S]
  double* rk;   // [R] q (RHS) or k_eff (Jacobian)
  double* rkr;  // [R] k_eff / K_c
  double* rdm;  // [R - R0] d q / d[M] of the third-body and falloff reactions
  double* rdt;  // [R] d q / dT at fixed C
  double* C;    // [64+1] concentrations, C[K] = 1 (padding species)
  double* g;    // [64+1] g/RT (reused for mass enthalpy in the Jacobian pass)
  double* hR;   // [64+1] h/RT
  double* lu;   // [256] scratch of the LU (overlays rk .. rdm)
};

// Everything of a wave's workspace but the Jacobian block.
__host__ __device__ inline int wave_rates_doubles(int R, int R0) {
  const int rates = 3 * R + (R - R0 + 1);
  return (rates > 256 ? rates : 256) + 3 * 66;  // the LU's scratch overlays the rates
}
// S = NP + 1, so reads of static columns j < NP + 1 from any row stay inside
// the J block (its last row is followed by the reaction arrays).
__host__ __device__ inline int cell_ws_doubles(int N, int S, int R, int R0) { return N * S + wave_rates_doubles(R, R0); }

// Workspace after base; with_J = false leaves J to be set from a slot.
__device__ inline CellWs make_ws(double* base, const MechDims& d, bool with_J = true) {
  CellWs w;
  w.J = with_J ? base : nullptr;
  w.rk = with_J ? base + d.N * d.S : base;
  w.rkr = w.rk + d.R;
  w.rdt = w.rkr + d.R;
  w.rdm = w.rdt + d.R;
  w.lu = w.rk;
  w.C = w.rk + (wave_rates_doubles(d.R, d.R0) - 3 * 66);
  w.g = w.C + 66;
  w.hR = w.g + 66;
  return w;
}

// Jacobian slots shared by the waves of a workgroup: a wave holds one from
// the start of the Jacobian's species pass until M is formed in registers, so
// a workgroup can run more cells than it has Jacobian blocks.  flags[s] is 0
// when slot s is free.  Acquisition is bounded: after `limit` sleeping polls a
// wave gives up (the caller marks its cell failed), so no wave can wait
// forever.
struct SlotPool {
  int* flags;
  double* base;
  int nslots;
  int slot_doubles;
  __device__ double* slot(int s) const { return base + (size_t)s * slot_doubles; }
  __device__ int acquire(unsigned limit) const {
    int got = -1;
    for (unsigned spin = 0; spin < limit; ++spin) {
      int v = -1;
      if (lane_id() == 0) {
        for (int s = 0; s < nslots; ++s) {
          int expected = 0;
          if (__hip_atomic_compare_exchange_strong(&flags[s], &expected, 1, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP)) {
            v = s;
            break;
          }
        }
      }
      got = __builtin_amdgcn_readlane(v, 0);
      if (got >= 0) break;
      __builtin_amdgcn_s_sleep(4);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return got;
  }
  __device__ void release(int s) const {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (lane_id() == 0) __hip_atomic_store(&flags[s], 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};

// Uniform mixture quantities of one evaluation point.
struct Mix {
  double T, lnT, iT, rho, iRho, Wbar, cp, Ctot, lnPRT;
};

// Per-phase cycle counters of one wave (compiled in only when PROF is true):
// 0 Jacobian pass (with f(y_n)), 1 forming M, 2 LU, 3 stage f evaluations,
// 4 triangular solves, 5 everything, 6 and 7 the reaction and species parts
// of the Jacobian pass.
template <bool PROF>
struct Prof {
  unsigned long long c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned long long t = 0;
  __device__ __forceinline__ void start() {
    if (PROF) t = __builtin_readcyclecounter();
  }
  __device__ __forceinline__ void add(int i, unsigned long long since) {
    if (PROF) c[i] += __builtin_readcyclecounter() - since;
  }
  __device__ __forceinline__ unsigned long long now() const { return PROF ? __builtin_readcyclecounter() : 0ull; }
  __device__ __forceinline__ void stop(int i) {
    if (PROF) {
      const unsigned long long n = __builtin_readcyclecounter();
      c[i] += n - t;
      t = n;
    }
  }
};

// Lane-local species thermo: NASA-7 cp/R, h/RT, s/R and d(cp/R)/dT.
struct SpThermo {
  double cpR, hRT, sR, dcpR;
};

__device__ inline SpThermo nasa7(const double* row, double T, double lnT, double iT) {
  // both ranges are loaded before T is known, so the loads overlap the log
  double lo[7], hi[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    lo[i] = row[1 + i];
    hi[i] = row[8 + i];
  }
  const bool high = T > row[0];
  double a[7];
#pragma unroll
  for (int i = 0; i < 7; ++i) a[i] = high ? hi[i] : lo[i];
  SpThermo t;
  t.cpR = a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4])));
  t.hRT = a[0] + T * (a[1] * 0.5 + T * (a[2] * (1.0 / 3.0) + T * (a[3] * 0.25 + T * a[4] * 0.2))) + a[5] * iT;
  t.sR = a[0] * lnT + T * (a[1] + T * (a[2] * 0.5 + T * (a[3] * (1.0 / 3.0) + T * a[4] * 0.25))) + a[6];
  t.dcpR = a[1] + T * (2.0 * a[2] + T * (3.0 * a[3] + T * 4.0 * a[4]));
  return t;
}

// Species phase shared by f and J: thermo at T, mixture density, and the
// concentrations / g/RT / h/RT the reaction lanes gather.  Returns the lane's
// species thermo (garbage on non-species lanes).
__device__ inline SpThermo species_phase(const MechView& m, const CellWs& w, double y, double p, int lane,
                                         Mix& x, double& Yk) {
  const int K = m.d.K;
  const bool isSp = lane >= 1 && lane <= K;
  const int k = isSp ? lane - 1 : 0;
  x.T = readlane(y, 0);
  x.lnT = log(x.T);
  x.iT = 1.0 / x.T;
  SpThermo t = nasa7(m.nasa + 16 * k, x.T, x.lnT, x.iT);
  Yk = isSp ? y : 0.0;
  const double iWk = m.iW[k];
  const double yw = Yk * iWk;
  const double sy = wave_sum(yw);
  x.Wbar = 1.0 / sy;
  x.rho = p * x.Wbar * x.iT / RU;
  x.iRho = 1.0 / x.rho;
  x.Ctot = p * x.iT / RU;
  x.lnPRT = log(PATM * x.iT / RU);
  x.cp = wave_sum(isSp ? Yk * t.cpR * RU * iWk : 0.0);
  if (isSp) {
    w.C[k] = x.rho * yw;
    w.g[k] = t.hRT - t.sR;
    w.hR[k] = t.hRT;
  }
  wsync();
  return t;
}

// One reaction's slot data from the packed word.
struct Slots {
  int r0, r1, r2, p0, p1, p2, dnu;
};
__device__ __forceinline__ Slots unpack(uint64_t s) {
  Slots o;
  o.r0 = (int)(s & 0xFF);
  o.r1 = (int)((s >> 8) & 0xFF);
  o.r2 = (int)((s >> 16) & 0xFF);
  o.p0 = (int)((s >> 24) & 0xFF);
  o.p1 = (int)((s >> 32) & 0xFF);
  o.p2 = (int)((s >> 40) & 0xFF);
  o.dnu = (int)((s >> 56) & 0xFF) - (int)((s >> 48) & 0xFF);
  return o;
}

__device__ __forceinline__ double third_body(const MechView& m, const CellWs& w, int r, double Ctot) {
  double M = Ctot;
  const int e1 = m.tbp[r - m.d.R0 + 1];
#pragma clang loop unroll(disable)
  for (int e = m.tbp[r - m.d.R0]; e < e1; ++e) M += m.tbd[e] * w.C[m.tbs[e]];
  return M;
}

// Troe falloff: k = kinf Pr/(1+Pr) F, Pr = k0 [M]/kinf.  Returns k and, when
// Deriv, d k / d[M] / net-factor pieces and d ln k / dT.
template <bool Deriv>
__device__ __forceinline__ double troe_k(const MechView& m, int r, const Mix& x, double kf, double dlnkf, double M,
                                         double& dk_dM, double& dlnk_dT) {
  const double* t = m.troe + TROE_STRIDE * (r - m.d.R1);
  const double alpha = t[0], iT3 = t[1], iT1 = t[2], T2 = t[3];
  const double k0 = exp(t[4] + t[5] * x.lnT - t[6] * x.iT);
  const double Pr = k0 * M / kf;
  const double e3 = exp(-x.T * iT3), e1 = exp(-x.T * iT1), e2 = exp(-T2 * x.iT);
  const double Fc = (1.0 - alpha) * e3 + alpha * e1 + e2;
  const double xF = log10(Fc);
  const double L = log10(Pr);
  const double c = -0.4 - 0.67 * xF;
  const double n = 0.75 - 1.27 * xF;
  const double d = n - 0.14 * (L + c);
  const double f1 = (L + c) / d;
  const double den = 1.0 + f1 * f1;
  const double F = exp10(xF / den);
  const double ipr = 1.0 / (1.0 + Pr);
  const double k = k0 * M * ipr * F;
  if (Deriv) {
    const double id2 = 1.0 / (d * d);
    const double dlgF_dL = -xF * 2.0 * f1 / (den * den) * n * id2;
    const double dlgF_dx = 1.0 / den - xF * 2.0 * f1 / (den * den) * (-0.67 * d + 1.1762 * (L + c)) * id2;
    const double gg = ipr + dlgF_dL;
    dk_dM = k0 * F * ipr * gg;
    const double dFc = -(1.0 - alpha) * iT3 * e3 - alpha * iT1 * e1 + T2 * x.iT * x.iT * e2;
    const double dlnk0 = t[5] * x.iT + t[6] * x.iT * x.iT;
    dlnk_dT = dlnkf + gg * (dlnk0 - dlnkf) + dlgF_dx * dFc / Fc;
  }
  return k;
}

// f(Phi) for the wave's cell: lane i gets f_i.
__device__ inline double rhs(const MechView& m, const CellWs& w, double y, double p, int lane) {
  const int K = m.d.K, R = m.d.R;
  Mix x;
  double Yk;
  SpThermo t = species_phase(m, w, y, p, lane, x, Yk);
#pragma clang loop unroll(disable)
  for (int r = lane; r < R; r += WAVE) {
    const Slots s = unpack(m.sp[r]);
    const double lnkf = m.lnA[r] + m.b[r] * x.lnT - m.th[r] * x.iT;
    const double Rf = w.C[s.r0] * w.C[s.r1] * w.C[s.r2];
    const double Rr = w.C[s.p0] * w.C[s.p1] * w.C[s.p2];
    const double sng = w.g[s.p0] + w.g[s.p1] + w.g[s.p2] - w.g[s.r0] - w.g[s.r1] - w.g[s.r2];
    const double kf = exp(lnkf);
    const double iKc = exp(sng - s.dnu * x.lnPRT);  // 1/K_c
    double q = kf * (Rf - iKc * Rr);
    if (r >= m.d.R0) {
      const double M = third_body(m, w, r, x.Ctot);
      if (r < m.d.R1) {
        q *= M;
      } else {
        double dk, dl;
        q = troe_k<false>(m, r, x, kf, 0.0, M, dk, dl) * (Rf - iKc * Rr);
      }
    }
    w.rk[r] = q;
  }
  // omega_k = sum_r nu_kr q_r on the balanced species schedule of the
  // Jacobian pass (every lane takes about L/64 entries), accumulated with LDS
  // atomics in w.hR, which f does not read (the next thermo pass rewrites it)
  const bool isSp = lane >= 1 && lane <= K;
  if (isSp) w.hR[lane - 1] = 0.0;
  wsync();
  {
    const uint32_t* js = m.jsched + lane;
    uint32_t ent = js[0];
#pragma clang loop unroll(disable)
    for (int it = 0; it < m.jit; ++it) {
      const uint32_t cur = ent;
      if (it + 1 < m.jit) ent = js[(it + 1) * WAVE];
      if (cur != ~0u) atomicAdd(w.hR + ((cur >> 8) & 0xFF), (double)(int8_t)(cur & 0xFF) * w.rk[cur >> 16]);
    }
  }
  lds_wait();
  wsync();
  const double om = isSp ? w.hR[lane - 1] : 0.0;
  const double Q = wave_sum(isSp ? t.hRT * om : 0.0);
  const double fT = -RU * x.T * Q * x.iRho / x.cp;
  wsync();
  if (lane == 0) return fT;
  return isSp ? m.W[lane - 1] * om * x.iRho : 0.0;
}

// Analytic Jacobian (section 2.3) into w.J and f(Phi) into the return value.
//   J_kj = (W_k/W_j) dw_k/dC_j + W_k Wbar/(rho W_j) (w_k - s_k),  s_k = sum_i C_i dw_k/dC_i
//   J_kT = (W_k/rho) (dw_k/dT - s_k/T + w_k/T)
//   J_Tj = -(sum_k hm_k J_kj + f_T cpm_j)/c_p,  J_TT = -(sum_k hm_k J_kT + sum_k cpm_k f_k + f_T dc_p/dT)/c_p
// (hm, cpm: mass-specific enthalpy and heat capacity).
// One-sided finite-difference Jacobian (the ablation of section 2.3): column
// j is (f(y + d_j e_j) - f(y)) / d_j with d_j = sqrt(eps) max(|y_j|, 1e-10)
// rounded to a representable step; N + 1 evaluations of f.  Returns f(y).
__device__ inline double jac_fd(const MechView& m, const CellWs& w, double y, double p, int lane) {
  const int N = m.d.N, S = m.d.S;
  const double f0 = rhs(m, w, y, p, lane);
#pragma clang loop unroll(disable)
  for (int j = 0; j < N; ++j) {
    const double yj = readlane(y, j);
    double d = 1.4901161193847656e-08 * fmax(fabs(yj), 1e-10);
    d = (yj + d) - yj;
    const double fj = rhs(m, w, lane == j ? yj + d : y, p, lane);
    if (lane < N) w.J[lane * S + j] = (fj - f0) / d;
  }
  if (lane < N)
    for (int j = N; j < S; ++j) w.J[lane * S + j] = 0.0;  // padding columns
  wsync();
  return f0;
}

template <int NP, bool PROF = false>
__device__ inline double jac_pass(const MechView& m, const CellWs& w, double y, double p, int lane,
                                  Prof<PROF>* pf = nullptr, bool fd = false) {
  if (PROF && fd) return jac_fd(m, w, y, p, lane);
  const int K = m.d.K, R = m.d.R, N = m.d.N, S = m.d.S;
  const unsigned long long t0 = PROF ? pf->now() : 0ull;
  Mix x;
  double Yk;
  SpThermo t = species_phase(m, w, y, p, lane, x, Yk);
#pragma clang loop unroll(disable)
  for (int r = lane; r < R; r += WAVE) {
    const Slots s = unpack(m.sp[r]);
    const double lnkf = m.lnA[r] + m.b[r] * x.lnT - m.th[r] * x.iT;
    const double Rf = w.C[s.r0] * w.C[s.r1] * w.C[s.r2];
    const double Rr = w.C[s.p0] * w.C[s.p1] * w.C[s.p2];
    const double sng = w.g[s.p0] + w.g[s.p1] + w.g[s.p2] - w.g[s.r0] - w.g[s.r1] - w.g[s.r2];
    const double snh = w.hR[s.p0] + w.hR[s.p1] + w.hR[s.p2] - w.hR[s.r0] - w.hR[s.r1] - w.hR[s.r2];
    const double kf = exp(lnkf);
    const double iKc = exp(sng - s.dnu * x.lnPRT);
    const double dlnkf = m.b[r] * x.iT + m.th[r] * x.iT * x.iT;
    const double dlnKc = (snh - (double)s.dnu) * x.iT;
    const double net = Rf - iKc * Rr;
    double keff = kf, dkM = 0.0, dqdT;
    if (r < m.d.R0) {
      dqdT = kf * (dlnkf * Rf - iKc * (dlnkf - dlnKc) * Rr);
    } else {
      const double M = third_body(m, w, r, x.Ctot);
      if (r < m.d.R1) {
        keff = kf * M;
        dkM = kf * net;
        dqdT = M * kf * (dlnkf * Rf - iKc * (dlnkf - dlnKc) * Rr);
      } else {
        double dlnk;
        keff = troe_k<true>(m, r, x, kf, dlnkf, M, dkM, dlnk);
        dkM *= net;
        dqdT = keff * (dlnk * net + iKc * Rr * dlnKc);
      }
    }
    w.rk[r] = keff;
    w.rkr[r] = keff * iKc;
    if (r >= m.d.R0) w.rdm[r - m.d.R0] = dkM;
    w.rdt[r] = dqdT;
  }
  if (PROF) pf->add(6, t0);
  const unsigned long long t1 = PROF ? pf->now() : 0ull;
  // species rows of dw/dC (sparse), scattered by the balanced schedule: lane l
  // takes entry it * 64 + l, species k and reaction r, and adds to row k of J.
  // While they are built, omega_k, d omega_k / dT and the row's dense
  // third-body sum are accumulated in J[k+1][0] (column 0, written after this
  // pass), hR[k] (free after the reaction phase) and J[0][k+1] (row 0, written
  // after this pass).  All additions are LDS atomics, in schedule order and,
  // within one instruction, in the hardware's lane order: deterministic.
  const bool isSp = lane >= 1 && lane <= K;
  double* Jr = w.J + lane * S;  // S = NP + 1: every static column index stays in the row
  if (lane < N) {
#pragma unroll
    for (int j = 0; j < NP + 1; ++j) Jr[j] = 0.0;
  }
  if (isSp) w.hR[lane - 1] = 0.0;
  wsync();
  {
    const uint32_t* js = m.jsched + lane;
    uint32_t ent = js[0];
#pragma clang loop unroll(disable)
    for (int it = 0; it < m.jit; ++it) {
      const uint32_t cur = ent;
      if (it + 1 < m.jit) ent = js[(it + 1) * WAVE];
      if (cur != ~0u) {
        const int r = (int)(cur >> 16), k = (int)((cur >> 8) & 0xFF);
        const double nu = (double)(int8_t)(cur & 0xFF);
        const Slots sl = unpack(m.sp[r]);
        const double c0 = w.C[sl.r0], c1 = w.C[sl.r1], c2 = w.C[sl.r2];
        const double d0 = w.C[sl.p0], d1 = w.C[sl.p1], d2 = w.C[sl.p2];
        const double kf = w.rk[r], kr = w.rkr[r], dq = w.rdt[r];
        double* Jk = w.J + (k + 1) * S;
        atomicAdd(Jk, nu * (kf * c0 * c1 * c2 - kr * d0 * d1 * d2));
        atomicAdd(w.hR + k, nu * dq);
        const double a = nu * kf, bb = -nu * kr;
        atomicAdd(Jk + 1 + sl.r0, a * c1 * c2);
        atomicAdd(Jk + 1 + sl.r1, a * c0 * c2);
        atomicAdd(Jk + 1 + sl.r2, a * c0 * c1);
        atomicAdd(Jk + 1 + sl.p0, bb * d1 * d2);
        atomicAdd(Jk + 1 + sl.p1, bb * d0 * d2);
        atomicAdd(Jk + 1 + sl.p2, bb * d0 * d1);
        if (r >= m.d.R0) {
          const double dm = nu * w.rdm[r - m.d.R0];
          atomicAdd(w.J + 1 + k, dm);
          const int t1 = m.tbp[r - m.d.R0 + 1];
#pragma clang loop unroll(disable)
          for (int q = m.tbp[r - m.d.R0]; q < t1; ++q) atomicAdd(Jk + 1 + m.tbs[q], dm * m.tbd[q]);
        }
      }
    }
  }
  lds_wait();
  wsync();
  double om = 0.0, dwdT = 0.0, adense = 0.0;
  if (isSp) {
    om = Jr[0];
    dwdT = w.hR[lane - 1];
    adense = w.J[lane];
  }
  // dense transform of the lane's row: rank-1 density term and W scaling
  // (uniform loop bounds: no per-column branches; padding columns set to 0)
  double fk = 0.0;
  if (isSp) {
    const int k = lane - 1;
    const double Wk = m.W[k];
    double sk = 0.0;
#pragma clang loop unroll_count(4)
    for (int j = 1; j < N; ++j) sk += w.C[j - 1] * (Jr[j] + adense);
    const double gam = Wk * x.Wbar * x.iRho * (om - sk);
#pragma clang loop unroll_count(4)
    for (int j = 1; j < N; ++j) Jr[j] = m.iW[j - 1] * (Wk * (Jr[j] + adense) + gam);
#pragma clang loop unroll(disable)
    for (int j = N; j < NP; ++j) Jr[j] = 0.0;
    Jr[0] = Wk * x.iRho * (dwdT - sk * x.iT + om * x.iT);
    fk = Wk * om * x.iRho;
    // mass-specific enthalpy for the T row (g/RT is no longer needed)
    w.g[k] = RU * x.T * t.hRT * m.iW[k];
  }
  const double Q = wave_sum(isSp ? t.hRT * om : 0.0);
  const double fT = -RU * x.T * Q * x.iRho / x.cp;
  const double cpm = isSp ? RU * t.cpR * m.iW[lane - 1] : 0.0;
  const double s1 = wave_sum(cpm * fk);
  const double dcpdT = wave_sum(isSp ? Yk * RU * t.dcpR * m.iW[lane - 1] : 0.0);
  wsync();
  // T row: column sums of the species rows weighted by mass enthalpy
  if (lane < N) {
    double acc = 0.0;
    double a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int k = 0;
#pragma clang loop unroll(disable)
    for (; k + 4 <= K; k += 4) {
      acc += w.g[k] * w.J[(1 + k) * S + lane];
      a1 += w.g[k + 1] * w.J[(2 + k) * S + lane];
      a2 += w.g[k + 2] * w.J[(3 + k) * S + lane];
      a3 += w.g[k + 3] * w.J[(4 + k) * S + lane];
    }
#pragma clang loop unroll(disable)
    for (; k < K; ++k) acc += w.g[k] * w.J[(1 + k) * S + lane];
    acc = (acc + a1) + (a2 + a3);
    w.J[lane] = (lane == 0) ? -(acc + s1 + fT * dcpdT) / x.cp : -(acc + fT * cpm) / x.cp;
  }
  wsync();
  if (PROF) pf->add(7, t1);
  return lane == 0 ? fT : fk;
}

// 1/x from the hardware estimate refined by two Newton steps (within an ulp
// or two of the correctly rounded quotient for normal x).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// What a factorisation leaves besides the factors in the row registers.  Rows
// stay in their lanes: the row chosen at step k is lane piv(k)'s, its L part in
// columns < k and its U part in columns >= k.  Padding rows (lane >= N) count as
// chosen at their own step.
template <int NP>
struct LuPiv {
  unsigned pk[NP / 4];  // piv(4P) .. piv(4P + 3), one per byte (wave-uniform)
  int step;             // the step at which this lane's row was the pivot
  int src;              // piv(lane)
  double rdiag;         // 1 / U_kk of this lane's row
  __device__ __forceinline__ int piv(int k) const { return (int)((pk[k / 4] >> (8 * (k % 4))) & 63u); }
};

// The outcomes of a pivot search other than one lane of largest upper half kmax:
// several share it (c), or no row is left (a padding step: the pivot is lane k).
// The largest lower half decides, then getrf's row order.  Returns a mask whose
// lowest lane is the pivot; records a zero pivot.
// getrf holds a row not yet chosen at the first x >= k of x = row, piv(row),
// piv(piv(row)), ...: step j puts the row at j where row piv(j) was (src: lane
// j < k holds piv(j)).  A row already chosen may lie on a cycle.
// Bound: the chain of the two reductions.  Matrices of a few magnitudes tie in
// most columns: walking the tied lanes and replaying the interchanges took
// 1,753 us for 20,000 periodic second differences of 64 (829 with the order kept
// up at every step), now 809; +-1 matrices of 55, solved, 574 (471), now 381.
__device__ inline unsigned long long lu_tie(bool elig, bool c, unsigned kmax, unsigned lo, int src, int k, int lane,
                                            int& info) {
  if (!ballot(elig)) return 1ull << k;
  c = c && elig;
  const unsigned lmax = wave_max_u32(c ? lo : 0u);
  c = c && lo == lmax;
  const unsigned long long cand = ballot(c);
  if ((kmax | lmax) == 0u && info == 0) info = k + 1;
  if ((cand & (cand - 1)) == 0ull) return cand;
  int x = c ? lane : k;
#pragma clang loop unroll(disable)
  for (int i = 0; i < k && ballot(x < k); ++i) {
    const int y = __builtin_amdgcn_ds_bpermute(4 * x, src);
    x = x < k ? y : x;
  }
  const unsigned early = c ? (unsigned)(WAVE - x) : 0u;
  const unsigned first = wave_max_u32(early);  // of all lanes, not behind the &&
  return ballot(c && early == first);
}

// Doubles of the LDS scratch that lu_factor uses (four rows of U).
constexpr int LU_SCRATCH = 4 * WAVE;

// The matrix as the factorisation takes it: 16 x 16 tiles of the transposed
// matrix, x[t][g] of lane l = element (row 16 t + l % 16, column 4 g + l / 16).
template <int NP>
struct MatTiles {
  static constexpr int NT = (NP + 15) / 16;
  double x[4][4 * NT];
};

// LU with partial pivoting, with getrf's pivot rule: at step k the pivot is the
// unpivoted row of largest |a|, exact ties going to the row that comes first in
// getrf's current row order.  No rows move; the factors come out row-per-lane.
// |a| is compared as an integer key: the upper 32 bits (sign cleared) by one
// wave max; only when several lanes share the largest upper half do the lower
// halves, and then the positions, decide.  Returns the 1-based step of the
// first zero pivot (the factors are then meaningless), or 0.
//
// Bound: VALU issue and, with few waves, the chain of pivot searches.  In
// row-per-lane form every column right of the pivot costs two readlanes and an
// FMA at every step, about 22 issue cycles, most of them spent on the
// broadcast.  So the columns are taken four at a time, and the rest of the
// matrix gets one rank-4 update per panel on the FP64 matrix cores
// (v_mfma_f64_16x16x4, 64 cycles for 1,024 FMAs: the FMA rate without the
// broadcasts).  In the tile layout the four columns of a panel are one register
// per row tile: a block_transpose turns them into row-per-lane columns for the
// pivot search, and the multipliers come out of a second one in the
// instruction's operand layout.  The instruction adds its four products in
// order with one rounding each, and a rank-4 update is four steps of the
// elimination, so the factors are those of the step-by-step elimination bit
// for bit.  The panel's pivot rows go through LDS (lane = column) for the 4 x 4
// triangular solve.  Within a column tile the four panels share one loop body:
// the tile's registers rotate by one column group per panel, so the current
// group is always the first (unrolled over all panels the code, 110 KB for the
// integrator, no longer fits the instruction cache).
// Measured for N = 55 in a loop of its own (shader cycles of one factorisation,
// two waves per SIMD / one wave): 87.9k / 67.5k row-per-lane with the rows permuted
// at the end, 54.7k / 42.3k this way.
// FACTORS: the factors are the result, and a NaN stays in the rows and columns
// that the elimination takes it to.  A solve needs no such care (a NaN
// multiplier makes every x NaN), and the integrators have no register for it
// (k_adjoint<56> would go from 12 to 1,244 bytes of scratch).
template <int NP, bool FACTORS = false>
__device__ __forceinline__ int lu_factor(MatTiles<NP>& M, double (&row)[NP], int N, int lane, LuPiv<NP>& f, double* ub,
                                         bool nopiv = false) {
  constexpr int NG = NP / 4, NT = MatTiles<NP>::NT;  // column groups; row and column tiles
  f.step = lane;
  f.src = lane;
  f.rdiag = 0.0;
  int info = 0;
  bool elig = lane < N;
  int packed = 0x03020100 + 0x04040404 * lane;  // lane g: piv(4 g) .. piv(4 g + 3)
  auto& X = M.x;
  const int n16 = lane & 15, cb = lane >> 4;
  static_for<0, NT>([&](auto Tcc) __attribute__((always_inline)) {
    constexpr int tc = decltype(Tcc)::value, g0 = 4 * tc;
    // column that this lane reads of the pivot rows; the lanes of the current
    // tile follow its rotation
    int ucol = lane;
#pragma clang loop unroll(disable)
    for (int v = 0; v < 4; ++v) {
      const int k0 = 16 * tc + 4 * v;
      // X[t][g0 + j]: column group g0 + (v + j) % 4; groups before v hold the
      // finished columns row-per-lane (X[q] = column 4 g + q)
      double c[4] = {X[0][g0], X[1][g0], X[2][g0], X[3][g0]};
      double nl[4] = {0.0, 0.0, 0.0, 0.0};  // minus the multipliers, 0 in the rows already chosen
      int p[4] = {k0, k0 + 1, k0 + 2, k0 + 3};
      const unsigned long long open = ballot(elig);  // rows not chosen before this panel
      if (k0 < N) {
        block_transpose(c);
        static_for<0, 4>([&](auto Qc) __attribute__((always_inline)) {
          constexpr int q = decltype(Qc)::value;
          const int k = k0 + q;
          // every lane's reciprocal is formed while the search runs (the asm keeps
          // it before the branch)
          double r = recip(c[q]);
          const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, c[q]) >> 32) & 0x7fffffffu;
          const unsigned key = elig ? hi : 0u;
          const unsigned kmax = wave_max_u32(key);
          const bool top = key == kmax;
          unsigned long long cand = ballot(top);
          asm volatile("" : "+v"(r));
          // one lane, unless several share the upper half or every key is 0
          if (__builtin_expect(__builtin_popcountll(cand) != 1, 0)) {
            const unsigned lo = (unsigned)__builtin_bit_cast(unsigned long long, c[q]);
            cand = lu_tie(elig, top, kmax, lo, f.src, k, lane, info);
          }
          int pq = uniform_int(__builtin_ctzll(cand));
          if (nopiv && k < N) {  // ablation: the pivot is row k itself
            pq = k;
            if (!(readlane(c[q], k) != 0.0) && info == 0) info = k + 1;
          }
          p[q] = pq;
          const bool me = lane == pq;
          const double rp = readlane(r, pq);
          f.src = writelane(pq, k, f.src);
          f.step = writelane(k, pq, f.step);
          f.rdiag = me ? r : f.rdiag;
          elig = elig && !me;
          const double nlq = -(c[q] * rp);
          nl[q] = elig ? nlq : 0.0;
          c[q] = elig ? -nlq : c[q];
#pragma unroll
          for (int j = q + 1; j < 4; ++j) c[j] = fma(nl[q], readlane(c[j], pq), c[j]);
        });
        packed = writelane(p[0] | (p[1] << 8) | (p[2] << 16) | (p[3] << 24), g0 + v, packed);
      }
      // the tile's groups move up by one; the finished one goes last
      static_for<0, 4>([&](auto Tc) __attribute__((always_inline)) {
        constexpr int t = decltype(Tc)::value;
        X[t][g0] = X[t][g0 + 1];
        X[t][g0 + 1] = X[t][g0 + 2];
        X[t][g0 + 2] = X[t][g0 + 3];
        X[t][g0 + 3] = c[t];
      });
      ucol = (lane >> 4) == tc ? (ucol & ~12) | ((ucol + 4) & 12) : lane;
      if (k0 + 4 < N) {
        // the panel's pivot rows, open columns, to LDS: ub[q][column]
        wsync();
        const unsigned tiles = (1u << (p[0] >> 4)) | (1u << (p[1] >> 4)) | (1u << (p[2] >> 4)) | (1u << (p[3] >> 4));
        auto put = [&](auto Tc) __attribute__((always_inline)) {
          constexpr int t = decltype(Tc)::value;
          const int r = 16 * t + n16;
          int q = r == p[0] ? 0 : -1;
          q = r == p[1] ? 1 : q;
          q = r == p[2] ? 2 : q;
          q = r == p[3] ? 3 : q;
          asm("" : "+v"(q));  // one compare, not four branches
          if (q >= 0) {
            double* d = ub + q * WAVE + cb;
            d[16 * tc + ((4 * v + 4) & 15)] = X[t][g0];
            d[16 * tc + ((4 * v + 8) & 15)] = X[t][g0 + 1];
            d[16 * tc + ((4 * v + 12) & 15)] = X[t][g0 + 2];
            static_for<g0 + 4, NG>([&](auto Hc) __attribute__((always_inline)) {
              constexpr int h = decltype(Hc)::value;
              d[4 * h] = X[t][h];
            });
          }
        };
        if (__builtin_expect((tiles & (1u << tc)) != 0u, 1)) put(Tcc);
        if (__builtin_expect((tiles & ~(1u << tc)) != 0u, 0)) {  // usually all four are rows of the diagonal tile
          static_for<0, NT>([&](auto Tc) __attribute__((always_inline)) {
            constexpr int t = decltype(Tc)::value;
            if constexpr (t != tc)
              if ((tiles >> t) & 1u) put(Tc);
          });
        }
        // 0 in the tile's finished columns, whose registers the update then leaves alone
        if (n16 < 4 * v + 4) ub[cb * WAVE + 16 * tc + n16] = 0.0;
        wsync();
        // lane = column: rows k0 .. k0 + 3 of U by forward substitution (columns
        // left of the tile are not used, nor are those past the last group)
        double u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = ub[q * WAVE + ucol];
#pragma unroll
        for (int q = 1; q < 4; ++q)
#pragma unroll
          for (int j = 0; j < q; ++j) u[q] = fma(readlane(nl[j], p[q]), u[j], u[q]);
        // A NaN among a row's multipliers (input that is not finite, a pivot below
        // the normal range) makes its open columns NaN.  The update would take it
        // to finished columns too (NaN times their 0): the row sits it out, and
        // the finished columns of U are 0 again where the substitution met one.
        unsigned long long bad = 0;
        if constexpr (FACTORS) {
          const bool num = __builtin_isfinite(nl[0] + nl[1] + nl[2] + nl[3]);
          bad = ballot(!num);
          if (__builtin_expect(bad != 0ull, 0)) {
            const bool done = (lane >> 4) == tc && (ucol & 15) < 4 * v + 4;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              nl[q] = num ? nl[q] : 0.0;
              u[q] = done ? 0.0 : u[q];
            }
          }
        }
        block_transpose(u);   // -> operand A of column tile c, lane i: U[k0 + i / 16][16 c + i % 16]
        block_transpose(nl);  // -> operand B of row tile t, lane i: -L[16 t + i % 16][k0 + i / 16]
        // The lane swaps write both operands, and the compiler (ROCm 7.2) does not
        // keep the wait states that an MFMA reading the second one needs: one
        // instruction after the swap it read the old value.  Every MFMA takes its
        // nl from the wait, and its u was taken up before it (volatile statements
        // keep their order), so neither swaps nor MFMAs can move across.  The
        // wait's length (4) is a margin over that observation, not a documented
        // figure.
        __builtin_amdgcn_sched_barrier(0);
        static_for<tc, NT>([&](auto Cc) __attribute__((always_inline)) {
          double& uc = u[decltype(Cc)::value];
          asm volatile("" : "+v"(uc));
        });
        if constexpr (NT == 1) asm volatile("s_nop 3" : "+v"(nl[0]));
        else if constexpr (NT == 2) asm volatile("s_nop 3" : "+v"(nl[0]), "+v"(nl[1]));
        else asm volatile("s_nop 3" : "+v"(nl[0]), "+v"(nl[1]), "+v"(nl[2]), "+v"(nl[3]));
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, NT>([&](auto Tc) __attribute__((always_inline)) {
          constexpr int t = decltype(Tc)::value;
          // a tile above the diagonal one has usually no open row left
          if (t >= tc || __builtin_expect(((open >> (16 * t)) & 0xffffull) != 0ull, 0)) {
            static_for<tc, NT>([&](auto Cc) __attribute__((always_inline)) {
              constexpr int ct = decltype(Cc)::value;
              dbl4 d = {X[t][4 * ct], X[t][4 * ct + 1], X[t][4 * ct + 2], X[t][4 * ct + 3]};
              d = __builtin_amdgcn_mfma_f64_16x16x4f64(u[ct], nl[t], d, 0, 0, 0);
              X[t][4 * ct] = d[0], X[t][4 * ct + 1] = d[1], X[t][4 * ct + 2] = d[2], X[t][4 * ct + 3] = d[3];
            });
          }
        });
        if (FACTORS && __builtin_expect(bad != 0ull, 0)) {
          static_for<0, NT>([&](auto Tc) __attribute__((always_inline)) {
            constexpr int t = decltype(Tc)::value;
            if ((bad >> (16 * t + n16)) & 1ull) {
              static_for<g0, 4 * NT>([&](auto Gc) __attribute__((always_inline)) {
                constexpr int g = decltype(Gc)::value;
                if (g >= g0 + 4 || g < g0 + 3 - v) X[t][g] = __builtin_nan("");
              });
            }
          });
        }
      }
    }
  });
  if (lane >= N) f.rdiag = 0.0;
  static_for<0, NG>([&](auto Gc) __attribute__((always_inline)) {
    constexpr int g = decltype(Gc)::value;
    f.pk[g] = (unsigned)__builtin_amdgcn_readlane(packed, g);
    row[4 * g] = X[0][g], row[4 * g + 1] = X[1][g], row[4 * g + 2] = X[2][g], row[4 * g + 3] = X[3][g];
  });
  return info;
}

// Solve M x = b with the factors as lu_factor leaves them; lane i holds b_i
// and gets x_i.  Forward substitution with the unit-lower L and back
// substitution with U, both by columns: the value of step k is broadcast from
// lane piv(k) and every lane applies the column's update (a lane past its own
// step only changes a value that has already been read), so no per-element
// triangle mask is formed.  y_k is kept in its row's lane, x_k goes to lane k.
template <int NP>
__device__ inline double lu_solve(const double (&row)[NP], const LuPiv<NP>& f, double b) {
  // padding rows carry b = 0 and zeros, so all NP steps run unconditionally
  double y = 0.0;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int pk = f.piv(k);
    const double yk = readlane(b, pk);
    y = writelane(yk, pk, y);
    b = fma(-row[k], yk, b);
  }
  b = y;
  double x = 0.0;
#pragma unroll
  for (int k = NP - 1; k >= 0; --k) {
    const double xk = readlane(b * f.rdiag, f.piv(k));
    x = writelane(xk, k, x);
    b = fma(-row[k], xk, b);
  }
  return x;
}

// M = I/(gamma h) - J from the LDS Jacobian into tiles.  Returns false if an
// entry is not finite.
template <int NP>
__device__ inline bool form_matrix(const CellWs& w, int N, int S, int lane, double d, MatTiles<NP>& M) {
  constexpr int NG = NP / 4, NT = MatTiles<NP>::NT;
  constexpr int NMIN = NP == 16 ? 1 : NP == 32 ? 17 : NP == 56 ? 33 : 57;  // smallest N this NP serves
  double chk = 0.0, jd = 0.0;
  if (lane < N) {
    jd = w.J[lane * S + lane];
    w.J[lane * S + lane] = jd - d;
  }
  wsync();
  static_for<0, 4>([&](auto Tc) __attribute__((always_inline)) {
    constexpr int t = decltype(Tc)::value;
    const int r = 16 * t + (lane & 15);
    static_for<0, 4 * NT>([&](auto Gc) __attribute__((always_inline)) { M.x[t][decltype(Gc)::value] = 0.0; });
    if constexpr (t < NT) {
      if (16 * t + 15 < NMIN || r < N) {
        // the Jacobian pass leaves zeros in the padding columns j < NP < S
        const double* Jr = w.J + r * S + (lane >> 4);
        static_for<0, NG>([&](auto Gc) __attribute__((always_inline)) {
          constexpr int g = decltype(Gc)::value;
          M.x[t][g] = -Jr[4 * g];
          chk += M.x[t][g];
        });
      }
    }
  });
  wsync();
  if (lane < N) w.J[lane * S + lane] = jd;
  return ballot(!__builtin_isfinite(chk)) == 0ull;
}

// A row-major n x n matrix in global memory into tiles (zeros in the padding).
template <int NP>
__device__ inline void load_tiles(const double* A, int n, int lane, MatTiles<NP>& M) {
  constexpr int NG = NP / 4, NT = MatTiles<NP>::NT;
  const int cb = lane >> 4;
  static_for<0, 4>([&](auto Tc) __attribute__((always_inline)) {
    constexpr int t = decltype(Tc)::value;
    const int r = 16 * t + (lane & 15);
    static_for<0, 4 * NT>([&](auto Gc) __attribute__((always_inline)) {
      constexpr int g = decltype(Gc)::value;
      M.x[t][g] = t < NT && g < NG && r < n && 4 * g + cb < n ? A[(size_t)r * n + 4 * g + cb] : 0.0;
    });
  });
}

// One Rosenbrock attempt from y with f0 = f(y) and J(y) in LDS.  Writes ynew
// and err (lane-local); returns 1 if M is singular and 2 if M holds a
// non-finite value.  Stage vectors live in a shift register: after stage i,
// K0 = K_i, K1 = K_{i-1}, ..., so coefficient a_ij multiplies K_{i-1-j}.
template <int NP, bool PROF>
__device__ inline int ros_attempt(const MechView& m, const CellWs& w, const RosTable& tab, double p, int lane,
                                  double y, double f0, double h, MatTiles<NP>& M, double (&row)[NP], double& ynew,
                                  double& err, LuPiv<NP>& lu, Prof<PROF>& pf, double* kst = nullptr, bool nopiv = false,
                                  int formed = -1) {
  const int N = m.d.N;
  // formed: -1 form M here from the LDS Jacobian; 1 / 0: M is already there
  // (formed by the caller while it held the Jacobian), finite / not finite
  bool okm = formed == 1;
  if (formed < 0) {
    pf.start();
    okm = form_matrix<NP>(w, N, m.d.S, lane, 1.0 / (tab.gamma * h), M);
    pf.stop(1);
  }
  if (!okm) return 2;
  const int info = lu_factor<NP>(M, row, N, lane, lu, w.lu, PROF && nopiv);
  pf.stop(2);
  if (info) return 1;
  const double ih = 1.0 / h;
  const int s = tab.s;
  double K0 = 0.0, K1 = 0.0, K2 = 0.0, K3 = 0.0;
  double fi = f0;
#pragma clang loop unroll(disable)
  for (int i = 0; i < s; ++i) {
    // contributions of K_{i-1}, K_{i-2}, K_{i-3}, one aligned row per stage
    const RosStage st = tab.stage[i];
    const double a0 = st.a[0], a1 = st.a[1], a2 = st.a[2], c0 = st.c[0], c1 = st.c[1], c2 = st.c[2];
    if (st.newf) {
      const double Yi = y + a0 * K0 + a1 * K1 + a2 * K2;
      pf.start();
      fi = rhs(m, w, lane < N ? Yi : 0.0, p, lane);
      pf.stop(3);
    }
    const double r = fi + ih * (c0 * K0 + c1 * K1 + c2 * K2);
    pf.start();
    const double ki = lu_solve<NP>(row, lu, lane < N ? r : 0.0);
    pf.stop(4);
    K3 = K2;
    K2 = K1;
    K1 = K0;
    K0 = ki;
  }
  if (kst) {  // stage order: kst[i] = K_i (four-stage tables)
    kst[0] = K3;
    kst[1] = K2;
    kst[2] = K1;
    kst[3] = K0;
  }
  // after s stages K0 = K_{s-1}, K1 = K_{s-2}, ...
  const double m0 = tab.mr[0], m1 = tab.mr[1], m2 = tab.mr[2], m3 = tab.mr[3];
  const double e0 = tab.er[0], e1 = tab.er[1], e2 = tab.er[2], e3 = tab.er[3];
  ynew = y + (m0 * K0 + m1 * K1 + m2 * K2 + m3 * K3);
  err = e0 * K0 + e1 * K1 + e2 * K2 + e3 * K3;
  return 0;
}

// Adaptive integration of cell c over [0, dt]; the step-size controller
// follows the constants in a.ctl (accept iff err <= 1, no growth right after a
// rejection, non-finite err rejects with fac_min, the last step is clipped to
// dt and h_out is the last unclipped proposal capped at dt).
//
// With a slot pool the Jacobian block is not the wave's own: each attempt
// takes a slot, runs the Jacobian pass (which also yields f(y)), forms M in
// registers and gives the slot back.  A rejected attempt therefore repeats
// the Jacobian pass; the values are the same bits as the first time, so the
// results equal those of a wave that keeps its Jacobian.
template <int NP, bool PROF>
__device__ __forceinline__ void integrate_cell(const MechView& m, const CellWs& w0, const IntArgs& a, int64_t c,
                               const SlotPool* pool = nullptr) {
  const int lane = lane_id();
  Prof<PROF> pf;
  const unsigned long long t_begin = PROF ? __builtin_readcyclecounter() : 0ull;
  const int N = m.d.N;
  CellWs w = w0;
  if (lane == 0) {  // padding species: C = 1, g/RT = h/RT = 0
    w.C[m.d.K] = 1.0;
    w.g[m.d.K] = 0.0;
    w.hR[m.d.K] = 0.0;
  }
  wsync();
  double y = lane < N ? a.state[(int64_t)lane * a.ld + c] : 0.0;
  const double dt = a.dt;
  const double hin = a.h[c];
  double hprop = (__builtin_isfinite(hin) && hin > 0.0) ? fmin(hin, dt) : dt;
  int status = ST_OK, steps = 0, rejects = 0, attempts = 0;
  const bool bad = lane < N && (!__builtin_isfinite(y) || (lane == 0 && !(y > 0.0)));
  if (ballot(bad)) status = ST_NONFINITE;
  double t = 0.0;
  bool rej_last = false;
  const int nck = a.tape_y ? a.max_tape / a.ckpt + 1 : 0;
  if (a.tape_y && lane < N) a.tape_y[(c * (int64_t)nck) * N + lane] = y;
  MatTiles<NP> M;
  double row[NP];
  LuPiv<NP> lu;
  int ntape = 0;
  const RosTable& tab = kTables[a.method];
  while (status == ST_OK && t < dt) {
    double f0 = 0.0;
    if (!pool) {
      pf.start();
      f0 = jac_pass<NP, PROF>(m, w, y, a.p, lane, &pf, PROF && a.jac_fd);
      pf.stop(0);
    }
    bool fresh = true;
    int nsing = 0;
    bool accepted = false;
    while (!accepted) {
      if (attempts >= a.ctl.max_steps) { status = ST_TOO_MANY; break; }
      if (!(hprop >= a.ctl.h_min)) { status = ST_UNDERFLOW; break; }
      double h = hprop;
      bool clipped = false;
      if (h >= dt - t) { h = dt - t; clipped = true; }
      ++attempts;
      int formed = -1;
      if (pool) {
        const int sl = pool->acquire(1u << 26);
        if (sl < 0) { status = ST_NONFINITE; break; }  // unreachable unless a slot is never returned
        w.J = pool->slot(sl);
        pf.start();
        f0 = jac_pass<NP, PROF>(m, w, y, a.p, lane, &pf, PROF && a.jac_fd);
        pf.stop(0);
        formed = form_matrix<NP>(w, N, m.d.S, lane, 1.0 / (tab.gamma * h), M) ? 1 : 0;
        pf.stop(1);
        pool->release(sl);
        w.J = nullptr;
      }
      if (fresh && ballot(lane < N && !__builtin_isfinite(f0))) { status = ST_NONFINITE; break; }
      double ynew, err;
      int rc = ros_attempt<NP, PROF>(m, w, tab, a.p, lane, y, f0, h, M, row, ynew, err, lu, pf, nullptr,
                                     PROF && a.lu_nopiv, formed);
      if (rc == 0 && c >= a.fail_lu_lo && c < a.fail_lu_hi) rc = 1;  // testing: as if M were singular
      if (rc == 2 && fresh) { status = ST_NONFINITE; break; }
      fresh = false;
      if (rc) {
        ++rejects;
        if (++nsing > 5) { status = ST_SINGULAR; break; }
        hprop = 0.5 * h;
        rej_last = true;
        continue;
      }
      double e = 0.0;
      if (lane < N) {
        const double sc = a.atol + a.rtol * fmax(fabs(y), fabs(ynew));
        e = err / sc;
      }
      const double en = sqrt(wave_sum(e * e) / N);
      const bool fin = __builtin_isfinite(en) && ballot(lane < N && !__builtin_isfinite(ynew)) == 0ull;
      if (!fin) {
        ++rejects;
        hprop = a.ctl.fac_min * h;
        rej_last = true;
        continue;
      }
      const double fac = fmin(a.ctl.fac_max, fmax(a.ctl.fac_min, a.ctl.fac_safe * pow(en, -1.0 / a.q)));
      if (uniform_int(en <= 1.0)) {
        accepted = true;
        ++steps;
        if (a.tape_h) {
          if (ntape < a.max_tape) {
            if (lane == 0) a.tape_h[c * (int64_t)a.max_tape + ntape] = h;
          }
          ++ntape;
        }
        t = clipped ? dt : t + h;
        y = ynew;
        double hn = h * fac;
        if (rej_last) hn = fmin(hn, h);
        if (clipped) hn = fmax(hn, hprop);
        hprop = hn;
        rej_last = false;
        if (a.tape_y && ntape <= a.max_tape && (ntape % a.ckpt) == 0 && lane < N)
          a.tape_y[(c * (int64_t)nck + ntape / a.ckpt) * N + lane] = y;
      } else {
        ++rejects;
        hprop = h * fac;
        rej_last = true;
      }
    }
  }
  if (a.tape_h && ntape > a.max_tape && status == ST_OK) status = ST_TAPE;
  if (lane < N) a.state[(int64_t)lane * a.ld + c] = y;
  if (lane == 0) {
    a.h[c] = fmin(hprop, dt);
    if (a.steps) a.steps[c] = steps;
    if (a.rejects) a.rejects[c] = rejects;
    if (a.status) a.status[c] = status;
    if (a.failed && status != ST_OK) atomicAdd(a.failed, 1ull);
  }
  if (PROF && a.prof && lane < 8) {
    unsigned long long v = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (lane == i) v = pf.c[i];
    if (lane == 5) v = __builtin_readcyclecounter() - t_begin;
    a.prof[c * 8 + lane] = v;
  }
}

}  // namespace chem
