// Gas-kinetic BGK flux at one face Gauss point (Pan & Xu, Sec. 3), written
// for one GPU lane.  Templated on the arithmetic type T (double or float).
//
// Everything is in the local frame of the Gauss point: u along the face
// normal n_x, v along n_y, w along n_z.  A Maxwellian with density rho,
// velocity (U, V, W) and lambda = rho / (2 p) has the variance h =
// 1/(2 lambda) = p / rho per velocity component and K = (5 - 3 gamma) /
// (gamma - 1) internal degrees of freedom; K + 3 = 2 / (gamma - 1).
//
// Moments are taken against psi = (1, u, v, w, (u^2+v^2+w^2+xi^2)/2).  Every
// micro-slope a.psi (Eq. (8)) of the paper is the logarithmic derivative of
// its Maxwellian, so it is carried as the derivative of the primitive state,
//   (r, m_x, m_y, m_z, th) = (d rho, rho dU, rho dV, rho dW, rho dh),
// nine operations from a derivative of the conservative variables, and no
// 5x5 moment system is solved.  With c = u - U, v' = v - V, w' = w - W and
// phi(u) the normal distribution of u (mean U, variance h),
//   rho a.psi phi = r phi - m_x phi' + (th/2) phi''   (tangential mean),
//   means of rho a.psi times v', w', e' = (v'^2 + w'^2 + xi^2)/2:
//     m_y phi,  m_z phi,  (K+2)/2 (h rho a.psi phi + th phi),
// and integration by parts turns its integrals over a half line into the
// u-moments m_k and phi at u = 0 (f0, signed: + for u > 0, - for u < 0):
//   int u^k phi' = -k m_{k-1}  (k = 0: -f0),
//   int u^k phi'' = -(U/h) f0, f0, 2 m_0, 6 m_1  for k = 0..3,
//   int u^k phi''' = (1/h - U^2/h^2) f0, (U/h) f0, -2 f0, -6 m_0.
// The u-moments obey m_0 = 1, m_1 = U, m_{k+1} = U m_k + k h m_{k-1} on the
// full line, and over u > 0 (u < 0) start from m_0 = erfc(-+ sqrt(lambda)
// U)/2, m_1 = U m_0 + h f0, f0 = +- sqrt(lambda/pi) exp(-lambda U^2).
//
// The time derivative A follows from the compatibility condition
// <a_1 u + a_2 v + a_3 w + A> = 0, which in primitive variables is the Euler
// equations in non-conservative form.  The sum N = a_1 u + a_2 v + a_3 w + A
// then is the first-order (Chapman-Enskog) polynomial of the peculiar
// velocities, with <N psi> = 0 on the full line:
//   N phi = D h phi'' - (th_x/2) h phi'''             (tangential mean),
//   times v': -S_y h phi' + (th_y/2) h phi''          (w' alike),
//   times e': D ((K+2)/2 h^2 phi'' - h phi) - th_x (K+2)/4 (h^2 phi''' + 2 h phi'),
//   D = rho (dU/dx - div U / (K+3)),  S_y = rho (dU/dy + dV/dx).
// On the full line <u N psi> is the viscous stress and the heat flux.
//
// The flux of Eq. (15), read with H(u) on the left state g_l and 1 - H(u) on
// the right state g_r (the compatibility condition that follows the equation
// takes u > 0 from the left), integrated over [0, delta], in the moments of
// N and A:
//   Fhat = T1 X1 + T2 N0 + (T3 - T2) A0 + T4 X4 - T5 N1 + (T5 - tau T4) A1,
//   X1 = rho_0 <u psi>_0,  N0 = <u N psi>_0,  A0 = <u A psi>_0 (equilibrium),
//   X4, N1, A1 the same moments of g_l over u > 0 plus g_r over u < 0,
// T1..T5 the time integrals of the five time factors of Eq. (15).  Since
// T1 = delta - T4, T2 = T5 - tau delta and T3 - T2 = delta^2/2 - (T5 - tau
// T4), the linear-in-time fit of Eq. (16) to Fhat(dt) and Fhat(dt/2), F =
// (4 Fhat(dt/2) - Fhat(dt)) / dt, dF = 4 (Fhat(dt) - 2 Fhat(dt/2)) / dt^2,
// needs the fits (c4, d4), (c5, d5) of T4 and T5 only (c6 = c5 - tau c4):
//   F  = X1 - tau N0 + c4 (X4 - X1) - c5 (N1 - N0) + c6 (A1 - A0),
//   dF = A0          + d4 (X4 - X1) - d5 (N1 - N0) + d6 (A1 - A0).
#pragma once

#include "common.h"

namespace hgks {

// Constants of the gas and of the collision time, in the arithmetic type.
template <typename T>
struct GasParams {
  T gm1;      // gamma - 1
  T inv_K3;   // 1 / (K + 3)
  T K2h;      // (K + 2) / 2
  T K3h;      // (K + 3) / 2
  T K4h;      // (K + 4) / 2
  T K5;       // K + 5
  T two_gm1;  // 2 / (gamma - 1)
  T mu;       // viscosity (0: inviscid collision time)
  T tau_eps, tau_C;
  int viscous;
  T mu_exp;   // viscosity law mu (T / T0)^mu_exp on the viscous branch (0: constant)
  T mu_iT0;   // 1 / T0
  T pr_fix;   // 1 / Pr - 1: weight of the heat flux added to the energy flux
  double gamma;  // ratio of specific heats (characteristic projection)
};

// Running sums over the two sides of the interface: the conservative
// variables Q0 of g_0 and their derivatives, X4 = rho <u psi>, X5 = <u N
// psi>, X6 = <u A psi>.  X4[0] is Q0[1] and is not kept.
//
// PARK: the first kParked entries of dQ0 live in LDS, entry k of a lane at
// slot[64 k] (slot: the lane's own column of its wave's area, which no other
// lane touches), so that they hold no registers while the right side is
// formed.
constexpr int kParked = 12;

template <typename T, bool PARK = false>
struct FluxAcc {
  T Q0[5];
  T dQ0[3][5];
  T* slot = nullptr;
  T X4[5], X5[5], X6[5];
  T p[2];
  // Prandtl correction only: <N psi> and <A psi> over the half lines, which
  // the heat flux needs (S5[1] is X5[0], S6[1] is X6[0]: not kept).
  T S5[5], S6[5];
};

// How the first side of a face enters the sums: assigned (true) or added to
// zeroed sums (false).  The values are the same; assigning saves an add and a
// register clear per sum.  Measured on gfx950, with longer side terms than
// the present ones, it shortened the FP64 flux launch by about 1% but
// lengthened the FP32 one by about 3% (the compiler's schedule of the mixed
// kernel lost more than the instructions saved), so the choice is per
// precision.
template <typename T>
inline constexpr bool kAssignFirst = sizeof(T) == 8;

template <typename T, bool PARK>
HGKS_FN void acc_zero(FluxAcc<T, PARK>& A) {
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    A.Q0[i] = T(0); A.X4[i] = T(0); A.X5[i] = T(0); A.X6[i] = T(0);
    A.dQ0[0][i] = T(0); A.dQ0[1][i] = T(0); A.dQ0[2][i] = T(0);
    A.S5[i] = T(0); A.S6[i] = T(0);
  }
}

// Ready the sums for the first side of a face: zeroed unless that side
// assigns them.
template <typename T, bool PARK>
HGKS_FN void acc_begin(FluxAcc<T, PARK>& A) {
  if constexpr (!kAssignFirst<T>) acc_zero(A);
}

// y (+)= x
template <bool ACC, typename T>
HGKS_FN void put(T& y, T x) {
  if (ACC)
    y += x;
  else
    y = x;
}

// Entry i of A.dQ0[j] (+)= x, and its value.
template <bool ACC, typename T, bool PARK>
HGKS_FN void put_dq(FluxAcc<T, PARK>& A, int j, int i, T x) {
  const int k = 5 * j + i;
  if (PARK && k < kParked)
    put<ACC>(A.slot[64 * k], x);
  else
    put<ACC>(A.dQ0[j][i], x);
}

template <typename T, bool PARK>
HGKS_FN T get_dq(const FluxAcc<T, PARK>& A, int j, int i) {
  const int k = 5 * j + i;
  return PARK && k < kParked ? A.slot[64 * k] : A.dQ0[j][i];
}

// Primitive quantities of a state with conservative variables Q, from one
// reciprocal: with p2 = 2 rho E - |M|^2 = 2 rho p / (gamma - 1) and
// R = 1 / (rho p2), 1/rho = p2 R and 2 lambda = rho/p = (2/(gamma-1)) rho^2/p2.
template <typename T>
struct Prim {
  T rho, ir, U, V, W, p, h, il;
};

template <typename T>
HGKS_FN void primitives(const T (&Q)[5], const GasParams<T>& g, Prim<T>& s) {
  const T rho = Q[0];
  const T p2 = T(2) * rho * Q[4] - (Q[1] * Q[1] + Q[2] * Q[2] + Q[3] * Q[3]);
  const T R = d_rcp(rho * p2);
  const T ir = p2 * R;
  s.rho = rho;
  s.ir = ir;
  s.U = Q[1] * ir;
  s.V = Q[2] * ir;
  s.W = Q[3] * ir;
  s.p = T(0.5) * g.gm1 * p2 * ir;
  s.h = s.p * ir;                            // 1 / (2 lambda)
  s.il = g.two_gm1 * (rho * rho) * (rho * R);  // 2 lambda
}

// A derivative of the primitive state, every entry times rho (but r).
template <typename T>
struct PGrad {
  T r, mx, my, mz, th;  // d rho, rho dU, rho dV, rho dW, rho dh
};

// From the derivative b of the conservative variables; k2 = |U|^2 / 2.  The
// energy is rho (K+3)/2 h + rho |U|^2 / 2.
template <typename T>
HGKS_FN void prim_grad(const T (&b)[5], const Prim<T>& P, T k2, const GasParams<T>& g, PGrad<T>& d) {
  d.r = b[0];
  d.mx = b[1] - P.U * b[0];
  d.my = b[2] - P.V * b[0];
  d.mz = b[3] - P.W * b[0];
  const T e = b[4] - k2 * b[0] - P.U * d.mx - P.V * d.my - P.W * d.mz;
  d.th = g.gm1 * e - P.h * b[0];
}

// Time derivative of the primitive state (Euler equations) from its spatial
// derivatives d[j]; div = rho div U.
template <typename T>
HGKS_FN void time_derivative(const Prim<T>& P, const PGrad<T> (&d)[3], T div, const GasParams<T>& g, PGrad<T>& a) {
  a.r = -(div + P.U * d[0].r + P.V * d[1].r + P.W * d[2].r);
  a.mx = -(P.h * d[0].r + d[0].th + P.U * d[0].mx + P.V * d[1].mx + P.W * d[2].mx);
  a.my = -(P.h * d[1].r + d[1].th + P.U * d[0].my + P.V * d[1].my + P.W * d[2].my);
  a.mz = -(P.h * d[2].r + d[2].th + P.U * d[0].mz + P.V * d[1].mz + P.W * d[2].mz);
  a.th = -(g.gm1 * P.h * div + P.U * d[0].th + P.V * d[1].th + P.W * d[2].th);
}

// Keeps the compiler from moving instructions across this point (no
// instruction of its own).
template <bool ON>
HGKS_FN void sched_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (ON) __builtin_amdgcn_sched_barrier(0);
#endif
}

// Contributions of one side (SIDE = +1: left state, particles with u > 0;
// -1: right state, u < 0).  P: the primitive state in the local frame; d[j]:
// its derivatives along n_x, n_y, n_z.  FIRST: the first side of the
// pair, whose terms are assigned to the sums rather than added to zeroed
// ones (the same values; an add to 0.0 cannot be dropped by the compiler,
// whereas here no zeroing or add is issued).
template <int SIDE, bool PR = false, bool FIRST = false, typename T, bool PARK>
HGKS_FN void side_core(const Prim<T>& P, const PGrad<T> (&d)[3], const GasParams<T>& g, FluxAcc<T, PARK>& A) {
  constexpr bool ACC = !FIRST;
  const T sg = T(SIDE);
  const T U = P.U, V = P.V, W = P.W, h = P.h;
  const T uu = U * U;
  const T k2t = T(0.5) * (V * V + W * W);  // tangential kinetic energy
  const T et = k2t + g.K2h * h;            // mean of (v^2 + w^2 + xi^2) / 2

  // half-line moments
  const T lam = T(0.5) * P.il;
  const T sl = d_sqrt(lam);
  const T z = lam * uu;
  const T ex = d_exp(-z);
  const T f0 = sg * T(0.56418958354775628694807945156077259) * sl * ex;  // 1/sqrt(pi)
  const T m0 = T(0.5) * d_erfc(-sg * sl * U, ex, z);
  const T hf = h * f0;
  const T m1 = U * m0 + hf;
  const T m2 = U * m1 + h * m0;
  const T m3h = T(0.5) * U * m2 + h * m1;
  const T m0h = T(0.5) * m0, m2h = T(0.5) * m2, f0h = T(0.5) * f0;

  sched_fence<PARK>();
  // rho <psi> and rho <u psi>
  {
    const T r0 = P.rho * m0, r1 = P.rho * m1;
    put<ACC>(A.Q0[0], r0);
    put<ACC>(A.Q0[1], r1);
    put<ACC>(A.Q0[2], V * r0);
    put<ACC>(A.Q0[3], W * r0);
    put<ACC>(A.Q0[4], et * r0 + P.rho * m2h);
    put<ACC>(A.X4[1], P.rho * m2);
    put<ACC>(A.X4[2], V * r1);
    put<ACC>(A.X4[3], W * r1);
    put<ACC>(A.X4[4], et * r1 + P.rho * m3h);
  }
  // <a psi> of a derivative a of the state: g_k = <u^k a>, s the tangential
  // and internal part of the energy moment
  sched_fence<PARK>();
  const T k0 = U * f0h * P.il;
  auto g0_of = [&](const PGrad<T>& a) { return a.r * m0 + a.mx * f0 - a.th * k0; };
  auto g1_of = [&](const PGrad<T>& a) { return a.r * m1 + a.mx * m0 + a.th * f0h; };
  auto g2h_of = [&](const PGrad<T>& a) { return a.r * m2h + a.mx * m1 + a.th * m0h; };
  auto s_of = [&](const PGrad<T>& a) { return V * a.my + W * a.mz + g.K2h * a.th; };
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const T q0 = g0_of(d[j]);
    put_dq<ACC>(A, j, 0, q0);
    put_dq<ACC>(A, j, 1, g1_of(d[j]));
    put_dq<ACC>(A, j, 2, V * q0 + d[j].my * m0);
    put_dq<ACC>(A, j, 3, W * q0 + d[j].mz * m0);
    put_dq<ACC>(A, j, 4, g2h_of(d[j]) + et * q0 + s_of(d[j]) * m0);
    sched_fence<PARK>();
  }
  const T div = d[0].mx + d[1].my + d[2].mz;
  // <u A psi> (and <A psi>)
  {
    PGrad<T> a;
    time_derivative(P, d, div, g, a);
    const T q1 = g1_of(a), q2h = g2h_of(a), s = s_of(a);
    const T q3h = a.r * m3h + T(3) * (a.mx * m2h + a.th * (T(0.5) * m1));
    put<ACC>(A.X6[0], q1);
    put<ACC>(A.X6[1], T(2) * q2h);
    put<ACC>(A.X6[2], V * q1 + a.my * m1);
    put<ACC>(A.X6[3], W * q1 + a.mz * m1);
    put<ACC>(A.X6[4], q3h + et * q1 + s * m1);
    if constexpr (PR) {
      const T q0 = g0_of(a);
      put<ACC>(A.S6[0], q0);
      put<ACC>(A.S6[2], V * q0 + a.my * m0);
      put<ACC>(A.S6[3], W * q0 + a.mz * m0);
      put<ACC>(A.S6[4], q2h + et * q0 + s * m0);
    }
  }
  sched_fence<PARK>();
  // <u N psi> (and <N psi>)
  {
    const T D = d[0].mx - g.inv_K3 * div, Dh = D * h;
    const T sy = d[1].mx + d[0].my, sz = d[2].mx + d[0].mz;
    const T tx = T(0.5) * d[0].th, ty = T(0.5) * d[1].th, tz = T(0.5) * d[2].th;
    const T n1 = f0 * (Dh - tx * U);
    const T y1 = h * (sy * m0) + ty * hf, w1 = h * (sz * m0) + tz * hf;
    put<ACC>(A.X5[0], n1);
    put<ACC>(A.X5[1], T(2) * (Dh * m0 + tx * hf));
    put<ACC>(A.X5[2], V * n1 + y1);
    put<ACC>(A.X5[3], W * n1 + w1);
    put<ACC>(A.X5[4], Dh * (T(2) * m1 + g.K2h * hf) + tx * (g.K5 * (h * m0) - g.K2h * (U * hf)) + k2t * n1 + V * y1 +
                          W * w1);
    if constexpr (PR) {
      const T n0 = f0 * (tx * (uu * P.il - T(1)) - D * U);
      const T y0 = f0 * (sy * h - ty * U), w0 = f0 * (sz * h - tz * U);
      put<ACC>(A.S5[0], n0);
      put<ACC>(A.S5[2], V * n0 + y0);
      put<ACC>(A.S5[3], W * n0 + w0);
      put<ACC>(A.S5[4], f0 * (tx * (g.K4h * h + g.K2h * uu) - Dh * (g.K2h * U)) + k2t * n0 + V * y0 + W * w0);
    }
  }
  A.p[SIDE > 0 ? 0 : 1] = P.p;
}

// The same from the conservative variables W in the local frame and their
// derivatives dW[j] along n_x, n_y, n_z.
template <int SIDE, bool PR = false, bool FIRST = false, typename T, bool PARK>
HGKS_FN void side_terms(const T (&W)[5], const T (&dW)[3][5], const GasParams<T>& g, FluxAcc<T, PARK>& A) {
  Prim<T> P;
  primitives(W, g, P);
  const T k2 = T(0.5) * (P.U * P.U + P.V * P.V + P.W * P.W);
  PGrad<T> d[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) prim_grad(dW[j], P, k2, g, d[j]);
  side_core<SIDE, PR, FIRST>(P, d, g, A);
}

// Register budget of the flux kernels: three waves per SIMD (168 registers
// in FP64).  The kernel is bound by its vector instruction count, and at
// two waves a SIMD issues on 75% of its cycles, at three on 94%: 128^3
// Taylor-Green FP64 launch 1.54 -> 1.39 ms (-> 1.34 with one-wave
// workgroups).  Three FP64 waves fit without spills because part of the
// sums is parked in LDS (kParked) and the sums are formed before
// finish_flux (pin_sums).  The per-face form (FS) holds the eigenvectors
// besides and keeps two waves: three spill 20 registers and lengthen the
// 100^3 characteristic step from 4.71 to 5.00 ms.  FP32 fits four.
#define HGKS_FLUX_OCCUPANCY __attribute__((amdgpu_waves_per_eu(sizeof(TC) == 8 && FS ? 2 : 3)))

// Orders the loads of the right cell after the left side's terms.  The
// address gets a dependence on the left side's last results through an
// empty asm, so the compiler cannot hoist the right cell's coefficient
// loads into the left side's work, where both sides' values would be live
// at once.
template <typename T, bool PARK>
__device__ __forceinline__ void after_left_side(unsigned& idx, const FluxAcc<T, PARK>& A) {
  asm volatile("" : "+v"(idx) : "v"(A.X6[0]), "v"(A.X6[4]), "v"(A.Q0[4]), "v"(A.X4[4]));
}

// Forms every sum here: the compiler would otherwise sink the sums that only
// the last part of finish_flux reads past the branches before it, and hold
// their operands (about 50 more registers) instead.
template <bool PR, typename T, bool PARK>
__device__ __forceinline__ void pin_sums(FluxAcc<T, PARK>& A) {
  auto pin = [](T& x) { asm volatile("" : "+v"(x)); };
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    pin(A.Q0[i]);
    if (i > 0) pin(A.X4[i]);
    pin(A.X5[i]);
    pin(A.X6[i]);
    if (PR && i != 1) {
      pin(A.S5[i]);
      pin(A.S6[i]);
    }
  }
#pragma unroll
  for (int k = kParked; k < 15; ++k) pin(A.dQ0[2][k - 10]);
}

// Collision time of Sec. 4 from the two sides' pressures and the state of
// g_0.  PR: the extended viscous model -- the viscosity law and the Prandtl
// correction (either may be trivial: mu_exp = 0, pr_fix = 0).
template <bool PR, typename T, bool PARK>
HGKS_FN T collision_time(const FluxAcc<T, PARK>& A, const Prim<T>& P, const GasParams<T>& g, T dt) {
  const T jump = d_abs(A.p[0] - A.p[1]) * d_rcp(A.p[0] + A.p[1]) * dt;
  // mu / p_0 = mu (rho_0 / p_0) (1 / rho_0); mu = mu0 (T / T0)^omega with
  // T = p_0 / rho_0 when a viscosity law is set
  T mu = g.mu;
  if constexpr (PR) {
    if (g.mu_exp != T(0)) mu *= exp(g.mu_exp * log(P.h * g.mu_iT0));
  }
  return g.viscous ? mu * P.il * P.ir + g.tau_C * jump : g.tau_eps * dt + g.tau_C * jump;
}

// Equilibrium part, collision time and the time fit.  On return F and dF
// hold the flux and its time derivative in the local frame.
template <bool PR = false, typename T, bool PARK>
HGKS_FN void finish_flux(const FluxAcc<T, PARK>& A, const GasParams<T>& g, T dt, T idt, T (&F)[5], T (&dF)[5]) {
  Prim<T> P;
  primitives(A.Q0, g, P);
  const T U = P.U, V = P.V, W = P.W, h = P.h;
  const T tau = collision_time<PR>(A, P, g, dt);
  // Fits of T4 = tau (1 - E) and T5 = tau (2 T4 - delta E), E = exp(-delta /
  // tau), over dt and dt / 2 (E over dt as the square).  Below 1e-4 dt the
  // collision time leaves E = 0 in either precision, so the reciprocal is
  // taken of a number that is never 0.
  T c4, d4, c5, d5;
  {
    const T Eh = d_exp(T(-0.5) * dt * d_rcp(d_max(tau, T(1e-4) * dt)));
    const T Ef = Eh * Eh;
    const T h4 = tau * (T(1) - Eh), f4 = tau * (T(1) - Ef);
    const T h5 = tau * (T(2) * h4 - T(0.5) * dt * Eh), f5 = tau * (T(2) * f4 - dt * Ef);
    const T idt2 = T(4) * idt * idt;
    c4 = (T(4) * h4 - f4) * idt;
    c5 = (T(4) * h5 - f5) * idt;
    d4 = (f4 - T(2) * h4) * idt2;
    d5 = (f5 - T(2) * h5) * idt2;
  }
  const T c6 = c5 - tau * c4, d6 = d5 - tau * d4;

  const T k2 = T(0.5) * (U * U + V * V + W * W);
  PGrad<T> d[3], a;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const T b[5] = {get_dq(A, j, 0), get_dq(A, j, 1), get_dq(A, j, 2), get_dq(A, j, 3), get_dq(A, j, 4)};
    prim_grad(b, P, k2, g, d[j]);
  }
  const T div = d[0].mx + d[1].my + d[2].mz;
  time_derivative(P, d, div, g, a);

  // X1 = rho_0 <u psi>_0 and X4 - X1 (both have Q0[1] as first entry)
  {
    const T M = A.Q0[1];
    const T x1[5] = {M, M * U + P.p, M * V, M * W, U * (A.Q0[4] + P.p)};
    F[0] = x1[0];
    dF[0] = T(0);
#pragma unroll
    for (int i = 1; i < 5; ++i) {
      const T x = A.X4[i] - x1[i];
      F[i] = x1[i] + c4 * x;
      dF[i] = d4 * x;
    }
  }
  // N0 = <u N psi>_0 (no mass) and N1 - N0
  {
    const T sxx = T(2) * (d[0].mx - g.inv_K3 * div);
    const T sy = d[1].mx + d[0].my, sz = d[2].mx + d[0].mz;
    const T n0[5] = {T(0), h * sxx, h * sy, h * sz, h * (U * sxx + V * sy + W * sz + T(0.5) * g.K5 * d[0].th)};
    F[0] -= c5 * A.X5[0];
    dF[0] -= d5 * A.X5[0];
#pragma unroll
    for (int i = 1; i < 5; ++i) {
      const T x = A.X5[i] - n0[i];
      F[i] = F[i] - tau * n0[i] - c5 * x;
      dF[i] -= d5 * x;
    }
  }
  // A0 = <u A psi>_0 and A1 - A0
  {
    const T q = U * a.r + a.mx;
    const T H = k2 + T(0.5) * g.K5 * h;  // total enthalpy
    const T a0[5] = {q, U * (q + a.mx) + h * a.r + a.th, V * q + U * a.my, W * q + U * a.mz,
                     H * q + U * (U * a.mx + V * a.my + W * a.mz + T(0.5) * g.K5 * a.th)};
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const T x = A.X6[i] - a0[i];
      F[i] += c6 * x;
      dF[i] += a0[i] + d6 * x;
    }
  }
  // Prandtl correction: the heat flux relative to the velocity (U, V, W) of
  // g_0 is the moment of (u - U)(|c|^2 + xi^2)/2, which expands into the
  // fluxes F and the state moments S of the same distribution:
  //   q = H(F) - U H(S),  H(X) = X_E - U.X_M + |U|^2/2 X_rho.
  // S over time has the form of the flux: Q0, 0 and <A psi>_0 in place of
  // X1, N0 and A0, and Q0, S5 and S6 in place of X4, X5 and X6; H(Q0) and
  // H(<A psi>_0) are the internal energy and its rate.
  if constexpr (PR) {
    auto form = [&](T x0, T x1, T x2, T x3, T x4) { return x4 - (U * x1 + V * x2 + W * x3) + k2 * x0; };
    const T hq = g.K3h * P.p, ha = g.K3h * (h * a.r + a.th);
    const T h5 = form(A.S5[0], A.X5[0], A.S5[2], A.S5[3], A.S5[4]);
    const T h6 = form(A.S6[0], A.X6[0], A.S6[2], A.S6[3], A.S6[4]) - ha;
    F[4] += g.pr_fix * (form(F[0], F[1], F[2], F[3], F[4]) - U * (hq - c5 * h5 + c6 * h6));
    dF[4] += g.pr_fix * (form(dF[0], dF[1], dF[2], dF[3], dF[4]) - U * (ha - d5 * h5 + d6 * h6));
  }
}

}  // namespace hgks
