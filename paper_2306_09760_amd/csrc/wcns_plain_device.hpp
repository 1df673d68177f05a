// The sweep's arithmetic for runs that are differentiated (SPEC_PLAIN_FE,
// SPEC_PLAIN): FE and PFE weights in the plainer form that the other
// specialisations were shortened from.
//
// The derivative of the FE map amplifies the last bit of the states it is taken
// at: where a field's differences are 1e-7 to 1e-3 of the field (next to a
// critical point), one ulp in a stage state moves single entries of a
// two-step gradient at 2D 1024^2 by up to 1e-8 to 1e-7 of the gradient's rms
// (norm: 7e-11), whichever way the states are rounded.  A gradient is therefore
// only reproducible, entry by entry, if its forward steps round as they always
// did, and they do here: every operation, its order and what the compiler is
// left to fuse is part of the result, so nothing in this file is to be
// shortened.  (The adjoint's own arithmetic is free to change: it moves an
// entry by less than 2e-9.)
// Bound by FP64 VALU issue like the other sweeps: 266 VALU instructions per FE
// task against 219; 2D 2048^2 residual 0.416 against 0.366 ms.  JS and Z weights
// have no such amplification (below 1e-9) and keep their own kernels.
#pragma once

#include "wcns_device.hpp"

namespace wcns {
namespace plain {

// One map's g(w) over prod_j D_j, D_j = 1 + E K_j, E = exp(2 xi (w - c)) (c: the
// mean of the map's null points, K_j = exp(2 xi (c - nu_j))), as polynomials in
// E divided by prod_j K_j; Pd, Pa, Pb hold their coefficients.
template <int NT>
__device__ __forceinline__ double fe_map_poly(double w, double E, const double* pd,
                                              const double* pa, const double* pb, double* den) {
  double t = E + pd[NT - 2];
#pragma unroll
  for (int r = NT - 3; r >= 0; --r) t = __builtin_fma(t, E, pd[r]);
  *den = __builtin_fma(t, E, pd[NT - 1]);
  double ta = pa[NT - 2], tb = pb[NT - 2];
#pragma unroll
  for (int r = NT - 3; r >= 0; --r) {
    ta = __builtin_fma(ta, E, pa[r]);
    tb = __builtin_fma(tb, E, pb[r]);
  }
  return __builtin_fma(w, *den, E * __builtin_fma(w, tb, ta));
}

// a b, never fused with what becomes of it: an interpolated value that stays in a
// register between two phases is the one that others pass through LDS.
__device__ __forceinline__ double product(double a, double b) {
#pragma clang fp contract(off)
  return a * b;
}

// The weights of weigh5 applied to eight times the candidates (c0, c1, c2); FE on
// p = 2 Z weights, or FE and PFE from the run-time parameters.  xt: 2^(k/64).
template <bool FE>
__device__ __forceinline__ double weigh5(const InterpParams& P, double c0, double c1, double c2,
                                         double b0, double b1, double b2, const double* xt) {
  if constexpr (FE) {
    const double tau = __builtin_fabs(b0 - b2);
    const double t2 = tau * tau;
    const double q0 = b0 * b0, q1 = b1 * b1, q2 = b2 * b2;
    const double z0 = (q0 + t2) * (q1 * q2);
    const double z1 = FamWcns::dr1 * (q1 + t2) * (q0 * q2);
    const double z2 = FamWcns::dr2 * (q2 + t2) * (q0 * q1);
    const double zi = rcp<true>(z0 + z1 + z2);
    const double xi2 = 2.0 * P.xi;
    const double w0 = z0 * zi, w1 = z1 * zi, w2 = z2 * zi;
    // E_0 E_1 E_2 = Ke (the weights sum to one)
    const double zE0 = __builtin_fma(xi2, w0, -P.C2[0]), zE1 = __builtin_fma(xi2, w1, -P.C2[1]);
    const double Ex0 = exp_tab(zE0, xt);
    const double Ex1 = exp_tab(zE1, xt);
    const double Ex2 = P.Ke * rcp1(Ex0 * Ex1);
    double e0, e1, e2;
    const double n0 = fe_map_poly<3>(w0, Ex0, P.Pd, P.Pa, P.Pb, &e0);
    const double n1 = fe_map_poly<4>(w1, Ex1, P.Pd + 3, P.Pa + 2, P.Pb + 2, &e1);
    const double n2 = fe_map_poly<3>(w2, Ex2, P.Pd + 7, P.Pa + 5, P.Pb + 5, &e2);
    const double A = n0 * e1, B = n1 * e0, C = n2 * (e0 * e1);
    const double num = __builtin_fma(e2, __builtin_fma(A, c0, B * c1), C * c2);
    return product(FamWcns::scale * num, rcp1(__builtin_fma(e2, A + B, C)));
  }
  double a0, a1, a2;
  if (P.weights == WJS) {
    const double r0 = rcp<true>(b0), r1 = rcp<true>(b1), r2 = rcp<true>(b2);
    a0 = D0 * r0 * r0;
    a1 = D1 * r1 * r1;
    a2 = D2 * r2 * r2;
  } else {
    const double tau = __builtin_fabs(b0 - b2);
    double q0 = tau * rcp<true>(b0), q1 = tau * rcp<true>(b1), q2 = tau * rcp<true>(b2);
    double p0 = q0, p1 = q1, p2 = q2;
    for (int k = 1; k < P.zpow; ++k) {
      p0 *= q0;
      p1 *= q1;
      p2 *= q2;
    }
    a0 = D0 * (1.0 + p0);
    a1 = D1 * (1.0 + p1);
    a2 = D2 * (1.0 + p2);
  }
  const double inv = rcp<true>(a0 + a1 + a2);
  double w0 = a0 * inv, w1 = a1 * inv, w2 = a2 * inv;
  bool map = P.weights == WFE;
  if (P.weights == WPFE) {
    const bool inside = __builtin_fabs(w0 - D0) <= P.cv && __builtin_fabs(w1 - D1) <= P.cv &&
                        __builtin_fabs(w2 - D2) <= P.cv;
    map = !inside;
  }
  if (map) {
    const double g0 = fe_g0<SPEC_GENERIC, true>(w0, P), g1 = fe_g1<SPEC_GENERIC, true>(w1, P),
                 g2 = fe_g2<SPEC_GENERIC, true>(w2, P);
    const double ginv = rcp<true>(g0 + g1 + g2);
    w0 = g0 * ginv;
    w1 = g1 * ginv;
    w2 = g2 * ginv;
  }
  return product(0.125, w0 * c0 + w1 * c1 + w2 * c2);
}

template <bool FE>
__device__ __forceinline__ void interp5_pair(const InterpParams& P, const double (&u)[6],
                                             double* left, double* right, const double* xt) {
  // candidates of eq. 5 (times 8) of both stencils
  const double c0 = 3.0 * u[0] - 10.0 * u[1] + 15.0 * u[2];
  const double c1 = -u[1] + 6.0 * u[2] + 3.0 * u[3];
  const double c2 = 3.0 * u[2] + 6.0 * u[3] - u[4];
  const double r0 = 3.0 * u[5] - 10.0 * u[4] + 15.0 * u[3];
  const double r1 = -u[4] + 6.0 * u[3] + 3.0 * u[2];
  const double r2 = 3.0 * u[3] + 6.0 * u[2] - u[1];
  if (!FE && P.weights == WLIN) {
    *left = 0.125 * (D0 * c0 + D1 * c1 + D2 * c2);
    *right = 0.125 * (D0 * r0 + D1 * r1 + D2 * r2);
    return;
  }
  const double d0 = u[1] - u[0], d1 = u[2] - u[1], d2 = u[3] - u[2], d3 = u[4] - u[3],
               d4 = u[5] - u[4];
  const double s0 = d1 - d0, s1 = d2 - d1, s2 = d3 - d2, s3 = d4 - d3;
  const double q1 = __builtin_fma(s1, s1, P.eps), q2 = __builtin_fma(s2, s2, P.eps);
  const double f0 = 0.5 * (3.0 * d1 - d0), f1 = 0.5 * (d1 + d2), f2 = 0.5 * (3.0 * d2 - d3);
  const double g0 = 0.5 * (3.0 * d3 - d4), g1 = 0.5 * (d2 + d3), g2 = 0.5 * (3.0 * d2 - d1);
  *left = weigh5<FE>(P, c0, c1, c2, __builtin_fma(f0, f0, __builtin_fma(s0, s0, P.eps)),
                     __builtin_fma(f1, f1, q1), __builtin_fma(f2, f2, q2), xt);
  *right = weigh5<FE>(P, r0, r1, r2, __builtin_fma(g0, g0, __builtin_fma(s3, s3, P.eps)),
                      __builtin_fma(g1, g1, q2), __builtin_fma(g2, g2, q1), xt);
}

// The fluxes' fused products are written out: left to the compiler, which of two
// products a sum fuses changes from one tile shape to another.
template <int NV, int DIR>
__device__ __forceinline__ void node_flux(const PhysParams& PP, const double (&U)[NV],
                                          double (&F)[NV]) {
#pragma clang fp contract(off)
  if constexpr (NV == 1) {
    F[0] = PP.adv * U[0];
  } else {
    constexpr int ND = NV - 2;
    const Prim<ND> q = primitives<ND, true>(U, PP.gamma);
    const double ei = __builtin_fma(-0.5, dot<ND>(U + 1, q.vel), U[ND + 1]);
    const double vn = q.vel[DIR];
    F[0] = U[1 + DIR];
#pragma unroll
    for (int k = 0; k < ND; ++k)
      F[1 + k] = k == DIR ? __builtin_fma(PP.gamma - 1.0, ei, U[1 + k] * vn) : U[1 + k] * vn;
    F[ND + 1] = q.ep * vn;
  }
}

template <int ND>
__device__ __forceinline__ void roe_derived(RoeState<ND>& r, double gamma) {
  double q2 = 0.0;
#pragma unroll
  for (int k = 0; k < ND; ++k) q2 += r.vel[k] * r.vel[k];
  r.q2h = 0.5 * q2;
  r.b1 = (gamma - 1.0) * r.ic * r.ic;
  r.b2 = r.q2h * r.b1;
}

template <int ND>
__device__ __forceinline__ RoeState<ND> roe_average(const double* UA, const double* UB,
                                                    double gamma) {
  const Prim<ND> A = primitives<ND, true>(UA, gamma);
  const Prim<ND> B = primitives<ND, true>(UB, gamma);
  const double s = sqrt_pos<true>(UB[0] * A.ir);
  const double wA = rcp<true>(1.0 + s), wB = s * wA;
  RoeState<ND> r;
  double q2 = 0.0;
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    r.vel[k] = wA * A.vel[k] + wB * B.vel[k];
    q2 += r.vel[k] * r.vel[k];
  }
  const double HA = A.ep * A.ir;
  const double HB = B.ep * B.ir;
  r.H = wA * HA + wB * HB;
  r.q2h = 0.5 * q2;
  r.c = sqrt_pos<true>((gamma - 1.0) * (r.H - r.q2h));
  r.ic = rcp<true>(r.c);
  r.b1 = (gamma - 1.0) * r.ic * r.ic;
  r.b2 = r.q2h * r.b1;
  return r;
}

template <int ND, int DIR>
__device__ __forceinline__ void field_row(const RoeState<ND>& r, int v, double (&l)[ND + 2]) {
  if (v == 1) {  // entropy: rho - theta
    l[0] = 1.0 - r.b2;
#pragma unroll
    for (int k = 0; k < ND; ++k) l[1 + k] = r.b1 * r.vel[k];
    l[ND + 1] = -r.b1;
    return;
  }
  // acoustic: (theta +- an) / 2, an = (vel_n rho - m_n) / c
  const double s = (v == 0) ? 0.5 : -0.5;
  const double hb1 = 0.5 * r.b1;
  l[0] = __builtin_fma(s * r.vel[DIR], r.ic, 0.5 * r.b2);
#pragma unroll
  for (int k = 0; k < ND; ++k) l[1 + k] = -hb1 * r.vel[k];
  l[1 + DIR] -= s * r.ic;
  l[ND + 1] = hb1;
}

template <int ND, int DIR>
__device__ __forceinline__ void unproject(const RoeState<ND>& r, const double* W, double* U) {
  const double sum = W[0] + W[1] + W[ND + 1];
  const double dif = W[ND + 1] - W[0];
  U[0] = sum;
  double E = r.H * (W[0] + W[ND + 1]) + r.vel[DIR] * r.c * dif + r.q2h * W[1];
#pragma unroll
  for (int k = 0; k < ND; ++k) U[1 + k] = r.vel[k] * sum;
  U[1 + DIR] += r.c * dif;
#pragma unroll
  for (int t = 0; t < ND - 1; ++t) {
    const int ax = tangential_axis<ND, DIR>(t);
    U[1 + ax] += W[2 + t];
    E += r.vel[ax] * W[2 + t];
  }
  U[ND + 1] = E;
}

// The local Lax-Friedrichs flux itself (llf_flux2 gives twice it).
template <int ND, int DIR>
__device__ __forceinline__ void llf_flux(const double* UL, const double* UR, double gamma,
                                         double* F) {
#pragma clang fp contract(off)
  constexpr int NV = ND + 2;
  const Prim<ND> L = primitives<ND, true>(UL, gamma);
  const Prim<ND> R = primitives<ND, true>(UR, gamma);
  const double cL = sqrt_pos<true>(gamma * L.p * L.ir);
  const double cR = sqrt_pos<true>(gamma * R.p * R.ir);
  const double vL = L.vel[DIR], vR = R.vel[DIR];
  const double lamL = __builtin_fabs(vL) + cL;
  const double lamR = __builtin_fabs(vR) + cR;
  const double ha = 0.5 * __builtin_fmax(lamL, lamR);
  F[0] = UL[1 + DIR] + UR[1 + DIR];
#pragma unroll
  for (int k = 0; k < ND; ++k)
    F[1 + k] = k == DIR ? __builtin_fma(UL[1 + k], vL, L.p) + __builtin_fma(UR[1 + k], vR, R.p)
                        : UL[1 + k] * vL + UR[1 + k] * vR;
  // (which of the two is fused differs between the systems)
  F[ND + 1] = ND == 2 ? __builtin_fma(L.ep, vL, R.ep * vR) : __builtin_fma(R.ep, vR, L.ep * vL);
#pragma unroll
  for (int v = 0; v < NV; ++v) F[v] = __builtin_fma(0.5, F[v], -(ha * (UR[v] - UL[v])));
}

}  // namespace plain
}  // namespace wcns
