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
// E divided by prod_j K_j; Pd, Pa, Pb hold their coefficients, t = E + pd[NT - 2].
template <int NT>
__device__ __forceinline__ double fe_map_poly(double w, double E, double t, const double* pd,
                                              const double* pa, const double* pb, double* den) {
#pragma clang fp contract(off)
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

// The weights of weigh5 applied to eight times the candidates (c0, c1, c2); FE on
// p = 2 Z weights, or FE and PFE from the run-time parameters.  xt: 2^(k/64).
template <bool FE>
__device__ __forceinline__ double weigh5(const InterpParams& P, double c0, double c1, double c2,
                                         double b0, double b1, double b2, const double* xt) {
#pragma clang fp contract(off)
  if constexpr (FE) {
    const double tau = b0 - b2;
    const double t2 = tau * tau;
    const double q0 = b0 * b0, q1 = b1 * b1, q2 = b2 * b2;
    const double s0 = __builtin_fma(b0, b0, t2), p12 = q1 * q2;
    const double s2 = FamWcns::dr2 * __builtin_fma(b2, b2, t2), p01 = q0 * q1;
    const double z0 = s0 * p12;
    const double z1 = (FamWcns::dr1 * __builtin_fma(b1, b1, t2)) * (q0 * q2);
    const double z2 = s2 * p01;
    const double zi = rcp<true>(__builtin_fma(s2, p01, __builtin_fma(s0, p12, z1)));
    const double xi2 = 2.0 * P.xi;
    const double w0 = z0 * zi, w1 = z1 * zi, w2 = z2 * zi;
    // E_0 E_1 E_2 = Ke (the weights sum to one)
    const double zE0 = __builtin_fma(xi2, w0, -P.C2[0]), zE1 = __builtin_fma(xi2, w1, -P.C2[1]);
    const double Ex0 = exp_tab(zE0, xt);
    const double Ex1 = exp_tab(zE1, xt);
    const double r01 = rcp1(Ex0 * Ex1), Ex2 = P.Ke * r01;
    double e0, e1, e2;
    const double n0 = fe_map_poly<3>(w0, Ex0, Ex0 + P.Pd[1], P.Pd, P.Pa, P.Pb, &e0);
    const double n1 = fe_map_poly<4>(w1, Ex1, Ex1 + P.Pd[5], P.Pd + 3, P.Pa + 2, P.Pb + 2, &e1);
    const double n2 = fe_map_poly<3>(w2, Ex2, __builtin_fma(P.Ke, r01, P.Pd[8]), P.Pd + 7,
                                     P.Pa + 5, P.Pb + 5, &e2);
    const double A = n0 * e1, B = n1 * e0, C = n2 * (e0 * e1);
    const double num = __builtin_fma(e2, __builtin_fma(A, c0, B * c1), C * c2);
    return (FamWcns::scale * num) * rcp1(__builtin_fma(e2, __builtin_fma(n0, e1, B), C));
  }
  const double tau = __builtin_fabs(b0 - b2);
  const double q0 = tau * rcp<true>(b0), q1 = tau * rcp<true>(b1), q2 = tau * rcp<true>(b2);
  double p0 = q0, p1 = q1, p2 = q2;
  for (int k = 1; k < P.zpow; ++k) {
    p0 *= q0;
    p1 *= q1;
    p2 *= q2;
  }
  const double a0 = D0 * (1.0 + p0);
  const double a1 = D1 * (1.0 + p1);
  const double a2 = D2 * (1.0 + p2);
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
  return 0.125 * __builtin_fma(w2, c2, __builtin_fma(w0, c0, w1 * c1));
}

template <bool FE>
__device__ __forceinline__ void interp5_pair(const InterpParams& P, const double (&u)[6],
                                             double* left, double* right, const double* xt) {
#pragma clang fp contract(off)
  // candidates of eq. 5 (times 8) of both stencils
  const double c0 = __builtin_fma(15.0, u[2], __builtin_fma(3.0, u[0], -10.0 * u[1]));
  const double c1 = __builtin_fma(3.0, u[3], __builtin_fma(6.0, u[2], -u[1]));
  const double c2 = __builtin_fma(3.0, u[2], 6.0 * u[3]) - u[4];
  const double r0 = __builtin_fma(15.0, u[3], __builtin_fma(3.0, u[5], -10.0 * u[4]));
  const double r1 = __builtin_fma(3.0, u[2], __builtin_fma(6.0, u[3], -u[4]));
  const double r2 = __builtin_fma(6.0, u[2], 3.0 * u[3]) - u[1];
  const double d0 = u[1] - u[0], d1 = u[2] - u[1], d2 = u[3] - u[2], d3 = u[4] - u[3],
               d4 = u[5] - u[4];
  const double s0 = d1 - d0, s1 = d2 - d1, s2 = d3 - d2, s3 = d4 - d3;
  const double q1 = __builtin_fma(s1, s1, P.eps), q2 = __builtin_fma(s2, s2, P.eps);
  const double f0 = 0.5 * __builtin_fma(3.0, d1, -d0), f1 = 0.5 * (d1 + d2),
               f2 = 0.5 * __builtin_fma(3.0, d2, -d3);
  const double g0 = 0.5 * __builtin_fma(3.0, d3, -d4), g1 = 0.5 * (d2 + d3),
               g2 = 0.5 * (FE ? __builtin_fma(3.0, d2, -d1) : 3.0 * d2 - d1);
  *left = weigh5<FE>(P, c0, c1, c2, __builtin_fma(f0, f0, __builtin_fma(s0, s0, P.eps)),
                     __builtin_fma(f1, f1, q1), __builtin_fma(f2, f2, q2), xt);
  *right = weigh5<FE>(P, r0, r1, r2, __builtin_fma(g0, g0, __builtin_fma(s3, s3, P.eps)),
                      __builtin_fma(g1, g1, q2), __builtin_fma(g2, g2, q1), xt);
}

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

// (c from the unrounded |u|^2 / 2)
template <int ND>
__device__ __forceinline__ RoeState<ND> roe_average(const double* UA, const double* UB,
                                                    double gamma) {
#pragma clang fp contract(off)
  const Prim<ND> A = primitives<ND, true>(UA, gamma);
  const Prim<ND> B = primitives<ND, true>(UB, gamma);
  const double s = sqrt_pos<true>(UB[0] * A.ir);
  const double wA = rcp<true>(1.0 + s), wB = s * wA;
  RoeState<ND> r;
#pragma unroll
  for (int k = 0; k < ND; ++k) r.vel[k] = __builtin_fma(wA, A.vel[k], wB * B.vel[k]);
  const double HA = A.ep * A.ir;
  const double HB = B.ep * B.ir;
  r.H = __builtin_fma(wA, HA, wB * HB);
  const double q2 = norm2<ND>(r.vel);
  r.q2h = 0.5 * q2;
  r.c = sqrt_pos<true>((gamma - 1.0) * __builtin_fma(-0.5, q2, r.H));
  r.ic = rcp<true>(r.c);
  r.b1 = (gamma - 1.0) * r.ic * r.ic;
  r.b2 = r.q2h * r.b1;
  return r;
}

template <int ND, int DIR>
__device__ __forceinline__ void field_row(const RoeState<ND>& r, int v, double (&l)[ND + 2]) {
#pragma clang fp contract(off)
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
  for (int k = 0; k < ND; ++k)
    l[1 + k] = k == DIR ? __builtin_fma(-hb1, r.vel[k], -(s * r.ic)) : -hb1 * r.vel[k];
  l[ND + 1] = hb1;
}

template <int ND, int DIR>
__device__ __forceinline__ void unproject(const RoeState<ND>& r, const double* W, double* U) {
#pragma clang fp contract(off)
  const double sum = W[0] + W[1] + W[ND + 1];
  const double dif = W[ND + 1] - W[0];
  U[0] = sum;
  const double cv = r.vel[DIR] * r.c;
  double E = __builtin_fma(r.q2h, W[1], __builtin_fma(r.H, W[0] + W[ND + 1], cv * dif));
  U[1 + DIR] = __builtin_fma(r.vel[DIR], sum, r.c * dif);
#pragma unroll
  for (int t = 0; t < ND - 1; ++t) {
    const int ax = tangential_axis<ND, DIR>(t);
    U[1 + ax] = __builtin_fma(r.vel[ax], sum, W[2 + t]);
    E = __builtin_fma(r.vel[ax], W[2 + t], E);
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

// The upwind flux (not twice it).
__device__ __forceinline__ double advection_flux(double adv, double uL, double uR) {
#pragma clang fp contract(off)
  return __builtin_fma(0.5 * adv, uL + uR, -((0.5 * __builtin_fabs(adv)) * (uR - uL)));
}

// The MND6 and MD6 differences of the midpoint fluxes f and the node fluxes nf, W apart.
template <int W, class F>
__device__ __forceinline__ double diff_mnd6(F f, F nf) {
#pragma clang fp contract(off)
  return __builtin_fma(1.0 / 30.0, f[3 * W] - f[0],
                       __builtin_fma(1.5, f[2 * W] - f[W], -0.3 * (nf[3 * W] - nf[W])));
}
template <int W, class F>
__device__ __forceinline__ double diff_md6(F f) {
#pragma clang fp contract(off)
  return __builtin_fma(3.0 / 640.0, f[5 * W] - f[0],
                       __builtin_fma(75.0 / 64.0, f[3 * W] - f[2 * W], (-25.0 / 384.0) * (f[4 * W] - f[W])));
}

}  // namespace plain
}  // namespace wcns
