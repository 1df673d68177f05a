// Reverse-mode (vector-Jacobian) versions of the device arithmetic in
// wcns_device.hpp, written by hand.  Each *_vjp recomputes the forward
// intermediates it needs and propagates a cotangent backwards through them.
// Conventions at non-smooth points: d|x|/dx = 0 at x = 0; the tie in
// max(a, b) goes to the first argument; the PFE switch differentiates the
// branch it takes.
#pragma once

#include "wcns_device.hpp"

namespace wcns {

// g_i(w) and g_i'(w) of eq. 20 (see fe_map; d tanh = 1 - tanh^2, exactly 0
// where tanh saturates to +-1).
template <int SPEC>
__device__ __forceinline__ double fe_g_d(int i, double w, const InterpParams& P, double* dg) {
  if (i == 0) return fe_g0<SPEC>(w, P, dg);
  if (i == 1) return fe_g1<SPEC>(w, P, dg);
  return fe_g2<SPEC>(w, P, dg);
}

// One map's g(w) and g'(w) on the forward fast path's variable X (see
// fe_map_poly), given v_j = 1 / (X + k_j): with i_j = k_j v_j and 1 - i_j =
// X v_j (the third map: i_j = X v_j, 1 - i_j = k_j v_j),
//   g = w - 2 sum_j A_j i_j,  g' = 1 - 2 sum_j b_j i_j + 4 xi sum_j A_j i_j (1 - i_j),
// term by term, so that a saturated g' keeps its relative accuracy.
template <int NT, bool THIRD>
__device__ __forceinline__ double fe_map_slope(double w, double X, const double (&v)[NT],
                                               const double* k, const double (&a)[NT],
                                               const double (&b)[NT], double xi2, double* slope) {
  double g = w, s = 1.0, t = 0.0;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const double kv = k[j] * v[j];
    const double i = THIRD ? X * v[j] : kv;
    const double p = (b[j] == 0.0 ? -2.0 * a[j] : __builtin_fma(-2.0 * b[j], w, -2.0 * a[j])) * i;
    g += p;
    if (b[j] != 0.0) s = __builtin_fma(-2.0 * b[j], i, s);
    const double o = THIRD ? kv : v[j];
    t = j == 0 ? p * o : __builtin_fma(p, o, t);
  }
  *slope = __builtin_fma(THIRD ? -xi2 : -xi2 * X, t, s);
  return g;
}

// The weights W_k and the cotangents bb_k of the regularised indicators b_k =
// IS_k + eps for the output (1/8) sum_k W_k x_k (x_k: the candidates'
// distances from the middle node, see weigh5): FE weights on p = 2 Z weights
// through the forward fast path's variables.  With alpha_k = d_k (1 + tau^2 /
// b_k^2) the Z weights' cotangents need 1 / b_k, one reciprocal of b_0 b_1 b_2
// (at least eps^3 = 1e-120) for all three; the three maps' reciprocals are one
// of the product of their denominators.
__device__ __forceinline__ void fe_weights_grad(const InterpParams& P, const double (&x)[3],
                                                const double (&b)[3], double (&W)[3],
                                                double (&bb)[3], const double* xt) {
#pragma clang fp contract(off)
  constexpr double dr[3] = {1.0, FamWcns::dr1, FamWcns::dr2};
  const double tau = b[0] - b[2], t2 = tau * tau;
  const double m[3] = {b[1] * b[2], b[0] * b[2], b[0] * b[1]};
  const double B = b[0] * m[0];
  const double PP = B * B;
  const double p[3] = {m[0] * m[0], m[1] * m[1], m[2] * m[2]};
  const double z0 = __builtin_fma(t2, p[0], PP), z1 = dr[1] * __builtin_fma(t2, p[1], PP),
               z2 = dr[2] * __builtin_fma(t2, p[2], PP);
  const double zi = rcp(z0 + z1 + z2);
  const double w[3] = {z0 * zi, z1 * zi, z2 * zi};
  const double X0 = exp2_tab(w[0], P.xa, xt), X1 = exp2_tab(w[1], P.xa, xt), X2 = X0 * X1;
  double y[10];
#pragma unroll
  for (int j = 0; j < 10; ++j) y[j] = (j < 3 ? X0 : j < 7 ? X1 : X2) + P.kap[j];
  const double a01 = y[0] * y[1], c01 = y[3] * y[4], c23 = y[5] * y[6], f01 = y[7] * y[8];
  const double e0 = a01 * y[2], e1 = c01 * c23, e2 = f01 * y[9];
  // one Newton step suffices where the error stays in proportion (as in weigh5)
  const double e01 = e0 * e1;
  const double r = rcp1(e01 * e2);
  const double r2 = r * e01, re2 = r * e2;
  const double r0 = re2 * e1, r1 = re2 * e0;
  const double v0[3] = {(y[1] * y[2]) * r0, (y[0] * y[2]) * r0, a01 * r0};
  const double c23r = c23 * r1, c01r = c01 * r1;
  const double v1[4] = {y[4] * c23r, y[3] * c23r, y[6] * c01r, y[5] * c01r};
  const double v2[3] = {(y[8] * y[9]) * r2, (y[7] * y[9]) * r2, f01 * r2};
  const double xi2 = 2.0 * P.xi;
  double s[3];
  const double g0 = fe_map_slope<3, false>(w[0], X0, v0, P.kap, kG0a, kG0b, xi2, &s[0]);
  const double g1 = fe_map_slope<4, false>(w[1], X1, v1, P.kap + 3, kG1a, kG1b, xi2, &s[1]);
  const double g2 = fe_map_slope<3, true>(w[2], X2, v2, P.kap + 7, kG2a, kG2b, xi2, &s[2]);
  const double gi = rcp1(g0 + g1 + g2);
  W[0] = g0 * gi;
  W[1] = g1 * gi;
  W[2] = g2 * gi;
  // W = g / sum g, then w = z / sum z
  const double mean = __builtin_fma(W[0], x[0], __builtin_fma(W[1], x[1], W[2] * x[2]));
  const double gi8 = 0.125 * gi;
  double h[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) h[k] = (x[k] - mean) * (s[k] * gi8);
  const double hm = __builtin_fma(h[0], w[0], __builtin_fma(h[1], w[1], h[2] * w[2]));
  // d w_k = (d_k / sum z) (p_k d tau^2 - 2 tau^2 p_k / b_k d b_k), up to a
  // part along w that the mean takes out
  const double iB = rcp(B), n2 = -2.0 * t2 * iB;
  double u[3], c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    u[k] = (h[k] - hm) * ((dr[k] * zi) * p[k]);
    c[k] = n2 * m[k];
  }
  const double tb = 2.0 * tau * (u[0] + u[1] + u[2]);
  bb[0] = __builtin_fma(c[0], u[0], tb);
  bb[1] = c[1] * u[1];
  bb[2] = __builtin_fma(c[2], u[2], -tb);
}

// The same for every other choice of weights (runtime parameters).
template <int SPEC>
__device__ __forceinline__ void weights_grad(const InterpParams& P, const double (&x)[3],
                                             const double (&b)[3], double (&W)[3],
                                             double (&bb)[3], const double* xt) {
  if constexpr (SPEC == SPEC_FE) {
    fe_weights_grad(P, x, b, W, bb, xt);
    return;
  }
  constexpr double d[3] = {D0, D1, D2};
  if (P.weights == WLIN) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      W[k] = d[k];
      bb[k] = 0.0;
    }
    return;
  }
  const bool js = P.weights == WJS;
  const double tau = b[0] - b[2], at = __builtin_fabs(tau);
  double r[3], q[3], dq[3], z[3];  // 1 / b, tau / b, d alpha / d q (Z), weights
  double sum = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    r[k] = rcp(b[k]);
    if (js) {
      z[k] = d[k] * r[k] * r[k];
    } else {
      q[k] = at * r[k];
      double pw = q[k];
      dq[k] = d[k] * P.zpow;
      for (int i = 1; i < P.zpow; ++i) {
        dq[k] *= q[k];
        pw *= q[k];
      }
      z[k] = d[k] * (1.0 + pw);
    }
    sum += z[k];
  }
  const double inv = rcp(sum);
#pragma unroll
  for (int k = 0; k < 3; ++k) z[k] *= inv;
  bool map = P.weights == WFE;
  if (P.weights == WPFE)
    map = !(__builtin_fabs(z[0] - D0) <= P.cv && __builtin_fabs(z[1] - D1) <= P.cv &&
            __builtin_fabs(z[2] - D2) <= P.cv);
  double s[3] = {1.0, 1.0, 1.0}, gi = 1.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) W[k] = z[k];
  if (map) {
#pragma unroll
    for (int k = 0; k < 3; ++k) W[k] = fe_g_d<SPEC>(k, z[k], P, &s[k]);
    gi = rcp(W[0] + W[1] + W[2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) W[k] *= gi;
  }
  const double mean = W[0] * x[0] + W[1] * x[1] + W[2] * x[2];
  double h[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) h[k] = 0.125 * (x[k] - mean) * gi * s[k];
  const double hm = h[0] * z[0] + h[1] * z[1] + h[2] * z[2];
  double tb = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double ab = (h[k] - hm) * inv;
    if (js) {  // alpha = d / b^2
      bb[k] = -2.0 * d[k] * r[k] * r[k] * r[k] * ab;
    } else {   // alpha = d (1 + q^p), q = |tau| / b
      const double qb = ab * dq[k];
      bb[k] = -qb * at * r[k] * r[k];
      tb += qb * r[k];
    }
  }
  if (!js) {
    tb *= tau > 0.0 ? 1.0 : (tau < 0.0 ? -1.0 : 0.0);
    bb[0] += tb;
    bb[2] -= tb;
  }
}

// One nonlinear interpolation from the value um of the stencil's middle node,
// the slopes f_k and second differences s_k of its three parabolas
// (interp5_pair), and its gradient G[i] = d / d d_i (at fixed um) for the
// stencil's first differences d_0 .. d_3.  Value and gradient come from the
// same intermediates, so the adjoint needs no second evaluation of the
// weights, and four numbers carry the gradient from this phase to the next.
template <int SPEC>
__device__ __forceinline__ double interp5_side(const InterpParams& P, double um,
                                               const double (&f)[3], const double (&s)[3],
                                               double (&G)[4], const double* xt) {
  double x[3], b[3], W[3], bb[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    x[k] = __builtin_fma(4.0, f[k], s[k]);
    b[k] = __builtin_fma(f[k], f[k], __builtin_fma(s[k], s[k], P.eps));
  }
  weights_grad<SPEC>(P, x, b, W, bb, xt);
  // x_k = 4 f_k + s_k, b_k = f_k^2 + s_k^2; f_0 = d_1 + s_0 / 2, f_1 = d_1 +
  // s_1 / 2, f_2 = d_2 - s_2 / 2; s_k = d_{k+1} - d_k
  double fb[3], sb[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double t = bb[k] + bb[k];
    fb[k] = __builtin_fma(f[k], t, 0.5 * W[k]);
    sb[k] = __builtin_fma(s[k], t, 0.125 * W[k]);
  }
  sb[0] = __builtin_fma(0.5, fb[0], sb[0]);
  sb[1] = __builtin_fma(0.5, fb[1], sb[1]);
  sb[2] = __builtin_fma(-0.5, fb[2], sb[2]);
  G[0] = -sb[0];
  G[1] = fb[0] + fb[1] + sb[0] - sb[1];
  G[2] = fb[2] + sb[1] - sb[2];
  G[3] = sb[2];
  return __builtin_fma(0.125,
                       __builtin_fma(W[0], x[0], __builtin_fma(W[1], x[1], W[2] * x[2])), um);
}

// The left-biased interpolation of the stencil (u_0 .. u_4) and its gradient;
// of the mirrored stencil (u_5 .. u_1), the right-biased one.
template <int SPEC>
__device__ __forceinline__ double interp5_grad_one(const InterpParams& P, const double (&u)[5],
                                                   double (&G)[4], const double* xt) {
  const double d0 = u[1] - u[0], d1 = u[2] - u[1], d2 = u[3] - u[2], d3 = u[4] - u[3];
  const double s[3] = {d1 - d0, d2 - d1, d3 - d2};
  const double f[3] = {__builtin_fma(0.5, s[0], d1), __builtin_fma(0.5, s[1], d1),
                       __builtin_fma(-0.5, s[2], d2)};
  return interp5_side<SPEC>(P, u[2], f, s, G, xt);
}

// Both interpolations of one field (interp5_pair) with their gradients, GL of
// u_1 - u_0 .. u_4 - u_3 and GR of the mirrored stencil's differences u_4 -
// u_5, u_3 - u_4, u_2 - u_3, u_1 - u_2.
template <int SPEC>
__device__ __forceinline__ void interp5_grad(const InterpParams& P, const double (&u)[6],
                                             double* left, double* right, double (&GL)[4],
                                             double (&GR)[4], const double* xt) {
  const double d0 = u[1] - u[0], d1 = u[2] - u[1], d2 = u[3] - u[2], d3 = u[4] - u[3],
               d4 = u[5] - u[4];
  const double s0 = d1 - d0, s1 = d2 - d1, s2 = d3 - d2, s3 = d4 - d3;
  {
    const double f[3] = {__builtin_fma(0.5, s0, d1), __builtin_fma(0.5, s1, d1),
                         __builtin_fma(-0.5, s2, d2)};
    const double s[3] = {s0, s1, s2};
    *left = interp5_side<SPEC>(P, u[2], f, s, GL, xt);
  }
  {
    const double f[3] = {__builtin_fma(0.5, s3, -d3), __builtin_fma(0.5, s2, -d3),
                         __builtin_fma(-0.5, s1, -d2)};
    const double s[3] = {s3, s2, s1};
    *right = interp5_side<SPEC>(P, u[3], f, s, GR, xt);
  }
}

// Cotangents of the six stencil values from those of the two interpolated
// ones (yl, yr) and interp5_grad's gradients.
__device__ __forceinline__ void interp5_vjp(double yl, double yr, const double (&GL)[4],
                                            const double (&GR)[4], double (&wb)[6]) {
  const double D0 = yl * GL[0], D4 = -yr * GR[0];
  const double D1 = __builtin_fma(yl, GL[1], -yr * GR[3]);
  const double D2 = __builtin_fma(yl, GL[2], -yr * GR[2]);
  const double D3 = __builtin_fma(yl, GL[3], -yr * GR[1]);
  wb[0] = -D0;
  wb[1] = D0 - D1;
  wb[2] = yl + (D1 - D2);
  wb[3] = yr + (D2 - D3);
  wb[4] = D3 - D4;
  wb[5] = D4;
}

// Ub += (dF/dU)^T Fb + (d lam/dU)^T lamb for the Euler flux along DIR and the
// wave speed lam = |u_n| + c of one state with primitives q.  c is used only
// where lamb != 0.
template <int ND, int DIR>
__device__ __forceinline__ void flux_speed_vjp(const double* U, const Prim<ND>& q, double gamma,
                                               double c, const double* Fb, double lamb,
                                               double* Ub) {
  const double vn = q.vel[DIR];
  double vnb = Fb[ND + 1] * q.ep;
#pragma unroll
  for (int k = 0; k < ND; ++k) vnb = __builtin_fma(Fb[1 + k], U[1 + k], vnb);
  const double Eb = Fb[ND + 1] * vn;
  double pb = Fb[1 + DIR] + Eb;
  double irb = 0.0;  // what the wave speed adds to the cotangent of 1 / rho, times 1 / rho
  if (lamb != 0.0) {
    vnb += lamb * (vn > 0.0 ? 1.0 : (vn < 0.0 ? -1.0 : 0.0));
    const double t = 0.5 * lamb * rcp(c) * gamma * q.ir;  // c^2 = gamma p / rho
    pb += t;
    irb = t * q.p;
  }
  // p = (gamma - 1)(E - |m|^2 / (2 rho)), vel = m / rho
  const double h = (gamma - 1.0) * pb;
  const double vi = vnb * q.ir;
  Ub[0] += 0.5 * h * norm2<ND>(q.vel) - __builtin_fma(vi, vn, irb * q.ir);
#pragma unroll
  for (int k = 0; k < ND; ++k)
    Ub[1 + k] += __builtin_fma(Fb[1 + k], vn, -h * q.vel[k]) + (k == DIR ? Fb[0] + vi : 0.0);
  Ub[ND + 1] += Eb + h;
}

// Cotangent of the Roe-averaged quantities that the back-projection reads.
template <int ND>
struct RoeSideBar {
  double vel[ND];
  double H, c, q2h;
};
// and of all of them.
template <int ND>
struct RoeBar {
  double vel[ND];
  double H, c, ic, q2h, b1, b2;
};

// Propagates rb back to the two node states: UbA, UbB = its parts.  With s =
// sqrt(rho_B / rho_A), w_A = 1 / (1 + s) and w_B = 1 - w_A, an average w_A a +
// w_B b has d w_A = -w_A^2 ds times (a - b).
template <int ND>
__device__ __forceinline__ void roe_vjp(const double* UA, const double* UB, double gamma,
                                        const RoeState<ND>& r, RoeBar<ND> rb, double* UbA,
                                        double* UbB) {
  // b2 = q2h b1 ; b1 = (g-1) ic^2 ; ic = 1/c
  rb.q2h += rb.b2 * r.b1;
  rb.b1 += rb.b2 * r.q2h;
  rb.ic += rb.b1 * 2.0 * (gamma - 1.0) * r.ic;
  rb.c += -rb.ic * r.ic * r.ic;
  // c = sqrt((g-1)(H - q2h))
  const double Yb = rb.c * 0.5 * r.ic * (gamma - 1.0);
  rb.H += Yb;
  rb.q2h -= Yb;
#pragma unroll
  for (int k = 0; k < ND; ++k) rb.vel[k] += rb.q2h * r.vel[k];
  const Prim<ND> A = primitives<ND>(UA, gamma);
  const Prim<ND> B = primitives<ND>(UB, gamma);
  const double s = sqrt_pos(UB[0] * A.ir);
  const double wA = rcp(1.0 + s), wB = s * wA;
  const double HA = A.ep * A.ir;
  const double HB = B.ep * B.ir;
  double wb = rb.H * (HA - HB);
#pragma unroll
  for (int k = 0; k < ND; ++k) wb = __builtin_fma(rb.vel[k], A.vel[k] - B.vel[k], wb);
  const double sb = -0.5 * wb * wA * wB;  // s / 2 times the cotangent of s
  // H = (E + p) / rho, vel = m / rho, p = (g-1)(E - |m|^2 / (2 rho))
  auto node = [&](const Prim<ND>& q, double H, double w, double rb0, double* Ub) {
    const double Hb = rb.H * w, pb = Hb * q.ir, h = (gamma - 1.0) * pb;
    double t = Hb * H;
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      const double vb = rb.vel[k] * w;
      t = __builtin_fma(vb, q.vel[k], t);
      Ub[1 + k] = __builtin_fma(vb, q.ir, -h * q.vel[k]);
    }
    Ub[0] = __builtin_fma(0.5 * h, norm2<ND>(q.vel), q.ir * (rb0 - t));
    Ub[ND + 1] = pb + h;
  };
  node(A, HA, wA, -sb, UbA);
  node(B, HB, wB, sb, UbB);
}

// Local Lax-Friedrichs flux F = (F(UL) + F(UR)) / 2 - alpha (UR - UL) / 2,
// alpha = max(lam(UL), lam(UR)): Ub = (dF/dU)^T Fb of the left (SIDE = 0) or
// the right state.
template <int ND, int DIR, int SIDE>
__device__ __forceinline__ void llf_vjp(const double* UL, const double* UR, double gamma,
                                        const double* Fb, double* Ub) {
  constexpr int NV = ND + 2;
  const Prim<ND> L = primitives<ND>(UL, gamma);
  const Prim<ND> R = primitives<ND>(UR, gamma);
  const double cL = sqrt_pos(gamma * L.p * L.ir), cR = sqrt_pos(gamma * R.p * R.ir);
  const double lamL = __builtin_fabs(L.vel[DIR]) + cL;
  const double lamR = __builtin_fabs(R.vel[DIR]) + cR;
  const bool takeL = lamL >= lamR;
  const double alpha = takeL ? lamL : lamR;
  const bool take = takeL == (SIDE == 0);
  double alphab = 0.0, Fh[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    alphab = __builtin_fma(-0.5 * (UR[v] - UL[v]), Fb[v], alphab);
    Fh[v] = 0.5 * Fb[v];
    Ub[v] = (SIDE == 0 ? alpha : -alpha) * Fh[v];
  }
  flux_speed_vjp<ND, DIR>(SIDE == 0 ? UL : UR, SIDE == 0 ? L : R, gamma, SIDE == 0 ? cL : cR, Fh,
                          take ? alphab : 0.0, Ub);
}

// Back-projection U = R W (see unproject): Wb = R^T Ub, and rb the cotangent
// of the Roe quantities R depends on.
template <int ND, int DIR>
__device__ __forceinline__ void unproject_vjp(const RoeState<ND>& r, const double* W,
                                              const double* Ub, double* Wb, RoeSideBar<ND>& rb) {
  const double ac = W[0] + W[ND + 1];
  const double sum = ac + W[1];
  const double dif = W[ND + 1] - W[0];
  const double Eb = Ub[ND + 1];
  double sumb = Ub[0];
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    rb.vel[k] = Ub[1 + k] * sum;
    sumb = __builtin_fma(Ub[1 + k], r.vel[k], sumb);
  }
  // U_n = vel_n sum + c dif, E = H ac + vel_n c dif + q2h W_1 + vel_t W_t
  const double cdb = __builtin_fma(Eb, r.vel[DIR], Ub[1 + DIR]);  // cotangent of c dif
  rb.vel[DIR] = __builtin_fma(Eb * r.c, dif, rb.vel[DIR]);
  rb.c = cdb * dif;
  rb.H = Eb * ac;
  rb.q2h = Eb * W[1];
  const double acb = __builtin_fma(Eb, r.H, sumb);
  const double difb = cdb * r.c;
  Wb[0] = acb - difb;
  Wb[ND + 1] = acb + difb;
  Wb[1] = __builtin_fma(Eb, r.q2h, sumb);
#pragma unroll
  for (int t = 0; t < ND - 1; ++t) {
    const int ax = tangential_axis<ND, DIR>(t);
    Wb[2 + t] = __builtin_fma(Eb, r.vel[ax], Ub[1 + ax]);
    rb.vel[ax] = __builtin_fma(Eb, W[2 + t], rb.vel[ax]);
  }
}

// Projection W = L U of one node (see project): Ub = L^T Wb.
template <int ND, int DIR>
__device__ __forceinline__ void project_vjp(const RoeState<ND>& r, const double* Wb, double* Ub) {
  const double thb = __builtin_fma(0.5, Wb[0] + Wb[ND + 1], -Wb[1]);
  const double ai = 0.5 * (Wb[0] - Wb[ND + 1]) * r.ic;
  const double t1 = thb * r.b1;
  double rho = __builtin_fma(ai, r.vel[DIR], __builtin_fma(thb, r.b2, Wb[1]));
  Ub[1 + DIR] = __builtin_fma(-t1, r.vel[DIR], -ai);
#pragma unroll
  for (int t = 0; t < ND - 1; ++t) {
    const int ax = tangential_axis<ND, DIR>(t);
    rho = __builtin_fma(-Wb[2 + t], r.vel[ax], rho);
    Ub[1 + ax] = __builtin_fma(-t1, r.vel[ax], Wb[2 + t]);
  }
  Ub[0] = rho;
  Ub[ND + 1] = t1;
}

// The cotangent of the Roe quantities that the projections of the six
// stencil nodes give, from the moments T[e] = sum_j thb_j U_j[e], A0, An =
// sum_j anb_j rho_j, m_n,j (thb = (Wb_0 + Wb_{ND+1}) / 2 - Wb_1, anb = (Wb_0 -
// Wb_{ND+1}) / 2) and S[t] = sum_j Wb_{2+t},j rho_j: added to rb.
template <int ND, int DIR>
__device__ __forceinline__ void project_roe_bar(const RoeState<ND>& r, const double* T, double A0,
                                                double An, const double* S, RoeBar<ND>& rb) {
  rb.vel[DIR] = __builtin_fma(r.ic, A0, rb.vel[DIR]);
  rb.ic += __builtin_fma(r.vel[DIR], A0, -An);
  rb.b2 += T[0];
  double t = T[ND + 1];
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    t = __builtin_fma(-r.vel[k], T[1 + k], t);
    rb.vel[k] = __builtin_fma(-r.b1, T[1 + k], rb.vel[k]);
  }
  rb.b1 += t;
#pragma unroll
  for (int k = 0; k < ND - 1; ++k) rb.vel[tangential_axis<ND, DIR>(k)] -= S[k];
}

// Component e (uniform) of (dF/dU)^T Fb for the physical flux at a node.
template <int NV, int DIR>
__device__ __forceinline__ double node_flux_vjp(const PhysParams& PP, const double (&U)[NV],
                                                const double (&Fb)[NV], int e) {
  if constexpr (NV == 1) {
    return PP.adv * Fb[0];
  } else {
    constexpr int ND = NV - 2;
    double Ub[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) Ub[v] = 0.0;
    flux_speed_vjp<ND, DIR>(U, primitives<ND>(U, PP.gamma), PP.gamma, 0.0, Fb, 0.0, Ub);
    double x = Ub[0];
#pragma unroll
    for (int v = 1; v < NV; ++v) x = e == v ? Ub[v] : x;
    return x;
  }
}

}  // namespace wcns
