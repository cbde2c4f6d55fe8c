// Collision of the isothermal (BGK) kernels, D2Q9 and D3Q27.
#pragma once

#include "device_common.h"

#include <type_traits>

namespace lbm {

// Psi(c; u, theta + u^2) for c = -1, 0, +1 at theta = 1/3 (Sec. II C).
__device__ __forceinline__ void psi3(double u, double (&p)[3]) {
  const double u2 = u * u;
  p[1] = (2.0 / 3.0) - u2;               // c = 0:  1 - theta - u^2
  p[2] = (1.0 / 6.0) + 0.5 * (u2 + u);   // c = +1: (theta + u^2 + u) / 2
  p[0] = (1.0 / 6.0) + 0.5 * (u2 - u);   // c = -1: (theta + u^2 - u) / 2
}

// Rest weights w_i = prod_a Psi(c_ia; 0, 1/3) as a function of the per-axis index k = c + 1.
__device__ __forceinline__ double w1(int k) { return k == 1 ? 2.0 / 3.0 : 1.0 / 6.0; }

// Moments of one node for the diagnostics: rho, rho u (with the half-step force term) and u.
struct NodeMoments {
  double rho, j[3], u[3];
};

// Collision of one node held shifted (h = f - w), Eq. (LBM_f) at theta = 1/3 (Phi = 0):
//   rho = sum f, rho u = sum c f + F/2,
//   f~ = f + omega (f^eq - f) + (1 - omega/2)(f^* - f^eq),
// where f^* is the equilibrium at u* = u + F/rho (Sec. II C; no heat source, theta* = theta).
// Without a force (FORCE = false) f^* = f^eq. `sink(i, h~_i)` receives the post-collision
// values in storage precision. D2Q9 and D3Q27 (D = 2, 3; i = (cx+1) + 3(cy+1) + 9(cz+1)).
template <int D, bool FORCE, typename S, typename Sink>
__device__ __forceinline__ void collide_bgk(const S (&hs)[D == 2 ? 9 : 27], double omega,
                                            const Force& F, NodeMoments& m, Sink&& sink) {
  constexpr int Q = D == 2 ? 9 : 27;
  double rho, j[3] = {0.0, 0.0, 0.0};
  if (D == 2) {
    double h[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) h[i] = (double)hs[i];
    // sum w_i = 1 and sum c_i w_i = 0, so rho = 1 + sum h and rho u = sum c h
    rho = 1.0 + (((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7])) + h[8]);
    j[0] = (h[2] + h[5] + h[8]) - (h[0] + h[3] + h[6]);
    j[1] = (h[6] + h[7] + h[8]) - (h[0] + h[1] + h[2]);
  } else {
    double drho = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int cx = i % 3 - 1, cy = (i / 3) % 3 - 1, cz = i / 9 - 1;
      const double v = (double)hs[i];
      drho += v;
      if (cx) j[0] += cx > 0 ? v : -v;
      if (cy) j[1] += cy > 0 ? v : -v;
      if (cz) j[2] += cz > 0 ? v : -v;
    }
    rho = 1.0 + drho;
  }
  if (FORCE) {
    j[0] += 0.5 * F.x;
    j[1] += 0.5 * F.y;
    if (D == 3) j[2] += 0.5 * F.z;
  }
  const Reciprocal inv(rho);
  double p[3][3], ps[3][3];
#pragma unroll
  for (int a = 0; a < D; ++a) {
    m.u[a] = inv.quotient(j[a]);
    psi3(m.u[a], p[a]);
  }
  if (FORCE) {
    const double fa[3] = {F.x, F.y, F.z};
#pragma unroll
    for (int a = 0; a < D; ++a) psi3(m.u[a] + inv.quotient(fa[a]), ps[a]);
  }
  const double keep = 1.0 - 0.5 * omega;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const int a = i % 3, b = (i / 3) % 3, c = i / 9;
    // rho p_a p_b (p_c), multiplied left to right so that rho p_a is shared between directions
    double feq = rho * p[0][a] * p[1][b];
    double ww = w1(a) * w1(b);
    if (D == 3) {
      feq *= p[2][c];
      ww *= w1(c);
    }
    const double heq = feq - ww;
    const double v = (double)hs[i];
    double out = v + omega * (heq - v);
    if (FORCE) {
      double fs = rho * ps[0][a] * ps[1][b];
      if (D == 3) fs *= ps[2][c];
      out += keep * (fs - feq);
    }
    sink(i, (S)out);
  }
  m.rho = rho;
#pragma unroll
  for (int a = 0; a < 3; ++a) m.j[a] = a < D ? j[a] : 0.0;
}

template <int D>
__device__ __forceinline__ void add_diag(double (&acc)[kDiagValues], const NodeMoments& m) {
  acc[0] += m.rho;
  acc[1] += m.j[0];
  acc[2] += m.j[1];
  if (D == 3) acc[3] += m.j[2];
  double u2 = m.u[0] * m.u[0] + m.u[1] * m.u[1];
  if (D == 3) u2 += m.u[2] * m.u[2];
  acc[4] += 0.5 * m.rho * u2;
}

// Calls fn(std::integral_constant<bool, b>{}): turns a run-time flag into a template argument.
template <typename Fn>
static void with_flag(bool b, Fn&& fn) {
  if (b)
    fn(std::true_type{});
  else
    fn(std::false_type{});
}

}  // namespace lbm
