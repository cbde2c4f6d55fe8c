// Double distribution, D2Q9: two time steps per launch (float32 storage, central Phi or none; every
// collision and wall type of k_ddf_d2q9, whose scheme and storage this shares).
//
// The one-step kernel moves 144 bytes per node and step and re-reads the halo rows of its four-row
// windows (1.33 x the reads): at 4096^2 it is bound by that traffic, its vector units 39% busy.
// Here a workgroup of 256 columns walks a tall window bottom to top and takes every row through
// both steps: the first step's rows go through LDS to the second one, 75 bytes per node and step
// from memory and no row of the window read twice (three halo rows each way, of about 137 at
// 4096^2). Measured on MI355X, us per step, one step -> two per launch: 4096^2 with walls 562 -> 324
// to 355, with force and heat source 582 -> 435, Pr 0.71 601 -> 450, NEQ walls 561 -> 365; 2048^2 plain
// 143 -> 89 to 103, force and heat source 167 -> 117, Pr 0.71 with NEQ walls 177 -> 127, van der Waals
// 194 -> 137; 1021 x 509 Pr 0.71 with NEQ walls 30.6 -> 27.7. Where it is taken: routes.h.
//
// One iteration, row r, one barrier:
//   gather   first step: row r (loaded during the iteration before), its moments; second step:
//            row r - 4, its populations from the first step's rows r - 3, r - 4, r - 5 (their
//            neighbours' columns read from s_row, the populations moving up kept for one and two
//            iterations), its moments;
//   barrier  orders the exchanged moments and, an iteration later, the rows in s_row (two
//            buffers each, by the parity of the iteration);
//   collide  first step: row r - 1, into s_row; second step: row r - 5, to memory.
// A row waits one iteration between gather and collision for its y derivatives: the first step's in
// s_wait, the second step's in registers. Two wavefronts per SIMD for the plain collision (255
// registers and 76 KB of LDS per workgroup without spills), one for the others. The rebuilt rows of
// the NEQ walls come from their neighbour row as it passes (row 0 one iteration late).
// The state between the steps is rounded to float32 like a stored one and the arithmetic rounds like
// the one-step kernel's, so the results are those of two launches of it, bit for bit.
#include "ddf_common.h"
#include "routes.h"

#include <type_traits>

namespace lbm {

template <typename S, int WALLS, int EXT>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(EXT == 0 && WALLS != 2 ? 2 : 1)))
k_ddf_pair(const S* __restrict__ A, S* __restrict__ B, int nx, int ny, int64_t pitch,
           int64_t plane, DdfParams prm, int rows, int nbx) {
  constexpr bool X = EXT > 0, VDW = EXT == 2, NEQ = WALLS == 2;
  constexpr int NM = X ? (VDW ? 9 : 8) : 6;
  constexpr int NX = X ? (VDW ? 4 : 3) : 1;  // values exchanged along x: phi_x [, T, u_x [, h]]
  __shared__ double s_x[2][2][NX][kBlock];   // [step][parity]
  __shared__ double s_wall[NEQ ? 2 : 1][NX][NEQ ? kBlock : 1];
  __shared__ S s_row[2][18][kBlock];         // rows after the first step, by parity
  __shared__ S s_wait[18][kBlock];           // the first step's row that waits for its collision
  __shared__ S s_up[2][6][kBlock];           // rows after the first step on their way up

  const int tid = threadIdx.x, nt = blockDim.x;
  const int tl = max(tid - 1, 0), tr = min(tid + 1, nt - 1);
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = tile % nbx, by = tile / nbx;
  const int xu = bx * (nt - 2 * kPairHalo) - kPairHalo + tid;
  const int x = ((xu % nx) + nx) % nx;
  const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const bool own = tid >= kPairHalo && tid < nt - kPairHalo && xu < nx;
  const int y0 = by * rows, yend = min(y0 + rows, ny);

  S f1[9], g1[9];                  // first step: row r (on its way, then gathered)
  S f2[2][9], g2[2][9];            // second step: rows r2, r2 - 1
  S mid_f[3], mid_g[3];
  double m1[2][NM], m2[2][NM];     // rho, u_x, u_y, theta, e, -d phi_x / dx [, dT/dx, du_x/dx, dh/dx]
  double v1[NX][3], v2[NX][3];     // phi_y [, T, u_y [, h]] of the last three rows

  auto lattice_row = [&](int r) {
    if (WALLS) return min(max(r, 0), ny - 1);
    while (r < 0) r += ny;
    while (r >= ny) r -= ny;
    return r;
  };
  auto fetch = [&](int r) {
    const int y = lattice_row(r);
    const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
    const int64_t r0 = (int64_t)y * pitch, rm = (int64_t)ym * pitch, rp = (int64_t)yp * pitch;
    const bool top = WALLS == 1 && y == ny - 1, bot = WALLS == 1 && y == 0;
    gather9(A, plane, r0, rm, rp, x, xm, xp, top, bot, f1);
    gather9(A + 9 * plane, plane, r0, rm, rp, x, xm, xp, top, bot, g1);
  };
  // moments of a gathered row; its values exchanged along x to sx, those along y to v
  auto moments = [&](const S(&f)[9], const S(&g)[9], double(&mm)[NM], double (&v)[NX],
                     double (&sx)[NX][kBlock]) {
    Moments m;
    moments_closure_dev<X, VDW>(f, g, prm, m, prm.Fx, prm.Fy, prm.Q);
    mm[0] = m.rho;
    mm[1] = m.ux;
    mm[2] = m.uy;
    mm[3] = m.theta;
    mm[4] = m.e;
    sx[0][tid] = m.rho * m.ux * (m.ux * m.ux + 3.0 * (m.theta - 1.0 / 3.0));
    v[0] = m.rho * m.uy * (m.uy * m.uy + 3.0 * (m.theta - 1.0 / 3.0));
    asm volatile("" : "+v"(v[0]));  // formed here, not where it is used (see collide)
    if constexpr (X) {
      const double T = node_temperature<VDW>(prm, m.rho, m.e, m.theta);
      sx[1][tid] = T;
      sx[2][tid] = m.ux;
      v[1] = T;
      v[2] = m.uy;
      if constexpr (VDW) {
        sx[3][tid] = m.e + m.theta;
        v[3] = m.e + m.theta;
      }
    }
  };
  auto shift = [&](double (&v)[NX][3]) {
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      v[k][0] = v[k][1];
      v[k][1] = v[k][2];
    }
  };
  // boundary row of the NEQ walls (App. B) from its neighbour row's populations
  auto wall_row = [&](int side, const S(&nf)[9], const S(&ng)[9], S(&bf)[9], S(&bg)[9]) {
    double f[9], g[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      f[i] = (double)nf[i] + prm.wf[i];
      g[i] = (double)ng[i] + prm.wg[i];
    }
    Moments m;
    moments_closure<false, VDW>(f, g, prm, m);
    double feN[9], geN[9], feB[9], geB[9];
    equilibria(m.rho, m.ux, m.uy, m.theta, m.e, feN, geN);
    const double TN = node_temperature<VDW>(prm, m.rho, m.e, m.theta);
    double rhoB, thetaW, eW;
    neq_wall_state<VDW>(prm, side, m.rho, TN, m.rho * m.theta, rhoB, thetaW, eW);
    equilibria(rhoB, side ? prm.uw[1][0] : prm.uw[0][0], side ? prm.uw[1][1] : prm.uw[0][1], thetaW,
               eW, feB, geB);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      bf[i] = (S)(feB[i] + (f[i] - feN[i]) - prm.wf[i]);
      bg[i] = (S)(geB[i] + (g[i] - geN[i]) - prm.wg[i]);
    }
  };
  auto x_derivatives = [&](double(&m)[NM], const double (&sx)[NX][kBlock]) {
    m[5] = prm.phi ? -(0.5 * (sx[0][tr] - sx[0][tl])) : 0.0;
    if constexpr (X) {
      m[6] = 0.5 * (sx[1][tr] - sx[1][tl]);
      m[7] = 0.5 * (sx[2][tr] - sx[2][tl]);
      if constexpr (VDW) m[8] = 0.5 * (sx[3][tr] - sx[3][tl]);
    }
  };
  auto collide = [&](int c, const S(&f)[9], const S(&g)[9], const double(&moments)[NM],
                     const double (&v)[NX][3], auto&& sink) {
    // the moments are re-declared here: half of the unrolled body would otherwise keep products of
    // them from the gather (10 registers more, spilled)
    double m[NM];
#pragma unroll
    for (int k = 0; k < NM; ++k) {
      m[k] = moments[k];
      if (k < 5) asm volatile("" : "+v"(m[k]));
    }
    double d[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      // zero-order ghosts beyond the walls
      const double lo = WALLS && c == 0 ? v[k][1] : v[k][0];
      const double hi = WALLS && c == ny - 1 ? v[k][1] : v[k][2];
      d[k] = 0.5 * (hi - lo);
    }
    double phxx = 0.0, phyy = 0.0;
    if (prm.phi) {
      const double inv_rho = 1.0 / m[0];
      phxx = m[5] * inv_rho;
      phyy = -d[0] * inv_rho;
    }
    collide_ddf<X, VDW, true>(f, g, m, phxx, phyy, d[1], d[2], d[3], prm, sink);
  };

  auto iteration = [&](int r, auto J) {
    constexpr int j = decltype(J)::value;
    // ---- gather: first step, row r --------------------------------------------------------
    double v[NX];
    shift(v1);
    if constexpr (NEQ) {
      if (r == ny - 1) {  // from row ny - 2, which waits for its collision
        S nf[9], ng[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
          nf[i] = s_wait[i][tid];
          ng[i] = s_wait[9 + i][tid];
        }
        wall_row(1, nf, ng, f1, g1);
      } else if (r == 1) {
        S bf[9], bg[9];
        wall_row(0, f1, g1, bf, bg);
        moments(bf, bg, m1[1 - j], v, s_wall[0]);
#pragma unroll
        for (int k = 0; k < NX; ++k) v1[k][1] = v[k];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
          s_wait[i][tid] = bf[i];
          s_wait[9 + i][tid] = bg[i];
        }
      }
    }
    moments(f1, g1, m1[j], v, s_x[0][j]);
#pragma unroll
    for (int k = 0; k < NX; ++k) v1[k][2] = v[k];
    // ---- gather: second step, row r - 4, from rows r - 3 (read now), r - 4 and r - 5 after the
    // first step ------------------------------------------------------------------------------
    const int r2 = r - 4;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int at = a == 0 ? tr : (a == 1 ? tid : tl);
      f2[j][3 + a] = mid_f[a];
      g2[j][3 + a] = mid_g[a];
      f2[j][6 + a] = s_up[j][a][tid];
      g2[j][6 + a] = s_up[j][3 + a][tid];
      f2[j][a] = s_row[j][a][at];
      g2[j][a] = s_row[j][9 + a][at];
      mid_f[a] = s_row[j][3 + a][at];
      mid_g[a] = s_row[j][12 + a][at];
      s_up[j][a][tid] = s_row[j][6 + a][at];
      s_up[j][3 + a][tid] = s_row[j][15 + a][at];
      if (WALLS == 1 && r2 == -1) {  // row 0's upward ones bounce back: its own downward ones
        s_up[1 - j][a][tid] = s_row[j][2 - a][tid];
        s_up[1 - j][3 + a][tid] = s_row[j][11 - a][tid];
      }
    }
    if (WALLS == 1 && r2 == ny - 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        f2[j][a] = s_row[1 - j][8 - a][tid];
        g2[j][a] = s_row[1 - j][17 - a][tid];
      }
    }
    shift(v2);
    if constexpr (NEQ) {
      if (r2 == ny - 1) {
        wall_row(1, f2[1 - j], g2[1 - j], f2[j], g2[j]);
      } else if (r2 == 1) {
        wall_row(0, f2[j], g2[j], f2[1 - j], g2[1 - j]);
        moments(f2[1 - j], g2[1 - j], m2[1 - j], v, s_wall[NEQ ? 1 : 0]);
#pragma unroll
        for (int k = 0; k < NX; ++k) v2[k][1] = v[k];
      }
    }
    moments(f2[j], g2[j], m2[j], v, s_x[1][j]);
#pragma unroll
    for (int k = 0; k < NX; ++k) v2[k][2] = v[k];
    __syncthreads();
    // ---- collide: first step, row r - 1 -------------------------------------------------------
    x_derivatives(m1[j], s_x[0][j]);
    if constexpr (NEQ)
      if (r == 1) x_derivatives(m1[1 - j], s_wall[0]);
    if (!WALLS || (r >= 1 && r <= ny)) {
      S wf[9], wg[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        wf[i] = s_wait[i][tid];
        wg[i] = s_wait[9 + i][tid];
      }
      collide(r - 1, wf, wg, m1[1 - j], v1, [&](int i, double htf, double, double htg, double) {
        s_row[j][i][tid] = (S)htf;
        s_row[j][9 + i][tid] = (S)htg;
      });
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      s_wait[i][tid] = f1[i];
      s_wait[9 + i][tid] = g1[i];
    }
    fetch(min(r + 1, yend + 2));
    // ---- collide: second step, row r2 - 1 -------------------------------------------------------
    x_derivatives(m2[j], s_x[1][j]);
    if constexpr (NEQ)
      if (r2 == 1) x_derivatives(m2[1 - j], s_wall[NEQ ? 1 : 0]);
    const int c = r2 - 1;
    if (own && c >= y0 && c < yend) {
      const int64_t off = (int64_t)c * pitch + x;
      collide(c, f2[1 - j], g2[1 - j], m2[1 - j], v2, [&](int i, double htf, double, double htg, double) {
        store_nt(B + i * plane + off, (S)htf);
        store_nt(B + (9 + i) * plane + off, (S)htg);
      });
    }
  };
  fetch(y0 - kPairHalo);
  // the last own row leaves at r = yend + 4
  for (int r = y0 - kPairHalo; r <= yend + 4; r += 2) {
    iteration(r, std::integral_constant<int, 0>{});
    iteration(r + 1, std::integral_constant<int, 1>{});
  }
}

// ---- launcher -------------------------------------------------------------------------------
template <typename S, int WALLS>
static void pair_launch(const S* A, S* B, const Layout& L, const DdfParams& prm, const PairShape& p,
                        hipStream_t s) {
  const dim3 grid((unsigned)p.nbx * p.parts), block(p.threads);
  if (prm.eos)
    k_ddf_pair<S, WALLS, 2><<<grid, block, 0, s>>>(A, B, L.nx, L.ny, L.pitch, L.plane, prm, p.rows, p.nbx);
  else if (prm.ext())
    k_ddf_pair<S, WALLS, 1><<<grid, block, 0, s>>>(A, B, L.nx, L.ny, L.pitch, L.plane, prm, p.rows, p.nbx);
  else
    k_ddf_pair<S, WALLS, 0><<<grid, block, 0, s>>>(A, B, L.nx, L.ny, L.pitch, L.plane, prm, p.rows, p.nbx);
}

hipError_t launch_ddf_pair(int fmt, bool walls, const void* A, void* B, const Layout& L,
                           const DdfParams& prm, const PairShape& shape, hipStream_t s) {
  if (fmt != 0 || prm.phi == 2) return hipErrorInvalidValue;
  if (prm.neq && (!walls || L.ny < 3 || prm.src)) return hipErrorInvalidValue;
  const float* a = static_cast<const float*>(A);
  float* b = static_cast<float*>(B);
  if (prm.neq) pair_launch<float, 2>(a, b, L, prm, shape, s);
  else if (walls) pair_launch<float, 1>(a, b, L, prm, shape, s);
  else pair_launch<float, 0>(a, b, L, prm, shape, s);
  return hipGetLastError();
}

}  // namespace lbm
