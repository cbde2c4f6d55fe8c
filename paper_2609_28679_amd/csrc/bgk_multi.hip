// Isothermal D2Q9, several time steps per launch on tiles held in LDS (float32 or float64
// storage, the paper's collision).
//
// One step per launch moves 72 bytes per node and step (float32) and is bound by that traffic;
// its arithmetic, 90 vector instructions per node, fills a fifth of the time. Six steps per
// launch move the state once for all six and recompute the nodes around each tile (1.4 x the
// arithmetic), which leaves the two about level. Measured on MI355X, us per step in calls of 600
// steps and more, one-step kernels -> this one: float32 64^2 2.54 -> 0.97 (launches), 2048^2 44.2 ->
// 22.1, with a force 45.9 -> 33.4, 4096^2 210 -> 88; float64 1001 x 515 11.3 -> 4.6, with walls and
// force 5.3, 2048^2 98 -> 37.8. Calls of 20 steps: 2048^2 24-27, 4096^2 99-109, float64 2048^2 43;
// one that begins at an odd step of the in-place layout also takes one or two one-step launches
// (2048^2 29.8).
#include "bgk_common.h"
#include "routes.h"

namespace lbm {

constexpr int kMsLanes = 64;  // region columns: one per lane

// T steps of k_bgk_d2q9 (T even), from state A to state B. A workgroup owns `rows` rows of
// 64 - 2 (T - 1) columns; its region is the owned rectangle and T - 1 nodes more on every side,
// one lane per column. The first step pulls the region from A, the last writes the owned nodes
// to B, the steps between stay in LDS, each on a region one node smaller per side. The LDS
// state is a single copy in the two-step in-place layout of k_bgk_d2q9_aa (a node reads and
// writes the same nine locations, so one barrier per step is enough):
//   after an odd step slot 8-i of a node holds its h~_i; after an even one slot i of node
//   x + c_i does (slot 8-i of the node itself where x + c_i lies beyond a y wall).
// Values are rounded to the storage type between steps like a stored state, so the result equals
// T launches of the one-step kernel. An LDS row holds its nine slots one after the other, so
// every location of a node is a constant offset from one lane address. Loads and stores keep the
// default cache policy: neighbouring tiles share the halo and the cache lines at the tile edges
// (non-temporal stores 24.3 -> 26.2 us at 2048^2, loads 25.4).
template <typename S, int T, bool WALLS, bool FORCE>
__global__ void __launch_bounds__(1024)
k_bgk_d2q9_multi(const S* __restrict__ A, S* __restrict__ B, int nx, int ny, int64_t pitch,
                 int64_t plane, double omega, Force F, int rows, int nbx) {
  static_assert(T % 2 == 0 && T >= 2, "the last step reads the layout of an odd step");
  constexpr int H = T - 1;                   // halo of the first step
  constexpr int OWN = kMsLanes - 2 * H;
  constexpr int ROW = 9 * kMsLanes;          // LDS elements of one region row
  extern __shared__ __align__(16) char lds_raw[];
  S* const lds = reinterpret_cast<S*>(lds_raw);

  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = tile % nbx, by = tile / nbx;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int y0 = by * rows - H;              // lattice row of region row 0
  const int nr = min(rows, ny - by * rows) + 2 * H;
  const int xr = bx * OWN - H + lane;        // unwrapped column
  const int x = ((xr % nx) + nx) % nx;
  const uint32_t xs[3] = {(uint32_t)(x == nx - 1 ? 0 : x + 1), (uint32_t)x,
                          (uint32_t)(x == 0 ? nx - 1 : x - 1)};  // x - c_x for c_x = -1, 0, +1
  // lattice row of the wave's first region row, stepped with it (periodic: wrapped)
  auto row_of = [&](int q) { return WALLS ? y0 + q : (((y0 + q) % ny) + ny) % ny; };
  auto advance = [&](int& y) {
    y += nw;
    if (!WALLS)
      while (y >= ny) y -= ny;
  };
  NodeMoments m;

  // first step: pull from A
  auto load = [&](int yr, S (&h)[9]) {
    const int y = WALLS ? min(max(yr, 0), ny - 1) : yr;
    const int ysrc[3] = {y == ny - 1 ? 0 : y + 1, y, y == 0 ? ny - 1 : y - 1};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int ka = i % 3, kb = i / 3;
      const bool bounce = WALLS && ((kb == 0 && y == ny - 1) || (kb == 2 && y == 0));
      const int k = bounce ? 8 - i : i;
      const S* row = A + k * plane + (int64_t)(bounce ? y : ysrc[kb]) * pitch;
      const uint32_t o = WALLS && bounce ? xs[1] : xs[ka];
      h[i] = at_byte(sbase(row), fresh(o * (uint32_t)sizeof(S)))[0];
    }
  };
  S nxt[9];
  int yn = row_of(wv);
  load(yn, nxt);
  for (int q = wv; q < nr; q += nw) {
    S h[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) h[i] = nxt[i];
    if (q + nw < nr) {
      advance(yn);
      load(yn, nxt);
    }
    S* const me = lds + q * ROW + lane;
    collide_bgk<2, FORCE>(h, omega, F, m, [&](int i, S v) { me[(8 - i) * kMsLanes] = v; });
  }

#pragma unroll
  for (int s = 2; s <= T; ++s) {
    __syncthreads();
    const bool in = lane >= s - 1 && lane <= kMsLanes - s;
    int y = row_of(s - 1 + wv);
    for (int q = s - 1 + wv; q <= nr - s; q += nw, advance(y)) {
      if (WALLS && (y < 0 || y >= ny)) continue;
      if (!in) continue;
      const bool bot = WALLS && y == 0, top = WALLS && y == ny - 1;
      S* const me = lds + q * ROW + lane;
      // location of the population i arriving at this node (even step), which is also where
      // its departing population 8 - i goes
      auto at = [&](int i) {
        const int cx = i % 3 - 1, cy = i / 3 - 1;
        const bool wall = (cy > 0 && bot) || (cy < 0 && top);
        return wall ? me + i * kMsLanes : me - cy * ROW + (8 - i) * kMsLanes - cx;
      };
      S h[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) h[i] = s % 2 == 0 ? *at(i) : me[i * kMsLanes];
      if (s == T) {
        const int64_t r = (int64_t)y * pitch;
        if (xr < nx) {
          collide_bgk<2, FORCE>(h, omega, F, m, [&](int i, S v) {
            at_byte(sbase(B + i * plane + r), fresh(xs[1] * (uint32_t)sizeof(S)))[0] = v;
          });
        }
      } else {
        collide_bgk<2, FORCE>(h, omega, F, m, [&](int i, S v) {
          if (s % 2 == 0) *at(8 - i) = v;
          else me[(8 - i) * kMsLanes] = v;
        });
      }
    }
  }
}

// ---- launcher -------------------------------------------------------------------------------
namespace {
struct MultiShape {
  int T, rows, waves;
};

// Steps per launch: six where the call has them left (kMultiSteps). Measured on MI355X (us per step; best
// rows for each count of 4 / 6 / 8 steps): float32 64^2 1.13 / 0.99 / 1.01, 256^2 1.41 / 1.34 /
// 1.40, 1024^2 6.64 / 6.73 / 7.3, 2048^2 24.7 / 24.3 / 27.0, 4096^2 88.4 / 86.7 / 94.8; float64
// 1001 x 515 5.78 / 5.10 / 5.89, 2048^2 41.2 / 39.4 / 41.9. More steps per launch save memory
// traffic and launches and cost halo nodes.
// Rows per workgroup: the least region rows walked by the busiest compute unit, counted as
// workgroups per unit x (region rows of all steps + a fixed part, the first loads and the
// barriers); at most 24 rows in float32 (two workgroups of 16 wavefronts per compute unit) and
// 20 in float64 (one), the best of the sweeps at 2048^2 and 4096^2. Small lattices get low tiles that
// fill the 256 compute units once (64^2 two rows: 0.99 us a step, eight rows: 1.2).
MultiShape multi_shape(const Layout& L, int elem, int steps) {
  MultiShape m;
  m.T = steps;
  const int own = kMsLanes - 2 * (m.T - 1);
  const int64_t nbx = (L.nx + own - 1) / own;
  const int max_rows = std::min(elem == 4 ? 24 : 20, L.ny);
  int64_t best = -1;
  for (int r = 1; r <= max_rows; ++r) {
    const int64_t blocks = nbx * ((L.ny + r - 1) / r);
    const int64_t cost = (blocks + kCus - 1) / kCus * (m.T * (r + m.T - 1) + 20);
    if (best < 0 || cost <= best) {
      best = cost;
      m.rows = r;
    }
  }
  m.waves = m.rows + 2 * (m.T - 1) >= 16 ? 16 : 8;
  return m;
}

template <typename S, int T>
hipError_t multi_t(const S* A, S* B, const Layout& L, int64_t plane, double omega, const Force& F,
                   bool walls, const MultiShape& m, hipStream_t s) {
  const int own = kMsLanes - 2 * (T - 1);
  const int nbx = (L.nx + own - 1) / own, nby = (L.ny + m.rows - 1) / m.rows;
  const size_t lds = (size_t)(m.rows + 2 * (T - 1)) * 9 * kMsLanes * sizeof(S);
  with_flag(walls, [&](auto W) {
    with_flag(F.on(), [&](auto Fo) {
      k_bgk_d2q9_multi<S, T, decltype(W)::value, decltype(Fo)::value>
          <<<dim3((unsigned)nbx * nby), dim3(64 * m.waves), lds, s>>>(
              A, B, L.nx, L.ny, L.pitch, plane, omega, F, m.rows, nbx);
    });
  });
  return hipGetLastError();
}

template <typename S>
hipError_t multi(const void* A, void* B, const Layout& L, bool swapped, double omega,
                 const Force& F, bool walls, const MultiShape& m, hipStream_t s) {
  const S* a = static_cast<const S*>(A);
  S* b = static_cast<S*>(B);
  int64_t plane = L.plane;
  if (swapped) {  // slot 8 - i holds population i
    a += 8 * plane;
    b += 8 * plane;
    plane = -plane;
  }
  switch (m.T) {
    case 6: return multi_t<S, 6>(a, b, L, plane, omega, F, walls, m, s);
    case 4: return multi_t<S, 4>(a, b, L, plane, omega, F, walls, m, s);
    default: return multi_t<S, 2>(a, b, L, plane, omega, F, walls, m, s);
  }
}
}  // namespace

hipError_t launch_bgk_d2q9_multi(int kind, const void* A, void* B, const Layout& L, bool swapped,
                                 double omega, const Force& F, bool walls, int steps,
                                 hipStream_t s) {
  if (steps != 2 && steps != 4 && steps != 6) return hipErrorInvalidValue;
  const MultiShape m = multi_shape(L, kind == 0 ? 4 : 8, steps);
  return kind == 0 ? multi<float>(A, B, L, swapped, omega, F, walls, m, s)
                   : multi<double>(A, B, L, swapped, omega, F, walls, m, s);
}

}  // namespace lbm
