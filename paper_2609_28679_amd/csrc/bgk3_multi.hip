// Isothermal D3Q27, two time steps per launch (float32 storage, two buffers, periodic, no force).
//
// A step per launch moves 216 bytes per node and step and is bound by that (256^3: 619 us, 5.85
// TB/s). Here a workgroup owns 64 columns and 9 rows and marches along z: every plane of its region
// (one node more on every side) takes the first step and passes through LDS to the second one, one
// plane behind. A node's populations arrive from three planes: those moving down are read when
// their plane is in LDS, the others wait in registers for one and two planes. The column left and
// right of the tile is a wavefront of its own (a node per lane), so rows stay 64 aligned columns
// wide; the rows above and below cost 11 wavefronts of arithmetic for 9 rows. The next plane's loads
// are issued before the second step. Twelve wavefronts, three per SIMD, 168 registers, 78 KB of
// LDS. Measured on MI355X, us per step, one -> two steps per launch: 256^3 619 -> 457, 160 x 180 x
// 170 197 -> 151. Region rows at 256^3: 11 460 us, 7 524, 14 882 (128 registers, spilled). Where it
// is taken: routes.h. What keeps one step per launch: walls and forces, whose second collision
// spills at 168 registers (256^3 612 -> 666 us and 619 -> 800; at 7 rows, without spills, 597 and 580,
// which a kernel of its own would give), and lattices of one in-place buffer (us per step in place /
// two buffers and two steps: 100^3 41 / 41, 120^3 58 / 58, but 140^3 140 / 99 and 150^3 154 / 111).
#include "bgk_common.h"
#include "routes.h"

namespace lbm {

constexpr int kP3Threads = 64 * (kP3Rows + 1);  // a wavefront per row, one for the halo columns

__global__ void __launch_bounds__(kP3Threads)
k_bgk_d3q27_pair(const float* __restrict__ A, float* __restrict__ B, int nx, int ny, int nz,
                 int64_t pitch, int64_t plane, double omega, int nbx, int nby, int nzc) {
  __shared__ float s[27][kP3Rows][66];  // one plane after the first step, columns -1 .. 64
  const int tiles = nbx * nby;
  const int bid = xcd_tile(blockIdx.x, gridDim.x);
  const int tile = bid % tiles, chunk = bid / tiles;
  const int bx = tile % nbx, by = tile / nbx;
  const int zb = (int)((int64_t)chunk * nz / nzc), ze = (int)((int64_t)(chunk + 1) * nz / nzc);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool halo = wv == kP3Rows;
  const int x0 = bx * 64, y0 = by * kP3Own;
  const int ncols = min(64, nx - x0);
  auto wrap = [](int v, int n) {
    while (v < 0) v += n;
    while (v >= n) v -= n;
    return v;
  };
  // this lane's node in a plane: a row wavefront's column, or a halo node (row lane / 2, the
  // column left of the tile or right of it); lanes without a node repeat one and store nothing
  const int row = halo ? min(lane >> 1, kP3Rows - 1) : wv;
  const int y = wrap(y0 - 1 + row, ny);
  const int x = halo ? ((lane & 1) ? (x0 + ncols == nx ? 0 : x0 + ncols) : (x0 == 0 ? nx - 1 : x0 - 1))
                     : x0 + min(lane, ncols - 1);
  const int col = halo ? ((lane & 1) ? ncols + 1 : 0) : lane + 1;
  const bool put = halo ? lane < 2 * kP3Rows : lane < ncols;
  const int yr = y0 - 1 + wv;  // row wavefronts
  const bool own = !halo && wv >= 1 && wv <= kP3Own && yr < ny && lane < ncols;
  const int xs[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
  const int ys[3] = {y == ny - 1 ? 0 : y + 1, y, y == 0 ? ny - 1 : y - 1};
  float h[27];
  auto fetch = [&](int zz) __attribute__((always_inline)) {
    const int z = wrap(zz, nz);
    const int zs[3] = {z == nz - 1 ? 0 : z + 1, z, z == 0 ? nz - 1 : z - 1};
    int64_t pl = plane;
    asm volatile("" : "+s"(pl));
    if (!halo) {
      const int yu = __builtin_amdgcn_readfirstlane(y);
      const int yn[3] = {yu == ny - 1 ? 0 : yu + 1, yu, yu == 0 ? ny - 1 : yu - 1};
      const uint32_t xo[3] = {fresh(4u * xs[0]), fresh(4u * xs[1]), fresh(4u * xs[2])};
#pragma unroll
      for (int i = 0; i < 27; ++i) {
        const int a = i % 3, b = (i / 3) % 3, c = i / 9;
        h[i] = *at_byte(sbase(A + i * pl + ((int64_t)zs[c] * ny + yn[b]) * pitch), xo[a]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 27; ++i) {
        const int a = i % 3, b = (i / 3) % 3, c = i / 9;
        h[i] = A[i * pl + ((int64_t)zs[c] * ny + ys[b]) * pitch + xs[a]];
      }
    }
  };
  float mid[9], up[2][9];  // rows after the first step that wait one and two planes
  NodeMoments m;
  const Force F{};
  auto iteration = [&](int zz, auto J) __attribute__((always_inline)) {
    constexpr int j = decltype(J)::value;
    collide_bgk<3, false>(h, omega, F, m, [&](int i, float v) {
      if (put) s[i][row][col] = v;
    });
    fetch(min(zz + 1, ze));
    __syncthreads();
    if (!halo && wv >= 1 && wv <= kP3Own) {
      // second step, plane zz - 1: populations from planes zz (now), zz - 1 and zz - 2
      float g[27];
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int a = k % 3 - 1, b = k / 3 - 1;
        auto pull = [&](int i) { return s[i][wv - b][lane + 1 - a]; };
        g[k] = pull(k);
        g[9 + k] = mid[k];
        g[18 + k] = up[j][k];
        mid[k] = pull(9 + k);
        up[j][k] = pull(18 + k);
      }
      const int z2 = zz - 1;
      if (own && z2 >= zb && z2 < ze) {
        float* out = B + ((int64_t)z2 * ny + __builtin_amdgcn_readfirstlane(y)) * pitch;
        const uint32_t xo = fresh(4u * xs[1]);
        int64_t pl = plane;
        asm volatile("" : "+s"(pl));
        collide_bgk<3, false>(g, omega, F, m, [&](int i, float v) {
          gstore_nt(at_byte(sbase(out + i * pl), xo), v);
        });
      }
    }
    __syncthreads();
  };
  fetch(zb - 1);
  for (int zz = zb - 1; zz <= ze; zz += 2) {
    iteration(zz, std::integral_constant<int, 0>{});
    if (zz + 1 <= ze) iteration(zz + 1, std::integral_constant<int, 1>{});
  }
}

hipError_t launch_bgk_d3q27_pair(const void* A, void* B, const Layout& L, const Pair3Shape& p,
                                 double omega, hipStream_t s) {
  k_bgk_d3q27_pair<<<(unsigned)((int64_t)p.nbx * p.nby * p.ranges), kP3Threads, 0, s>>>(
      static_cast<const float*>(A), static_cast<float*>(B), L.nx, L.ny, L.nz, L.pitch, L.plane,
      omega, p.nbx, p.nby, p.ranges);
  return hipGetLastError();
}

}  // namespace lbm
