// Host rules of the kernels that come in several shapes: which launches a lattice takes and how they
// are cut into workgroups. No device code.
#pragma once

#include <algorithm>
#include <climits>
#include <cstdlib>

#include "lbm_internal.h"

namespace lbm {

constexpr int kCus = 256;  // compute units

inline int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- double distribution, D2Q9: one step per launch ----------------------------------------------
// Columns owned by a workgroup: its threads less the halo and, when the rows are staged (the kernel's
// TXI), one staging-only thread per side.
inline Grid make_grid_ddf(const Layout& L, int halo, bool reduced) {
  Grid G;
  G.bx = kBlock;
  const int txi = kBlock - 2 * halo - (reduced ? 2 : 0);
  G.nbx = (L.nx + txi - 1) / txi;
  // rows per workgroup from sweeps on MI355X at 4096^2 with walls (float32, central Phi:
  // 2 -> 588 us, 4 -> 553, 8 -> 580, 16 -> 599; float32, upwind Phi: 4 -> 646, 8 -> 596,
  // 16 -> 586; reduced bf16: 8 -> 676, 16 -> 602, 32 -> 604): short windows give more
  // workgroups in flight, taller ones amortise the halo rows (two per side for the upwind
  // stencil) and the staged kernel's 2-row staging halo
  G.rows = reduced ? 16 : (halo == 2 ? 16 : 4);
#ifdef LBM_TUNING_ENV
  if (const char* v = getenv("LBM_DDF_ROWS")) G.rows = atoi(v);
#endif
  fit_rows(G, L.ny);
  return G;
}

// Rows per workgroup of the extended collisions (sources, transport control, van der Waals):
// their longer per-row arithmetic favours taller windows than the plain step's. Measured at
// 4096^2 with walls, central Phi, float32 (4 / 6 / 8 / 10 rows): sources 618 / 589 / 582 /
// 583 us, Pr 0.71 646 / 613 / 601 / 599, van der Waals 719 / 673 / 649 / 644; the plain and NEQ
// steps keep their 4 (552 / 568 at 6 and 561 / 580).
constexpr int kDdfExtRows = 8;

// The collision of a step: plain, with sources or transport control, of a van der Waals fluid.
enum DdfCollision { kDdfPlain, kDdfExtended, kDdfVdw };

// Workgroups that share a compute unit, by the registers of the kernel (wavefronts per SIMD in the
// compiler's resource report): three of the plain float32 step with central Phi, one of the upwind
// steps in float64 or of a van der Waals fluid or between bounce-back walls, all but the plain ones;
// two otherwise.
inline int ddf_per_cu(int halo, int fmt, DdfCollision c, bool bounce) {
  if (fmt == 0 && halo == 1 && c == kDdfPlain) return 3;
  return halo == 2 && c != kDdfPlain && (fmt == 1 || c == kDdfVdw || bounce) ? 1 : 2;
}

// Window rows that the chip walks one after the other: rounds of resident workgroups x (rows + 2
// halo + 1 for the start), in tenths. Each of three workgroups of a unit beyond the first costs a
// fifth where all workgroups are resident at once (700 x 640: 4 rows, two workgroups per unit, 19.3
// us; 3 rows, three per unit, 21.5).
inline int64_t ddf_turns(int64_t blocks, int rows, int halo, int per_cu) {
  int64_t rounds = 10 * div_up(blocks, (int64_t)kCus * per_cu);
  if (per_cu == 3 && rounds == 10) rounds += 2 * (div_up(blocks, kCus) - 1);
  return rounds * (rows + 2 * halo + 1);
}

// Lattices that do not fill the chip several times over get lower windows: the rows in
// [1, G.rows] with the least turns, where those are 5% fewer (4096^2 bfloat16 / float16: 14 rows, 1%
// fewer turns, 527 / 538 us, 16 rows 514 / 521, whose halo rows are fewer). us per step, the fixed rows -> these: 64^2 plain 9.6 -> 5.9,
// upwind 28.1 -> 7.9, float16 44.6 -> 11.5, Pr 0.71 with NEQ walls 21.9 -> 10.5; 512^2 plain 16.0 ->
// 13.8, upwind 38.5 -> 22; 1021 x 509 Pr 0.71 with NEQ walls 38.3 -> 30.6, float16 48.7 -> 32. Of 28
// sizes from 40 x 20 to 2048^2 in 18 configurations these rows are within 3% of the best ones on
// average (512^2 with a force 4 rows 17.9, 2 rows 18.2; 768^2 float64 Pr 0.71 upwind 12 rows 54.4, 16
// rows 65.1).
inline Grid ddf_fill(Grid G, const Layout& L, int halo, int per_cu) {
  auto turns = [&](int r) { return ddf_turns(G.nbx * div_up(L.ny, r), r, halo, per_cu); };
  int64_t best = -1;
  int rows = G.rows;
  for (int r = 1; r <= G.rows; ++r)
    if (best < 0 || turns(r) <= best) {
      best = turns(r);
      rows = r;
    }
  if (best * 100 > turns(G.rows) * 95) rows = G.rows;
  G.rows = rows;
  fit_rows(G, L.ny);
  return G;
}

// Launch grid of one step, from the plan's grid: taller windows for the extended collisions. A step
// that writes its diagnostics records keeps the plan's windows where the lower ones would write
// more than there is room for.
inline Grid ddf_step_grid(Grid G, const Layout& L, int phi, int fmt, DdfCollision c, bool bounce,
                          int room) {
  if (fmt < 2 && c != kDdfPlain && G.rows < kDdfExtRows) {
    G.rows = kDdfExtRows;
    fit_rows(G, L.ny);
  }
  // 16-bit storage stages two rows more per window: lower ones pay up to two rounds only (2048^2, three
  // rounds: 13 rows 146 us, 16 rows 137; 3000^2 15 rows 305, 16 rows 282-295)
  if (fmt >= 2 && G.blocks() > 2 * 2 * kCus) return G;
  const int halo = phi == 2 ? 2 : 1;
  const Grid filled = ddf_fill(G, L, halo, ddf_per_cu(halo, fmt, c, bounce));
  return filled.blocks() <= room ? filled : G;
}

// Most diagnostics records any step of the format writes (grid G of the plan).
inline int ddf_max_records(const Layout& L, const Grid& G, int phi, int fmt) {
  int most = 0;
  for (DdfCollision c : {kDdfPlain, kDdfExtended, kDdfVdw})
    for (bool bounce : {false, true})
      most = std::max(most, ddf_step_grid(G, L, phi, fmt, c, bounce, INT_MAX).blocks());
  return most;
}

// ---- double distribution, D2Q9: two steps per launch ----------------------------------------------
constexpr int kPairHalo = 3;  // columns per side that only supply neighbours

// Shape of k_ddf_pair: the rows per workgroup that the chip walks in the least turns, one workgroup
// per compute unit (two for the plain collision without NEQ walls) x (rows + 8 of both steps' halo
// + 4 for the start).
inline PairShape ddf_pair_shape(const Layout& L, const DdfParams& prm) {
  PairShape s;
  s.threads = std::min(kBlock, (L.nx + 2 * kPairHalo + 63) / 64 * 64);
  s.nbx = (int)div_up(L.nx, s.threads - 2 * kPairHalo);
  const int64_t slots = kCus * (int64_t)(prm.ext() || prm.eos || prm.neq ? 1 : 2) * kBlock / s.threads;
  const int max_rows = std::min(L.ny, 512);
  for (int r = 1; r <= max_rows; ++r) {
    const int64_t cost = div_up(s.nbx * div_up(L.ny, r), slots) * (r + 8 + 4);
    if (s.turns < 0 || cost <= s.turns) {
      s.turns = cost;
      s.rows = r;
    }
  }
  s.parts = (int)div_up(L.ny, s.rows);
  s.rounds = (int)div_up((int64_t)s.nbx * s.parts, slots);
  return s;
}

// Where two steps per launch are taken, float32 with central Phi or none. A window row costs more
// serial time here than in the one-step kernel, and a workgroup walks 12 rows besides its own; what
// is gained is the memory traffic of large lattices, half of it. us per step, one step / two:
//   - from 700 000 nodes on, NEQ walls 400 000 (512^2 plain 13.8 / 19.4, 1021 x 509 24.3 / 25.1, 1024^2
//     46.0 / 35.6, with NEQ walls 512^2 23.3 / 23.9 and 700 x 600 24.4 / 20.0);
//   - six rows per workgroup or more (240000 x 3 plain 30.5 / 35.6, force 31.6 / 59; 120000 x 6 plain
//     29.1 / 25.8);
//   - full workgroups, or for the plain collision those of 64 and 128 threads: the LDS of a workgroup
//     does not shrink with its threads (10 x 70000 plain 322 / 167, force 351 / 384; 130 x 6000 plain
//     40.3 / 41.7, with NEQ walls 42.8 / 59.1);
//   - collisions with a force or heat source, transport control or a van der Waals fluid, which run
//     one workgroup per compute unit: turns up to 2.46 x those of the one-step launch, with NEQ walls,
//     whose rows that launch takes from one of their own, 3 x, and where fewer than 63% of the threads
//     own a column 1.9 x (turns, times: 1000 x 768 with a force 2.67, 31.2 / 31.1, van der Waals 34.2 /
//     36.3; 900^2 2.45, 37.4 / 36.3 and 41.3 / 41.3; 1024^2 1.83, 51.3 / 44.5 and 58.7 / 51.2; 1021 x
//     509 Pr 0.71 with NEQ walls 2.75, 29.5 / 28.5; 270 x 2000 the same 2.55, 33.8 / 36.7; 304 x 10605
//     1.58, 9% faster); with NEQ walls also one round or 16 rows (200000 x 12 van der Waals 134 / 150).
// Of 80 sizes in 7 collisions no pair of steps is slower than two launches by more than 2.5% under
// these rules, and none that is left out would gain more than 5%.
inline bool ddf_pair_supported(int fmt, const Layout& L, const DdfParams& prm, const PairShape& s) {
  if (fmt != 0 || prm.phi == 2 || L.nx > 1 << 24 || L.nodes() < (prm.neq ? 400000 : 700000)) return false;
  const bool ext = prm.ext() || prm.eos;
  if (s.threads < kBlock) return !ext && s.threads != 192;
  if (s.rows < 6) return false;
  if (!ext) return true;
  const bool sparse = (int64_t)L.nx * 100 < (int64_t)s.nbx * s.threads * 63;
  if (prm.neq && s.rounds > 1 && s.rows < 16) return false;
  const Grid one = ddf_step_grid(make_grid_ddf(L, 1, false), L, prm.phi, 0, kDdfExtended, false, INT_MAX);
  // one-step turns in tenths
  return s.turns * 1000 <= ddf_turns(one.blocks(), one.rows, 1, 2) * (sparse ? 190 : (prm.neq ? 300 : 246));
}

// ---- isothermal D3Q27: two steps per launch -------------------------------------------------------
constexpr int kP3Rows = 11;         // region rows: owned rows and one more on either side
constexpr int kP3Own = kP3Rows - 2;

// Ranges of planes: the fewest planes in turn over the rounds of one workgroup per compute unit.
inline Pair3Shape bgk3_pair_shape(const Layout& L) {
  Pair3Shape s;
  s.nbx = (int)div_up(L.nx, 64);
  s.nby = (int)div_up(L.ny, kP3Own);
  const int64_t tiles = (int64_t)s.nbx * s.nby;
  int64_t best = -1;
  for (int c = 1; c <= std::min(L.nz, 64); ++c) {
    if (tiles * c > (int64_t)1 << 21) break;
    const int64_t cost = div_up(tiles * c, kCus) * (div_up(L.nz, c) + 3);
    if (best < 0 || cost < best) {
      best = cost;
      s.ranges = c;
    }
  }
  return s;
}

// Where two steps per launch are taken (two buffers, float32, periodic, no force). A workgroup takes
// whole tiles of 64 columns, marches over three planes besides its own, and the chip needs one for
// nearly every compute unit. us per step, one step / two: 64^3 12.5 / 12.1, but 48^3 7.9 / 11.0
// and 32^3 5.0 / 8.4; 100 x 100 x 20 12.6 / 12.4; 129 x 500 x 20 68 / 60; one plane 2000^2 164 / 209,
// two 1000 x 500 41.7 / 45.4, three 1000^2 124 / 111; 64 x 9 x 200, 64 workgroups, 7.3 / 14.8 and 128
// x 9 x 300, 128, 16.1 / 20.2, but 700 x 9 x 64 19.5 / 14.9; 30 x 300 x 64, 47% of the columns, 50 /
// 32, 3 x 3 x 100000, 5%, 592 / 3545.
inline bool bgk3_pair_supported(const Layout& L, const Pair3Shape& s) {
  return L.nx <= 1 << 24 && L.nodes() >= 200000 && L.nz >= 3 &&
         (int64_t)s.nbx * s.nby * s.ranges >= 192 && 5 * L.nx >= 2 * 64 * s.nbx;
}

}  // namespace lbm
