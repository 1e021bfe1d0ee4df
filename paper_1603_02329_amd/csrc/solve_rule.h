// Resident solves (passes_solve.h): which grids they take, how a grid's tiles
// are dealt to workgroups, and when they pay.  Host and constant expressions
// only, no HIP types.
#pragma once

namespace pat {

constexpr int kSolveXcds = 8;        // MI355X: 8 accelerator complex dies (XCDs), one L2 each
constexpr int kSolveCus = 32;        // compute units per die
constexpr int kSolveDomains = 16;    // most domains per die

// Grids above this run on one domain over every die, the others on one die.
// Per step (forward, lossy), on one die and over all: 256^2 22.9 and 25.8 us;
// 512 x 128 22.3 and 24.9; 128 x 512 24.7 and 28.5; 512 x 256 50.2 and 31.5,
// 512^2 87.6 and 39.5 (both before the barrier's words were spread).
constexpr int kSolveDiePoints = 65536;
constexpr bool solve_whole(int nx, int ny) { return nx * ny > kSolveDiePoints; }
// Rows and columns are carried by two lanes where the per-launch passes have
// one (PairStage): 4 values per lane; 8 for columns of 512 points, which would
// not fit one wavefront otherwise.
constexpr bool solve_pair_col(int ny) { return ny <= 256; }
// rows of nx points that one wavefront carries
constexpr int solve_rows(int nx) { return 512 / nx; }
// wavefronts that a row pass of both parts can use
constexpr int solve_waves(int nx, int ny) { return 2 * (ny / solve_rows(nx)); }
// compute units of a domain
constexpr int solve_cus(int nx, int ny) { return kSolveCus * (solve_whole(nx, ny) ? kSolveXcds : 1); }
// wavefronts per member: two at least (the two parts of a tile exchange
// through LDS), more once the tiles fill every compute unit
constexpr int solve_nw(int nx, int ny) {
  int nw = 2;
  while (nw < 8 && nw * solve_cus(nx, ny) < solve_waves(nx, ny)) nw *= 2;
  return nw;
}
// members the tiles keep busy, at most one per compute unit
constexpr int solve_members(int nx, int ny) {
  const int m = solve_waves(nx, ny) / solve_nw(nx, ny), cap = solve_cus(nx, ny);
  return m < 1 ? 1 : m < cap ? m : cap;
}

// whether there is a resident kernel for the grid
inline bool solve_shape(int ndim, int nx, int ny) {
  return ndim == 2 && nx >= 32 && nx <= 512 && ny >= 32 && ny <= 512;
}
// Whether `steps` of its time loop run as one resident solve: the workgroups of
// a domain over every die take some 20 us to meet and to form their
// multipliers, so one step alone is faster in launches of its own.  Forward,
// resident and launches (us, the whole call): one step of 512^2 lossy 78 and
// 71, lossless 64 and 52, 512 x 256 71 and 64, 61 and 48; two steps of 512^2
// 111 and 125, 87 and 88, 512 x 256 99 and 110, 80 and 80; one step of 256^2
// 52 and 57, 44 and 47, of 64^2 37 and 46, 32 and 38.
constexpr bool solve_pays(int nx, int ny, int steps) { return steps > 1 || !solve_whole(nx, ny); }

}  // namespace pat
