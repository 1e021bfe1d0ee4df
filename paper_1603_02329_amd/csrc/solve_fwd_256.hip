// Resident forward solves with columns of 256 points (passes_solve.h).
#include "passes_solve.h"

namespace pat {
hipError_t launch_solve_fwd_256(int nx, int lossy, const SolveArgs& a, hipStream_t st) {
  return launch_solve_nd<256, 0>(nx, lossy, a, st);
}
}  // namespace pat
