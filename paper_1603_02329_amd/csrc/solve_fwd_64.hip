// Resident forward solves with columns of 64 points (passes_solve.h).
#include "passes_solve.h"

namespace pat {
hipError_t launch_solve_fwd_64(int nx, int lossy, const SolveArgs& a, hipStream_t st) {
  return launch_solve_nd<64, 0>(nx, lossy, a, st);
}
}  // namespace pat
