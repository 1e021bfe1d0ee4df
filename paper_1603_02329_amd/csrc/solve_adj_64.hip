// Resident adjoint solves with columns of 64 points (passes_solve.h).
#include "passes_solve.h"

namespace pat {
hipError_t launch_solve_adj_64(int nx, int lossy, const SolveArgs& a, hipStream_t st) {
  return launch_solve_nd<64, 1>(nx, lossy, a, st);
}
}  // namespace pat
