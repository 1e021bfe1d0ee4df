// Resident adjoint solves with columns of 32 points (passes_solve.h).
#include "passes_solve.h"

namespace pat {
hipError_t launch_solve_adj_32(int nx, int lossy, const SolveArgs& a, hipStream_t st) {
  return launch_solve_nd<32, 1>(nx, lossy, a, st);
}
}  // namespace pat
