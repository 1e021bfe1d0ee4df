// Host check of the resident solves' rules (solve_rule.h): what a wavefront, a
// workgroup and a domain hold, and the solves that are left to launches.
// Exit code 0 when every check holds.
#include <cstdio>

#include "../paper_1603_02329_amd/csrc/solve_rule.h"

using namespace pat;

static int fails = 0;
#define CHECK(c, ...)                                                                   \
  do {                                                                                  \
    if (!(c)) std::printf("FAIL line %d: ", __LINE__), std::printf(__VA_ARGS__), ++fails; \
  } while (0)

int main() {
  for (int nx = 32; nx <= 512; nx *= 2)
    for (int ny = 32; ny <= 512; ny *= 2) {
      CHECK(solve_shape(2, nx, ny), "%d x %d is no shape\n", nx, ny);
      const int m = solve_members(nx, ny), nw = solve_nw(nx, ny);
      CHECK(m >= 1 && m <= solve_cus(nx, ny) && nw >= 2 && nw <= 8, "%d x %d: %d members of %d\n", nx, ny, m, nw);
      CHECK(solve_whole(nx, ny) == (nx * ny > 256 * 256), "%d x %d: whole\n", nx, ny);
      // one step over every die is left to the launches, everything else is not
      CHECK(solve_pays(nx, ny, 1) == !solve_whole(nx, ny), "%d x %d: one step\n", nx, ny);
      CHECK(solve_pays(nx, ny, 2) && solve_pays(nx, ny, 2400), "%d x %d: more steps\n", nx, ny);
    }
  CHECK(!solve_shape(3, 64, 64) && !solve_shape(2, 16, 64) && !solve_shape(2, 64, 1024), "shapes\n");
  if (!fails) std::printf("all checks passed\n");
  return fails != 0;
}
