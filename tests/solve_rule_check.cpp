// Host check of the resident solves' rules (solve_rule.h): what a wavefront, a
// workgroup and a domain hold, the solves that are left to launches, and the
// side that batches take.
// Exit code 0 when every check holds.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../paper_1603_02329_amd/csrc/solve_rule.h"

using namespace pat;

static int fails = 0;
#define CHECK(c, ...)                                                                   \
  do {                                                                                  \
    if (!(c)) std::printf("FAIL line %d: ", __LINE__), std::printf(__VA_ARGS__), ++fails; \
  } while (0)

// The batches measured on both sides (200 steps; us per step as resident solves
// and as launches): the rule takes the faster one wherever they differ by more
// than 15 %.  `shared`: the shapes share their launches.
struct Part {
  int count, nx, ny, steps, lossy;
};
static void batch(const std::vector<Part>& parts, bool shared, double resident, double launches) {
  BatchCost c;
  int longest = 0;
  for (const auto& p : parts) {
    for (int i = 0; i < p.count; ++i) c.instance(p.nx, p.ny, p.steps, p.lossy != 0);
    longest = std::max(longest, p.steps);
    if (!shared) c.set(p.steps, p.lossy != 0, false);
  }
  if (shared) c.set(longest, parts[0].lossy != 0, true);
  if (std::max(resident, launches) < 1.15 * std::min(resident, launches)) return;
  CHECK(c.resident_pays() == (resident < launches), "%d of %d x %d ...: %.1f and %.1f us estimated, %.1f and %.1f\n",
        parts[0].count, parts[0].nx, parts[0].ny, c.resident_us() / 200, c.launches_us() / 200, resident, launches);
}

static void batches() {
  for (int lossy = 0; lossy < 2; ++lossy) {
    const double f = lossy ? 1.0 : 0.68;
    for (int k : {1, 2, 4, 8, 16, 24}) {
      batch({{k, 32, 32, 200, lossy}}, false, 14.0 * f, 42.0 * f);
      batch({{k, 64, 64, 200, lossy}}, false, 13.5 * f, 43.0 * f);
      batch({{k, 128, 64, 200, lossy}}, false, (k > 16 ? 28.5 : 14.5) * f, 45.5 * f);
      batch({{k, 128, 128, 200, lossy}}, false, (k > 16 ? 49.8 : k > 8 ? 33.5 : 16.5) * f, 50.0 * f);
      batch({{k, 256, 64, 200, lossy}}, false, (k > 16 ? 48.6 : k > 8 ? 32.7 : 16.4) * f, 51.5 * f);
      batch({{k, 256, 256, 200, lossy}}, false, (k > 16 ? 73.1 : k > 8 ? 48.5 : 24.4) * f, (52.0 + 0.95 * k) * f);
    }
    for (int k : {1, 2, 4}) {
      batch({{k, 512, 256, 200, lossy}}, false, 27.3 * k * f, (k > 1 ? 62.0 : 54.6) * f);
      batch({{k, 512, 512, 200, lossy}}, false, 34.4 * k * f, (k > 2 ? 78.0 : k > 1 ? 72.0 : 62.7) * f);
    }
    batch({{1, 512, 512, 200, lossy}, {1, 256, 256, 100, lossy}}, true, 34.9 * f, 60.5 * f);
    batch({{1, 512, 512, 200, lossy}, {1, 128, 128, 200, lossy}}, true, 35.5 * f, 59.9 * f);
    batch({{4, 128, 128, 200, lossy}, {4, 256, 256, 200, lossy}}, true, 26.5 * f, 62.5 * f);
    batch({{8, 256, 256, 200, lossy}, {8, 64, 64, 200, lossy}}, false, 27.0 * f, 97.0 * f);
    batch({{6, 128, 128, 200, lossy}, {6, 128, 64, 200, lossy}, {6, 64, 64, 200, lossy}}, false, 20.8 * f, 95.0 * f);
    batch({{2, 64, 64, 200, lossy}, {2, 32, 32, 200, lossy}}, false, 14.0 * f, 84.3 * f);
    batch({{4, 32, 256, 100, lossy}, {2, 256, 32, 200, lossy}}, false, 7.9 * f, 49.0 * f);
    batch({{3, 512, 64, 200, lossy}, {3, 64, 512, 200, lossy}}, false, 23.5 * f, 102.5 * f);
    // 48 grids of three sizes, 100 steps of the smallest: launches by far
    batch({{16, 128, 128, 50, lossy}, {16, 256, 256, 100, lossy}, {16, 512, 512, 200, lossy}}, true, 680.0 * f, 145.0 * f);
  }
  batch({{2, 128, 128, 200, 1}, {2, 128, 128, 200, 0}}, false, 16.5, 69.3);
  batch({{4, 256, 256, 200, 1}, {4, 256, 256, 200, 0}}, false, 25.4, 84.2);
  // both physics of shapes that would share their launches: two sets
  BatchCost two, one;
  two.set(200, true, true);
  one.set(200, true, true);
  two.set(200, false, true);
  CHECK(two.launches_us() > 1.15 * one.launches_us(), "two sets cost more than one\n");
}

int main() {
  batches();
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
