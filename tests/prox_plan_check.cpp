// Host check of how proximal maps are cut into launches (prox_plan.h): the
// parts cover every iteration, the windows keep something, and images are sent
// the way that measured faster.  Exit code 0 when every check holds.
#include <cstdio>

#include "../paper_1603_02329_amd/csrc/prox_plan.h"

using namespace pat;

static int fails = 0;
static void pays(int n0, int n1, int it, bool want) {
  ProxCost c(it);
  c.add(n0, n1);
  if (c.windows_pay() != want) std::printf("FAIL %d x %d, %d iterations: windows %d\n", n0, n1, it, !want), ++fails;
}

int main() {
  for (int n = 1; n < 200; ++n) {
    int k0, k1;
    prox_split(n, k0, k1);
    const int last = n - k1;
    const bool ok = k0 >= 1 && k0 <= k1 && k1 <= n && k0 <= kProxHalf && last <= kProxHalf &&
                    prox_keep_x(k0, k0 == n) > 0 && prox_keep_y(k0, k0 == n) > 0 &&
                    (k0 < n ? last >= 1 && prox_keep_x(last, true) > 0 && prox_keep_y(last, true) > 0 : k1 == n);
    if (!ok) std::printf("FAIL split of %d: %d %d\n", n, k0, k1), ++fails;
  }
  for (int it : {1, 2, 5, 10, 13, 20, 32, 40}) {
    pays(1, 1000000, it, false);
    pays(1000000, 1, it, false);
    pays(1000, 1000, it, true);
    pays(256, 256, it, true);
    pays(62500, 16, it, true);
  }
  for (int it : {5, 10, 20}) {
    pays(16, 62500, it, true);
    pays(30, 1024, it, true);
    pays(1024, 30, it, true);
    pays(4096, 4096, it, true);
    pays(4096, 1, it, true);
    pays(1, 4096, it, true);
    pays(250000, 4, it, true);
    pays(4, 250000, it, false);
    pays(2, 500000, it, false);
  }
  pays(1, 100000, 20, false);
  pays(100000, 1, 20, true);
  pays(8, 125000, 20, false);
  // images that run together are judged together
  ProxCost mixed(20);
  mixed.add(1, 1000000);
  for (int i = 0; i < 10; ++i) mixed.add(64, 64);
  if (mixed.windows_pay()) std::printf("FAIL mixed\n"), ++fails;
  if (!fails) std::printf("all checks passed\n");
  return fails != 0;
}
