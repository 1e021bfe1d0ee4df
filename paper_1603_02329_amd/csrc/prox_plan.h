// How a proximal map of n_iter FGP iterations is cut into launches (host code
// only): several iterations per launch on windows of a 2D image (aux.hip,
// k_prox_steps), or two launches an iteration.
#pragma once

#include <algorithm>

namespace pat {

constexpr int kProxWaves = 16, kProxRows = 3, kProxH = kProxWaves * kProxRows;

// Columns and rows that a launch of k iterations keeps of a window (64 x
// kProxH); one less where it ends in the result.
inline int prox_keep_x(int k, bool last) { return 64 - 2 * k - last; }
inline int prox_keep_y(int k, bool last) { return kProxH - 2 * k - last; }
inline long prox_tiles(int n0, int n1, int tx, int ty) {
  return (long)((n0 + tx - 1L) / tx) * ((n1 + ty - 1L) / ty);
}

// [0, k0) and [k1, n_iter) run in one launch each, [k0, k1) two launches an
// iteration: the workspace holds one copy of r and p_prev, which launches of
// several iterations cannot update in place.  Up to 12 iterations one launch
// is faster than two (14 iterations at 512^2: 31.9 us in one, 27.8 in two);
// in halves a launch may take up to 16 (30 iterations: 67 us; 111 with at
// most 12 and the rest two launches an iteration).
constexpr int kProxOne = 12, kProxHalf = 16;
inline void prox_split(int n_iter, int& k0, int& k1) {
  k0 = n_iter <= kProxOne ? n_iter : std::min(kProxHalf, (n_iter + 1) / 2);
  k1 = std::max(k0, n_iter - kProxHalf);
}

// Whether the windows are the faster way for a set of images that run
// together: a window costs much the same however little of it is image, so
// thin images fill the chip with windows that keep few points.  A window takes
// 5.5 ns of the whole chip's time and 0.8 to 3.5 ns per iteration (a row, and
// all the rows it keeps); two launches of one iteration 8 us, or 15.5 ns per
// 1000 points.  20 iterations of 10^6 points, windows and launches (us), n0 x
// n1: 1000^2 102 and 373; 62500 x 16 95 and 369, 16 x 62500 213 and 337;
// 125000 x 8 118 and 344, 8 x 125000 387 and 331; 500000 x 2 365 and 353; 10^6
// x 1 668 and 300, 1 x 10^6 2845 and 304.  10^5 points: 10^5 x 1 86 and 155, 1
// x 10^5 324 and 160.  One iteration: 10^6 x 1 107 and 41.
struct ProxCost {
  double window_ns = 0, points = 0;
  int n_iter;
  explicit ProxCost(int n) : n_iter(n) {}
  void add(int n0, int n1) {
    int k0, k1;
    prox_split(n_iter, k0, k1);
    add_launch(n0, n1, k0, k0 == n_iter);
    if (k1 < n_iter) add_launch(n0, n1, n_iter - k1, true);
    points += (double)n0 * n1;
  }
  bool windows_pay() const {
    int k0, k1;
    prox_split(n_iter, k0, k1);
    return window_ns < (n_iter - (k1 - k0) + 1) * std::max(8000.0, 0.0155 * points);
  }

 private:
  void add_launch(int n0, int n1, int k, bool last) {
    const int ty = prox_keep_y(k, last);
    window_ns += (double)prox_tiles(n0, n1, prox_keep_x(k, last), ty) *
                 (5.5 + k * (0.8 + 2.7 * std::min(1.0, (double)n1 / ty)));
  }
};

}  // namespace pat
