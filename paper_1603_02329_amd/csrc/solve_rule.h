// Resident solves (passes_solve.h): which grids they take, how a grid's tiles
// are dealt to workgroups, and when they pay.  Host and constant expressions
// only, no HIP types.
#pragma once

#include <algorithm>
#include <vector>

namespace pat {

constexpr int kSolveXcds = 8;        // MI355X: 8 accelerator complex dies (XCDs), one L2 each
constexpr int kSolveCus = 32;        // compute units per die
constexpr int kSolveDomains = 16;    // most domains per die

// Grids above this run on one domain over every die, the others on one die.
// Per step (forward, lossy, calls of 400 steps), on one die and over all: 256^2
// 24.3 and 25.3 us; 512 x 128 24.0 and 24.1; 128 x 512 25.8 and 28.0; 512 x 256
// 46.7 and 26.7; 256 x 512 43.9 and 30.8; 512^2 80.9 and 33.5.
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

// domains per die for a queue with at most `deep` instances on a die
constexpr int solve_domains(int nx, int ny, int deep) {
  if (solve_whole(nx, ny)) return 1;
  const int most = std::min({deep, kSolveDomains, kSolveCus / solve_members(nx, ny)});
  return most < 1 ? 1 : most;
}

// Whether a batch's time loops run as resident solves: when their estimated
// time is below that of the batched launches (microseconds; measured from one
// to 64 instances of 32^2 to 512^2; the adjoint within 3 % of the forward,
// lossless steps 0.68 of lossy ones either way).
// A resident step takes 11.5 us + 0.17 us per 1000 points on its die, the dies
// working side by side and each holding 32 / members domains; over every die
// 20.5 us + 0.053 us per 1000 points and 20 us to start, one instance at a
// time.  The instances over every die and those on one run side by side too,
// at 0.4 of the shorter part's time.
// A step of the batched launches takes 42 us + 0.02 us per 1000 points of all
// its instances, 54 us where classes of several shapes share their launches
// (512^2 with 256^2 60 us, 4 of 128^2 with 4 of 256^2 65 us), and 0.71 of all
// sets' times where there are several (8 of 256^2 with 8 of 64^2 104 us, 6
// each of 128^2, 128 x 64 and 64^2 91 us, lossy and lossless 128^2 69 us).
class BatchCost {
 public:
  void instance(int nx, int ny, long steps, bool lossy) {
    const double w = weight(lossy) * (double)steps, kpts = 1e-3 * nx * ny;
    points_ += 0.02 * w * kpts;
    if (steps < 1) return;
    if (solve_whole(nx, ny)) {
      whole_ += 20.0 + w * (20.5 + 0.053 * kpts);
      return;
    }
    const double t = w * (11.5 + 0.17 * kpts);
    shares_.push_back(t * solve_members(nx, ny) / kSolveCus);
    for (auto& q : queues_)
      if (q.nx == nx && q.ny == ny && q.lossy == lossy) {
        ++q.n;
        q.longest = std::max(q.longest, t);
        return;
      }
    queues_.push_back(Queue{nx, ny, lossy, 1, t});
  }
  // one set of launches: the classes that step together
  void set(long steps, bool lossy, bool shared) {
    const double t = weight(lossy) * (double)steps * (shared ? 54.0 : 42.0);
    longest_set_ = std::max(longest_set_, t);
    sets_ += t;
  }
  double resident_us() const {
    double die[kSolveXcds] = {}, dies = 0;
    std::vector<double> s = shares_;
    std::sort(s.rbegin(), s.rend());
    for (double c : s) *std::min_element(die, die + kSolveXcds) += c;
    dies = *std::max_element(die, die + kSolveXcds);
    for (const auto& q : queues_) {
      const int deep = (q.n + kSolveXcds - 1) / kSolveXcds, d = solve_domains(q.nx, q.ny, deep);
      dies = std::max(dies, (deep + d - 1) / d * q.longest);
    }
    return std::max(whole_, dies) + 0.4 * std::min(whole_, dies);
  }
  double launches_us() const { return std::max(longest_set_, 0.71 * sets_) + points_; }
  bool resident_pays() const { return resident_us() < launches_us(); }

 private:
  struct Queue {
    int nx, ny;
    bool lossy;
    int n;
    double longest;
  };
  static double weight(bool lossy) { return lossy ? 1.0 : 0.68; }
  std::vector<Queue> queues_;
  std::vector<double> shares_;  // time on a die, by the share of it that the instance holds
  double whole_ = 0, points_ = 0, sets_ = 0, longest_set_ = 0;
};

}  // namespace pat
