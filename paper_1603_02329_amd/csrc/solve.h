// Resident solves, host and device declarations (passes_solve.h).
#pragma once

#include "pat_internal.h"
#include "solve_rule.h"

namespace pat {

constexpr int kSolveQueue = 32768;   // most instances of a queue (16 bits hold a claim)
constexpr int kSolveSpin = 1 << 24;  // polls after which a wait gives up (seconds), if not set otherwise
constexpr uint32_t kSolveClosed = 0x80000000u;
// A domain whose members are held up (solves on other streams have their
// places) waits for them rather than run without: one missing of 256 doubles
// its time.  Solve time in ticks of the 100 MHz clock, 25 us a step; the wait
// ends after half a second in any case (before the others give up on it).
constexpr uint64_t kSolveRollTicks = 50000000;
constexpr uint32_t solve_ticks(long steps) { return steps > 10000 ? 25000000u : (uint32_t)(2500 * steps); }

// One domain: its roll, the instance its first member claimed, and the
// barrier's words: one per die, each on a line of its own (over every die:
// in every die's entry), and one per member, two on a line.  (Words on one line
// queue up at the L2 when all are stored and polled at once.  Per step, when the
// layout was chosen, the members' words 32, 8, 2 and 1 on a line: 128^2 17.6,
// 16.2, 15.3, 15.0 us, 256^2 26.1, 24.0, 23.1, 23.5; then the dies' words 8 and
// 1 on a line: 512^2 38.3 and 36.0.)
constexpr int kSolveLine = 32;  // words
constexpr int kSolveFlagLines = 16;
constexpr int solve_flag(int member) {
  return member % kSolveFlagLines * kSolveLine + member / kSolveFlagLines;
}
struct alignas(128) SolveDom {
  uint32_t roll, n, claim, ready;
  uint32_t count[kSolveXcds];  // members per die (domains over every die)
  alignas(128) uint32_t lead[kSolveXcds * kSolveLine];
  alignas(128) uint32_t flag[kSolveFlagLines * kSolveLine];  // (over every die: die x's are in the x-th entry)
};
struct alignas(128) SolveCtl {
  uint32_t ticket[kSolveXcds][32];  // blocks seen per die
  uint32_t head[kSolveXcds][32];    // next instance of each die's list
  alignas(128) uint32_t claimed;    // instances taken
};

struct SolveArgs {
  const DevPlan* const* list;  // queued instances, the dies' lists one after another
  const DevPlan* one;          // the instance when there is no list
  const Tw* tw;                // the global twiddle table
  SolveCtl* ctl;
  SolveDom* doms;              // [die][domains]; domains over every die: one
  int32_t first[kSolveXcds + 1];  // where each die's list begins
  int32_t members, domains;    // members per domain, domains per die
  int32_t s0, s1;
  uint32_t solve_ticks;
  int32_t polls;               // polls after which a wait gives up
};

// The kBadOpen word of an instance: set before the queue starts, then each of
// the n members of its domain adds its share once its own part of the time
// loop is done.  Zero again only if all of them came to the end.
constexpr uint32_t kSolveOpen = 0x10000;
constexpr uint32_t solve_share(int rank, int n) { return rank == 0 ? 0u - kSolveOpen - (uint32_t)(n - 1) : 1u; }

constexpr size_t solve_ctl_bytes(int domains) { return sizeof(SolveCtl) + sizeof(SolveDom) * kSolveXcds * domains; }

// clears the control block, marks the instances as open (open: the kBadOpen
// word of the one instance when there is no list) and runs the queue's time
// loops, all of one shape
hipError_t launch_solve(int nx, int ny, int dir, int lossy, SolveArgs a, int32_t* open, hipStream_t st);

}  // namespace pat
