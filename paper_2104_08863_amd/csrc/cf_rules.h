// Launch rules in plain C++ (host only), shared by the launches and the CPU tests.
#pragma once

#include <cstddef>

namespace cf {

// Graphs a time loop replays: one step, one step with statistics, or two steps
// without.
enum LoopGraph { kOneStep, kStatsStep, kTwoSteps, kLoopGraphs };

// Whether step k of a loop (counted from 0) takes statistics.
inline bool loop_stats_at(int k, int stats_every) { return stats_every > 0 && (k + 1) % stats_every == 0; }

// The graph that runs step k, and step k + 1 when it is kTwoSteps.
inline LoopGraph loop_graph(int k, int nsteps, int stats_every) {
  if (loop_stats_at(k, stats_every)) return kStatsStep;
  return k + 1 < nsteps && !loop_stats_at(k + 1, stats_every) ? kTwoSteps : kOneStep;
}

// Graphs a plan keeps recorded.  A loop over one set of arrays and parameters
// replays at most five (two steps and the statistics step from either set of
// arrays, and a last single step), so two such loops in turn record nothing anew.
constexpr size_t kMaxGraphs = 10;

}  // namespace cf
