// Launch rules in plain C++ (host only), shared by the launches and the CPU tests.
#pragma once

#include <cstddef>

namespace cf {

// Most planes of one y-chunk of the split RK stages and the transposed stencil.
constexpr int kMaxChunk = 32;

// Planes per y-chunk of a marching kernel: `cols` column tiles, `slots` blocks
// on the chip at a time, `extra` plane times a chunk spends before its first
// plane.  The longest chunk within 4 % of the least rounds * (planes + extra): a
// grid of few columns is cut until its blocks fill the chip once, and one of many
// keeps long chunks (there the blocks do not run in rounds: FP64 split stages on
// 1024x256x512 in 29 instead of 32 planes, 0.5 % less by this count, are 4 %
// slower).
inline int chunk_planes(long cols, int ny, long slots, int max_planes, int extra) {
  const int top = max_planes < ny ? max_planes : ny;
  auto cost = [&](int cy) { return (cols * ((ny + cy - 1) / cy) + slots - 1) / slots * (cy + extra); };
  long least = cost(top);
  for (int cy = top - 1; cy >= 1; --cy) least = cost(cy) < least ? cost(cy) : least;
  for (int cy = top; cy > 1; --cy)
    if (100 * cost(cy) <= 104 * least) return cy;
  return 1;
}

// Threads per block (a pair of points each) of the pressure corrections.  Blocks
// are dealt to the 8 XCDs in turn, so where a row takes a multiple of 8 blocks the
// block with the z- or y-neighbours of a block's pressure is on the same XCD and
// finds them in its L2: rows of a multiple of 1024 points take 8 blocks of 64 to 256
// threads.  us of the two corrections of a step and its adjoint, 256 threads / this
// rule: 2048x256x1024 FP32 3477, 3504 / 3022, 3122 (one point per thread of 256 had
// 8 blocks too: 3376, 3128), 2048x768x2048 FP32 20493, 21001 / 19021, 19195,
// 2048x128x1024 FP64 2668, 2670 / 2450, 2562, 1024x256x512 FP64 1283, 1338 / 1228,
// 1259, FP32 781, 785 / 781, 779, 3072x64x512 FP64 995, 1028 / 997, 1012.  Blocks of
// 64 threads on shorter rows are slower (512x192x512 FP32 308, 303 / 319, 316).
inline int correction_threads(int nx) { return nx % 1024 == 0 && nx <= 4096 ? nx / 16 : 256; }

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
