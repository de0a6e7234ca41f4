// How the steps of a batch are divided into blocks (host arithmetic only).
#pragma once

#include <algorithm>
#include <cstdint>

namespace lbm {

// Steps of the next block, of the `left` ones of a call: a captured block of
// `graph` steps, or fewer.  span: the least steps that multi-step launches share
// (0: the batch takes one step per launch).  next_end(s): steps from now to the
// first end of a run's budget after s (INT64_MAX: none).
//
// Multi-step launches stop at a budget's end.  One-step launches look at the
// budgets themselves, so a batch without others is not cut there and replays
// whole graphs (64 channels of 24 rows, walls and none, that end one step apart:
// 860 steps 2.33 ms, cut at every end 2.42).  Pieces too short for multi-step
// launches are joined over the budgets that end that close together (64 channels
// of 40 rows in tiles 1.35 and 1.43).
template <typename NextEnd>
int64_t batch_block(int64_t left, int64_t graph, int64_t span, NextEnd next_end) {
  const int64_t blk = std::min(left, graph);
  if (span == 0) return blk;
  int64_t e = std::min(blk, next_end(0));
  if (e >= span) return e;
  while (e < blk) {
    const int64_t n = std::min(blk, next_end(e));
    if (n - e >= span) break;
    e = n;
  }
  return e;
}

}  // namespace lbm
