// Several time steps of one channel in one pass over memory.
//
// A step reads and writes 19 values per node and runs at the rate of a
// device copy with half its arithmetic issue slots idle, so the way to a
// faster step is to move the state less often.  Here a wavefront takes a
// strip of columns, one lane per column, and marches along y: it pulls row r
// of the stored state, updates it (level 1), and updates row r - 1 a second
// time (level 2) from the level-1 rows r - 2, r - 1 and r, which it still
// holds in registers; only the last level is stored.  Values that move along
// x come from the neighbouring lanes.  Each level loses one column at either
// side of the strip and one row at either end of the march, which the
// neighbouring wavefronts compute again; wavefronts share no data, so there is
// no LDS.  A barrier in each row only keeps the strips of a block in step, so
// that the cache lines which neighbours share are still in the L2.
//
// Of a level's row the next level needs its planes in three consecutive
// rows: the five moving down at once (row r for row r - 1), the nine along
// the row one row later, the five moving up two rows later: 19 values per
// lane are carried between two levels.
//
// Measured on MI355X at 4096^2 (us a step, single steps against this kernel):
// FP32 storage 427 -> 242-269 from rest and 277-290 from a random state, now
// bound by its arithmetic: 520 VALU instructions per node update, the lanes
// and rows computed twice included, issue in 94% of the busy cycles at 2.1
// GHz, HBM at 3.4 TB/s.  FP64 storage 921 -> 296-299 (56 G node updates/s):
// 363 instructions, 60% of the issue slots at 2 wavefronts per SIMD, 4.9 TB/s,
// as fast as a device copy.  An odd width costs it little, as its stores leave
// through the L2: 3001 x 2110 in FP64 488 -> 124 us.
//
// Every level rounds its values to the storage type (with the random words
// of its own step index) and calls node_finish, as the single-step kernel
// does, so the result is that of single steps bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include "lks_common.hpp"

namespace lks {

// How a launch cuts the rows: groups of chunks, rows per chunk, and whether
// a group's blocks stay on one XCD.
struct RowCut {
  int rows = 0, groups = 0;
  bool by_xcd = false;
};

// A channel's march: the steps a launch may take (1: none go through
// launch_march) and the cut of its rows for 2, 3 and 4 of them, found at the
// first launch of each (up to 780 cuts are priced for tall, narrow channels).
struct MarchPlan {
  int most = 1;
  int units = kCardUnits; // compute units of the device
  RowCut cut[3];
};

struct MarchArgs {
  Geom geom;
  const Coef<double> *kd;
  int precision;      // LKS_FP64 or LKS_FP32
  int scheme;         // scheme_of the channel
  const void *src;
  void *dst;
  uint32_t *ctr;
  int parity;
  int steps;
  hipStream_t stream;
};

// MarchPlan::most of a channel.
int march_most(const Channel &c);

// Advance src by a.steps steps (2..most) into dst.
hipError_t launch_march(MarchPlan &plan, const MarchArgs &a);

} // namespace lks
